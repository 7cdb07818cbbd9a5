// fp32 products on the bf16 matrix instruction.
//
// v_mfma_f32_16x16x4_f32 does 32 multiply-adds per SIMD and cycle, v_mfma_f32_16x16x32_bf16 sixteen times as many.  An
// fp32 value is the sum of three bf16 values exactly (24 bits of mantissa, 8 each):
//     x = h + m + l,   h = x truncated to 8 bits,  m = x - h rounded to 8,  l = x - h - m.
// Of the nine products of two such sums l*l, below 2^-32 of the whole, is dropped, and m*l and l*m, up to 2^-23 of it each, only
// where a sum has products enough (few_live_products); six cost 6 x 16 cycles for 32 channels where the fp32 instruction
// takes 8 x 32.
//
// Precision.  What an fp32 sum loses is in the roundings of the accumulator, one per instruction and 4 channels or more.  Here h*h,
// which holds all but the last 7 bits of a product, goes to an accumulator of its own, rounded once or twice per 32
// channels, and the small products to a second one, whose roundings are 2^-7 of that; they are added at the end.
// Relative error (2-norm) of random sums against 64 bits, fp32 instruction / six products: K = 32 6.3e-8 / 3.8e-8, 576
// 2.5e-7 / 0.9e-7, 4608 7.1e-7 / 2.9e-7; a sum that is split over four accumulators before (the K-split kernels): 5.4e-8,
// 1.3e-7, 3.5e-7.  (All six into one accumulator would be less precise than the fp32 instruction: 3.3e-7 at 576.)
// Short sums have few roundings to save, and the dropped m*l and l*m count in full.  1x1 kernels with k live weights per group,
// 2-norm and (largest error in 2^-24 of the sum of magnitudes), fp32 instruction / six / eight products:
//     Ci =  1, k = 2 (0-1 live)  2.5e-8 (1.0) / 3.7e-8 (3.6) / 2.5e-8 (1.0)     Ci = 20, k = 2 (4.4)  4.2e-8 (3.0) / 3.4e-8 (3.3) / 2.6e-8 (2.2)
//     Ci =  8, k = 2 (1.8)       3.3e-8 (2.5) / 3.5e-8 (4.0) / 2.5e-8 (2.1)     Ci = 48, k = 2 (11)   6.1e-8 (3.2) / 3.5e-8 (1.7) / 2.7e-8 (1.8)
// where half of the activations are zero (ReLU):
//     Ci =  8, k = 2             3.0e-8 (2.3) / 3.5e-8 (3.9) / 2.5e-8 (1.9)     Ci = 24, k = 5 (13)   5.1e-8 (3.2) / 3.5e-8 (3.5) / 2.7e-8 (2.3)
//     Ci = 40, k = 2 (8.9)       4.3e-8 (2.9) / 3.4e-8 (3.6) / 2.6e-8 (2.2)     Ci = 72, k = 2 (16)   5.5e-8 (3.7) / 3.4e-8 (3.0) / 2.7e-8 (2.6)
// (At two to four live products the largest error of eight is 2.3 where the fp32 instruction's is 1.9, with the smaller 2-norm: the
// sum of h*h and the last addition round once each.)
// An infinite value has h = itself and NaN for m and l: the sum of h*h alone is then the result (split_sum).  Limits: a signalling
// NaN whose payload lies in its low 16 bits has an infinite h (quieting every value first: 3x3 64 -> 64 on 80x80 7.2 -> 7.5 us, 96 -> 96
// on 2x80x100 25.5 -> 26.9, 256 -> 256 on 4x80x80 130.9 -> 133.9; activations are finite by contract); l of a value below 2^-110 is
// subnormal or lost.
#pragma once
#include "common.h"
#include "dtypes.h"
#include "mma.h"

namespace rtoss {

// Whether six products would be less precise than the fp32 instruction, in the 2-norm or in the largest error: 1x1 sums of fewer than
// some 14 live products (k of 9 input channels) then take eight, 3x3 sums of fewer than 24 (Ci * k; four ninths of that in a
// corner of the image) the fp32 instruction, which for so few channels is 6 % (stride 1) and 20 % (stride 2) slower.
inline bool few_live_products(const rtoss_wdesc& d) { return d.Ci * d.k < (d.ksize == 1 ? 128 : 24); }

// The bf16 parts of eight fp32 values, as operands of v_mfma_f32_16x16x32_bf16.
struct Split8 {
    u32x4 h, m, l;
};

__device__ __forceinline__ void split2(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l)
{
    const uint32_t ua = __builtin_bit_cast(uint32_t, a), ub = __builtin_bit_cast(uint32_t, b);
    h = __builtin_amdgcn_perm(ub, ua, 0x07060302u);
    const float ra = a - __builtin_bit_cast(float, ua & 0xffff0000u), rb = b - __builtin_bit_cast(float, ub & 0xffff0000u);
    m = pack2_from_f32<bf16_t>(ra, rb);
    l = pack2_from_f32<bf16_t>(ra - __builtin_bit_cast(float, m << 16), rb - __builtin_bit_cast(float, m & 0xffff0000u));
}

// (values in the order of a lane's K slots: any order will do as long as both operands use it)
__device__ __forceinline__ Split8 split8(u32x4 first, u32x4 second)
{
    Split8 s;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const f32x4 v = __builtin_bit_cast(f32x4, i < 2 ? first : second);
        uint32_t h, m, l;
        split2(v[2 * (i & 1)], v[2 * (i & 1) + 1], h, m, l);
        s.h[i] = h;
        s.m[i] = m;
        s.l[i] = l;
    }
    return s;
}

// The products, smallest first, in steps so that a caller can interleave several accumulators: all eight, or the last six.
constexpr int kSplitAll = 8, kSplitSix = 6;
template <int STEP> __device__ __forceinline__ void split_step(const Split8& a, const Split8& b, f32x4& main, f32x4& small)
{
    if constexpr (STEP == 0) small = Dense16<bf16_t>::mma(a.l, b.m, small);
    if constexpr (STEP == 1) small = Dense16<bf16_t>::mma(a.m, b.l, small);
    if constexpr (STEP == 2) small = Dense16<bf16_t>::mma(a.l, b.h, small);
    if constexpr (STEP == 3) small = Dense16<bf16_t>::mma(a.h, b.l, small);
    if constexpr (STEP == 4) small = Dense16<bf16_t>::mma(a.m, b.m, small);
    if constexpr (STEP == 5) small = Dense16<bf16_t>::mma(a.m, b.h, small);
    if constexpr (STEP == 6) small = Dense16<bf16_t>::mma(a.h, b.m, small);
    if constexpr (STEP == 7) main = Dense16<bf16_t>::mma(a.h, b.h, main);
}
template <int STEPS, typename F> __device__ __forceinline__ void split_steps(F&& f)
{
    static_for<STEPS>([&](auto i) { f(std::integral_constant<int, kSplitAll - STEPS + decltype(i)::value>{}); });
}

// The result.  Infinite terms stand in `main` with their signs and make `small` NaN (inf - inf when split, inf * 0), so an
// infinite `main` is the result as it is; terms of both signs, 0 * inf and NaN have made `main` NaN.
__device__ __forceinline__ f32x4 split_sum(f32x4 main, f32x4 small)
{
    f32x4 sum = main + small;
#pragma unroll
    for (int e = 0; e < 4; ++e) sum[e] = __builtin_isinf(main[e]) ? main[e] : sum[e];
    return sum;
}

}  // namespace rtoss
