// fp32 products on the bf16 matrix instruction.
//
// v_mfma_f32_16x16x4_f32 does 32 multiply-adds per SIMD and cycle, v_mfma_f32_16x16x32_bf16 sixteen times as many.  An
// fp32 value is the sum of three bf16 values exactly (24 bits of mantissa, 8 each):
//     x = h + m + l,   h = x truncated to 8 bits,  m = x - h rounded to 8,  l = x - h - m.
// Of the nine products of two such sums the three below 2^-23 of the whole are dropped (m*l, l*m, l*l); the other six
// cost 6 x 16 cycles for 32 channels where the fp32 instruction takes 8 x 32.
//
// Precision.  What an fp32 sum loses is in the roundings of the accumulator, one per instruction and 4 channels.  Here h*h,
// which holds all but the last 7 bits of a product, goes to an accumulator of its own, rounded once or twice per 32
// channels, and the five small products to a second one, whose roundings are 2^-7 of that; they are added at the end.
// Relative error (2-norm) of random sums against 64 bits, fp32 instruction / this: K = 32 6.3e-8 / 3.8e-8, 576
// 2.5e-7 / 0.9e-7, 4608 7.1e-7 / 2.9e-7; a sum that is split over four accumulators before (the K-split kernels): 5.4e-8,
// 1.3e-7, 3.5e-7.  (All six into one accumulator would be less precise than the fp32 instruction: 3.3e-7 at 576.)
// An infinite value has h = itself and NaN for m and l: the sum of h*h alone is then the result (split_sum).  Limits: a signalling
// NaN whose payload lies in its low 16 bits has an infinite h; l of a value below 2^-110 is subnormal or lost.
#pragma once
#include "dtypes.h"
#include "mma.h"

namespace rtoss {

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

// The six products, smallest first, as steps 0..5 so that a caller can interleave several accumulators.
template <int STEP> __device__ __forceinline__ void split_step(const Split8& a, const Split8& b, f32x4& main, f32x4& small)
{
    if constexpr (STEP == 0) small = Dense16<bf16_t>::mma(a.l, b.h, small);
    if constexpr (STEP == 1) small = Dense16<bf16_t>::mma(a.h, b.l, small);
    if constexpr (STEP == 2) small = Dense16<bf16_t>::mma(a.m, b.m, small);
    if constexpr (STEP == 3) small = Dense16<bf16_t>::mma(a.m, b.h, small);
    if constexpr (STEP == 4) small = Dense16<bf16_t>::mma(a.h, b.m, small);
    if constexpr (STEP == 5) main = Dense16<bf16_t>::mma(a.h, b.h, main);
}
constexpr int kSplitSteps = 6;

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
