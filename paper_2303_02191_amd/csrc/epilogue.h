// Fused output stage shared by the convolution kernels:
//     y = act(scale[co] * conv + bias[co]) + residual
// (a folded batch normalisation, the activation and a shortcut connection of the detector
// blocks the pruned layers sit in; Section V reports whole-model inference).  All arithmetic is
// fp32; the result is rounded once when it is stored.
#pragma once
#include <type_traits>

#include "common.h"
#include "dtypes.h"
#include "mma.h"
#include "row_pieces.h"

namespace rtoss {

struct Epilogue {
    const float* scale;    // [Co] or nullptr (= 1); 16-byte aligned
    const float* bias;     // [Co] or nullptr (= 0); 16-byte aligned
    const void* residual;  // tensor of the output's type and shape, or nullptr
    int act;               // rtoss_act: 0 none, 1 ReLU, 2 SiLU
    // Channels-last tensors: elements from one position's channel 0 to the next position's.  Co for a plain
    // tensor; larger when the convolution writes (or the shortcut reads) a channel slice of a wider buffer,
    // e.g. its part of a concatenation (the slice's first channel is folded into the pointer).
    int ldy;               // of the output
    int ldr;               // of the residual
};

struct ConvParams : rtoss_cdesc {
    Epilogue ep;
    DeviceInfo dev;  // asked for once per call
};

// Stores in whole rows are 32-bit offsets from a position, of up to 64 positions from there: an output pitch that passes them takes a
// kernel that stores at 64-bit addresses.
inline bool stores_in_reach(const ConvParams& c) { return (int64_t)c.ep.ldy * 64 * elem_bytes(c.out_dt) < kNoStore; }

template <typename TO> __device__ __forceinline__ u32x4 pack8_from_f32(const float* v)
{
    u32x4 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = pack2_from_f32<TO>(v[2 * i], v[2 * i + 1]);
    return o;
}

// v[i] / (1 + exp(-v[i])), each quotient correctly rounded, whatever type the result is stored in.
//
// The IEEE division is ten vector instructions, four cycles each, and would be most of the output stage (a 57-layer
// forward, batch 16: 944 us, against 861 with the form below).  The hardware reciprocal (1 ulp) alone is cheaper and not exact:
// 2.4 % of all floats v come out one ulp off.  One correction with the quotient's own remainder (Markstein, IBM J. Res.
// Dev. 34, 1990) makes up for that: compared with the division for every one of the 2^32 values of v on the device, no bit
// differs.  That holds while nothing in between leaves the normal range, so runs with a large |v| take the division.
// (The remainder is formed as d * q - v: with the other sign -0 would turn into +0.)
constexpr float kSiluInRange = 80.f;  // the largest |v| that takes the corrected reciprocal
__device__ __forceinline__ float silu_divided(float v) { return v / (1.f + __expf(-v)); }
// (d: 1 + exp(-v); r: its reciprocal)
__device__ __forceinline__ float silu_corrected(float v, float d, float r)
{
    const float q = v * r;
    return __builtin_fmaf(-__builtin_fmaf(d, q, -v), r, q);
}
template <int N> __device__ __forceinline__ void epi_silu(float (&v)[N])
{
    float top = 0.f;
#pragma unroll
    for (int i = 0; i < N; ++i) top = __builtin_fmaxf(top, __builtin_fabsf(v[i]));  // (a NaN stays one either way)
    if (__builtin_expect(__ballot(top > kSiluInRange) != 0, 0)) {  // (the whole wave: a scalar branch)
#pragma unroll
        for (int i = 0; i < N; ++i) {
            asm volatile("" : "+v"(v[i]));  // keeps the exponentials, which both sides need, from being held across the branch
            v[i] = silu_divided(v[i]);
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const float d = 1.f + __expf(-v[i]);
        v[i] = silu_corrected(v[i], d, __builtin_amdgcn_rcpf(d));
    }
}
// The same in N + 2 parts without a branch, for kernels that put matrix instructions between them, and an end: part J takes value
// J's exponential, the reciprocal of the value before and the quotient of the one before that; the end divides where that
// does not hold.
template <int J, int N>
__device__ __forceinline__ void epi_silu_part(const float (&u)[N], float (&v)[N], float (&d)[N], float& top)
{
    if constexpr (J < N) {
        top = __builtin_fmaxf(top, __builtin_fabsf(u[J]));
        d[J] = 1.f + __expf(-u[J]);
    }
    if constexpr (J >= 1 && J - 1 < N) v[J - 1] = __builtin_amdgcn_rcpf(d[J - 1]);
    if constexpr (J >= 2) v[J - 2] = silu_corrected(u[J - 2], d[J - 2], v[J - 2]);
}
template <int N> __device__ __forceinline__ void epi_silu_end(const float (&u)[N], float (&v)[N], float top)
{
#pragma unroll
    for (int i = 0; i < N; ++i) asm volatile("" : "+v"(v[i]));  // keeps the parts in front of the branch
    if (__builtin_expect(__ballot(top > kSiluInRange) != 0, 0)) {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = silu_divided(u[i]);
    }
}
// (one uniform branch per activation around the whole run, not one per value)
template <int N> __device__ __forceinline__ void epi_act(float (&v)[N], int act)
{
    if (act == 1) {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = __builtin_fmaxf(v[i], 0.f);
    } else if (act == 2) {
        epi_silu<N>(v);
    }
}

// v[0..N) are N consecutive output channels, starting at channel co, of one position (N and co are
// multiples of 4).  Scale, bias and activation; the branches are uniform over the launch.  `scale` and `bias` point at
// the run's first channel (in device memory, or at a copy in LDS) and are read only where ep has them.
template <int N>
__device__ __forceinline__ void epi_scale_bias(float (&v)[N], const Epilogue& ep, const float* scale, const float* bias)
{
    static_assert(N % 4 == 0, "runs of 4 channels");
    if (ep.scale) {
#pragma unroll
        for (int g = 0; g < N / 4; ++g) {
            const f32x4 s = *(const f32x4*)(scale + 4 * g);
#pragma unroll
            for (int i = 0; i < 4; ++i) v[4 * g + i] *= s[i];
        }
    }
    if (ep.bias) {
#pragma unroll
        for (int g = 0; g < N / 4; ++g) {
            const f32x4 b = *(const f32x4*)(bias + 4 * g);
#pragma unroll
            for (int i = 0; i < 4; ++i) v[4 * g + i] += b[i];
        }
    }
}
template <int N>
__device__ __forceinline__ void epi_scale_bias_act(float (&v)[N], const Epilogue& ep, const float* scale, const float* bias)
{
    epi_scale_bias<N>(v, ep, scale, bias);
    epi_act<N>(v, ep.act);
}
template <int N> __device__ __forceinline__ void epi_scale_bias_act(float (&v)[N], const Epilogue& ep, int co)
{
    epi_scale_bias_act<N>(v, ep, ep.scale + co, ep.bias + co);
}

// The forms of the stage that a kernel may have code of its own for, chosen once per workgroup (epi_by_form): nothing at all, the
// folded normalisation with SiLU (scale and bias in one rounding), and everything else.  A branch around a run of values costs
// a copy of every value where its paths meet, a quarter of the instructions of a short output loop (3 -> 32 channels on
// 16x640x640, where the vector instructions bound the kernel: 42.4 us with the branches inside, 38.3; a 1x1 of 400 positions 3.3 and 3.0).
// NONE: a form for nothing at all, where the plain convolution gains too (1x1, 8x80x80 128 -> 128: 12.1 and 11.5 us).
enum EpiForm { kEpiAny = 0, kEpiNone, kEpiSilu };
template <bool NONE = true, typename F> __device__ __forceinline__ void epi_by_form(const Epilogue& ep, F&& run)
{
    if (ep.act == 2 && ep.scale && ep.bias) run(std::integral_constant<int, kEpiSilu>{});
    else if (NONE && ep.act == 0 && !ep.scale && !ep.bias) run(std::integral_constant<int, NONE ? kEpiNone : kEpiAny>{});
    else run(std::integral_constant<int, kEpiAny>{});
}
template <int FORM, int N>
__device__ __forceinline__ void epi_scale_bias_of(float (&v)[N], const Epilogue& ep, const float* scale, const float* bias)
{
    if constexpr (FORM == kEpiSilu) {
#pragma unroll
        for (int g = 0; g < N / 4; ++g) {
            const f32x4 s = *(const f32x4*)(scale + 4 * g), b = *(const f32x4*)(bias + 4 * g);
#pragma unroll
            for (int i = 0; i < 4; ++i) v[4 * g + i] = __builtin_fmaf(v[4 * g + i], s[i], b[i]);
        }
    } else if constexpr (FORM == kEpiAny) {
        epi_scale_bias<N>(v, ep, scale, bias);
    }
}
template <int FORM, int N>
__device__ __forceinline__ void epi_scale_bias_act_of(float (&v)[N], const Epilogue& ep, const float* scale, const float* bias)
{
    epi_scale_bias_of<FORM, N>(v, ep, scale, bias);
    if constexpr (FORM == kEpiSilu) epi_silu<N>(v);
    else if constexpr (FORM == kEpiAny) epi_act<N>(v, ep.act);
}

// Adds the residual's N consecutive channels, starting at channel co, of position number `pos` (n, oh, ow
// flattened) (8-byte aligned runs for 16-bit types, 16-byte aligned for fp32).
template <typename TO, int N> __device__ __forceinline__ void epi_residual(float (&v)[N], const Epilogue& ep, int64_t pos, int co)
{
    static_assert(N % 4 == 0, "runs of 4 elements");
    if (!ep.residual) return;
    const TO* r = (const TO*)ep.residual + pos * ep.ldr + co;
#pragma unroll
    for (int g = 0; g < N / 4; ++g) {
        if constexpr (sizeof(TO) == 4) {
            const f32x4 t = *(const f32x4*)(r + 4 * g);
#pragma unroll
            for (int i = 0; i < 4; ++i) v[4 * g + i] += t[i];
        } else {
            TO t[4];
            *(uint2*)t = *(const uint2*)(r + 4 * g);
#pragma unroll
            for (int i = 0; i < 4; ++i) v[4 * g + i] += to_f32(t[i]);
        }
    }
}

// The same in two steps for kernels that have something to do while the shortcut is on its way: N channels of the
// residual as they lie in memory, and their addition.
template <typename TO, int N> struct EpiResidual {
    static constexpr int kWords = N * (int)sizeof(TO) / 4;
    uint32_t w[kWords];
    __device__ __forceinline__ void load(const Epilogue& ep, int64_t pos, int co)
    {
        const char* r = (const char*)((const TO*)ep.residual + pos * ep.ldr + co);
#pragma unroll
        for (int g = 0; g < kWords / 4; ++g) *(u32x4*)(w + 4 * g) = *(const u32x4*)(r + 16 * g);
        if constexpr (kWords % 4 == 2) *(uint2*)(w + kWords - 2) = *(const uint2*)(r + 4 * (kWords - 2));
    }
    __device__ __forceinline__ void add(float (&v)[N]) const
    {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            if constexpr (sizeof(TO) == 4) {
                v[i] += __builtin_bit_cast(float, w[i]);
            } else {
                TO t;
                t.bits = (uint16_t)(w[i / 2] >> (16 * (i & 1)));
                v[i] += to_f32(t);
            }
        }
    }
};

// Scale and bias of the N <= 256 channels of a workgroup of 256 lanes, copied to LDS ([0, N) scale, [N, 2N) bias;
// nothing where ep has none), so that the output stage reads LDS instead of memory no one has touched yet behind the
// last matrix instruction.  In two steps: load() goes in front of a kernel's own first loads, store() behind the wait
// for those, before a barrier.
template <int N> struct EpiScaleBias {
    static_assert(N <= 256, "one channel per lane");
    static constexpr int kBytes = 8 * N;
    float s = 0.f, b = 0.f;
    __device__ __forceinline__ void load(const Epilogue& ep, int co0, int Co, int tid)
    {
        if (!(ep.scale || ep.bias)) return;  // uniform, here and below: a plain convolution pays one branch
        const bool mine = tid < N && co0 + tid < Co;
        if (ep.scale && mine) s = ep.scale[co0 + tid];
        if (ep.bias && mine) b = ep.bias[co0 + tid];
    }
    __device__ __forceinline__ void store(float* lds, const Epilogue& ep, int tid) const
    {
        if (!(ep.scale || ep.bias)) return;
        if (tid < N) {
            lds[tid] = s;
            lds[N + tid] = b;
        }
    }
};

// The whole output stage for a run of N channels of which only those below Co exist (layers whose channel count is
// no multiple of a matrix tile): element by element, nothing past channel Co is read.
template <typename TO, int N> __device__ __forceinline__ void epi_ragged(float (&v)[N], const Epilogue& ep, int64_t pos, int co, int Co)
{
#pragma unroll
    for (int i = 0; i < N; ++i) {
        if (co + i >= Co) break;
        if (ep.scale) v[i] *= ep.scale[co + i];
        if (ep.bias) v[i] += ep.bias[co + i];
    }
    epi_act<N>(v, ep.act);
    if (!ep.residual) return;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        if (co + i >= Co) break;
        v[i] += to_f32(((const TO*)ep.residual)[pos * ep.ldr + co + i]);
    }
}

// ... and its store.  `yp` is the position's channel 0.  Whole runs of rows whose pitch keeps them aligned go out as
// vectors (16-bit types: N % 4 == 0, 8 bytes at a time), anything else element by element.
template <typename TO, int N> __device__ __forceinline__ void store_ragged(TO* yp, const float (&v)[N], int co, int Co, int ldy)
{
    if (co + N <= Co && ldy % 4 == 0) {
#pragma unroll
        for (int g = 0; g < N / 4; ++g) {
            if constexpr (sizeof(TO) == 4) {
                *(f32x4*)(yp + co + 4 * g) = f32x4{v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
            } else {
                uint2 o;
                o.x = pack2_from_f32<TO>(v[4 * g], v[4 * g + 1]);
                o.y = pack2_from_f32<TO>(v[4 * g + 2], v[4 * g + 3]);
                *(uint2*)(yp + co + 4 * g) = o;
            }
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < N; ++i)
        if (co + i < Co) store_from_f32<TO>(yp + co + i, v[i]);
}

// Lanes 2i and 2i + 1 hold 16 channels each of two positions side by side, in two pieces of 16 bytes.  Exchanged between them, so that `a` is piece
// lane % 2 of the even position and `b` of the odd one, and four such pairs with neighbouring channels store rows of 128 bytes, without
// a detour through LDS and the barrier in front of it.  All lanes of the wave take part.
__device__ __forceinline__ void pair_pieces(u32x4& a, u32x4& b, bool odd)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t away = odd ? a[i] : b[i];
        const uint32_t here = (uint32_t)__builtin_amdgcn_mov_dpp((int)away, 0xb1, 0xf, 0xf, true);  // quad_perm: lane ^ 1
        a[i] = odd ? here : a[i];
        b[i] = odd ? b[i] : here;
    }
}

// A lane's run of 16 channels in 16 bits.
template <typename TO> struct Run16 {
    u32x4 half[2];
    __device__ __forceinline__ explicit Run16(const float (&v)[16]) : half{pack8_from_f32<TO>(v), pack8_from_f32<TO>(v + 8)} {}
    __device__ __forceinline__ void store(TO* yp) const
    {
        *(u32x4*)yp = half[0];
        *(u32x4*)(yp + 8) = half[1];
    }
};

// Output of a tile of 16 positions x 64 channels (16-bit, 2 KB) by one wave in whole rows: put() takes a lane's run of 16 channels (position
// lane % 16, run lane / 16), store() writes the tile 16 bytes a lane, eight lanes to a row of 128 bytes.  `area` is the wave's own.
template <typename TO> struct RowTile {
    static constexpr int kBytes = 2048;
    static __device__ __forceinline__ int chunk_at(int row, int c) { return (row * 8 + (c ^ ((row >> 1) & 7))) * 16; }
    static __device__ __forceinline__ void put(char* area, int lane, const Run16<TO>& run) { put(area, lane, run.half[0], run.half[1]); }
    static __device__ __forceinline__ void put(char* area, int lane, u32x4 a, u32x4 b)
    {
        *(u32x4*)(area + chunk_at(lane & 15, (lane >> 4) * 2)) = a;
        *(u32x4*)(area + chunk_at(lane & 15, (lane >> 4) * 2 + 1)) = b;
    }
    // offset(row, chunk): in bytes from base, or kNoStore
    template <typename F> static __device__ __forceinline__ void store(const char* area, int lane, __amdgpu_buffer_rsrc_t base, F&& offset)
    {
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            const int row = 8 * g + (lane >> 3), c = lane & 7;
            store16_through(base, offset(row, c), *(const u32x4*)(area + chunk_at(row, c)));
        }
    }
};

}  // namespace rtoss
