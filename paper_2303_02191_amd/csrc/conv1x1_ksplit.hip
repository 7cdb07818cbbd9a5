// 1x1 pattern-pruned convolution for launches too small for the streaming kernel: the input channels are split over the
// waves of a workgroup and every operand is loaded once, straight into registers.  Reads the streaming kernel's packed
// section (pack_plan.h).
//
// What bounds these launches (a few hundred to a few thousand positions of 128 to 1024 channels) is latency: the
// streaming kernel first loads a workgroup's weights -- up to 128 KB, for as little as two buffers of activations -- and
// then hands buffers of 16 positions through LDS, one barrier each.  Here a workgroup owns a tile of 16*TM channels x
// 16*TN positions, wave v takes stages v, v + 4, ... of 64 bytes of input channels, and a lane's operands (16 bytes of a
// fragment, 16 bytes of a position) are what the matrix instruction takes: no LDS, no barrier, all of a wave's loads in
// flight at once.  The four partial sums meet in LDS, where each lane picks up the runs of channels it stores.
// Measured, 512 -> 256 channels on 400 positions in fp16: 3.0 us, against 4.8 us.
#include <algorithm>

#include "common.h"
#include "dtypes.h"
#include "epilogue.h"
#include "fp32_split.h"
#include "mma.h"
#include "work_order.h"
#include "pack_plan.h"

namespace rtoss {

namespace {

constexpr int kFrag = 1024;  // 64 lanes x 16 bytes = 16 output channels x 64 bytes of input channels

template <typename T, typename TO, int KS, int TM, int TN>
__global__ __launch_bounds__(256) void conv1x1_ksplit_kernel(const T* __restrict__ x, TO* __restrict__ y,
                                                             const char* __restrict__ wfrag, int P, int Co, Divisor co_blocks,
                                                             int total, int work_per_xcd, Epilogue ep)
{
    constexpr int MINE = KS / 4;                        // stages of a wave
    constexpr int U = MINE < 4 ? MINE : 4;              // ... in registers at once
    constexpr int MT = stream_mt_of(KS), RUNT = MT < TM ? MT : TM;  // tiles whose channels are consecutive for a lane
    constexpr int ROW = 64 * KS;                        // bytes of a position
    static_assert(KS % 4 == 0 && MINE % U == 0 && TM % RUNT == 0, "whole rounds of stages");
    __shared__ __attribute__((aligned(16))) char part[4 * TM * TN * 1024];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // XCD-contiguous work order, channel block fastest: the workgroups of one position tile share an L2
    const int work = (blockIdx.x % 8) * work_per_xcd + blockIdx.x / 8;
    if (work >= total) return;
    const int all_tile = co_blocks.quotient(work), p0 = all_tile * (16 * TN);
    const int f0 = co_blocks.remainder(work, all_tile) * TM;  // first channel tile
    const int nn = lane & 15, qq = lane >> 4;

    const char* a_src = wfrag + ((int64_t)f0 * KS + wave) * kFrag + lane * 16;
    const char* x_src[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int p = min(p0 + 16 * j + nn, P - 1);     // (positions past the end: any, they are not stored)
        x_src[j] = (const char*)x + (int64_t)p * ROW + wave * 64 + qq * 16;
    }
    f32x4 acc[TM][TN];
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[m][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int base = 0; base < MINE; base += U) {
        u32x4 a[U][TM], b[U][TN];
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int m = 0; m < TM; ++m) a[u][m] = *(const u32x4*)(a_src + (m * KS + 4 * (base + u)) * kFrag);
#pragma unroll
            for (int j = 0; j < TN; ++j) b[u][j] = *(const u32x4*)(x_src[j] + 4 * (base + u) * 64);
        }
        __builtin_amdgcn_sched_barrier(0);  // (the scheduler would rather save registers than have the loads in flight together)
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int m = 0; m < TM; ++m)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[m][j] = Dense16<T>::mma(a[u][m], b[u][j], acc[m][j]);
    }

    // ---- the outputs this lane stores: runs of 4*RUNT consecutive channels of one position ----
    constexpr int GROUPS = TM / RUNT;                   // runs per (position, quarter)
    constexpr int ITEMS = GROUPS * TN * 64;             // (run, block, position, quarter)
    constexpr int PER = (ITEMS + 255) / 256, RUN = 4 * RUNT;
    int o_co[PER];
    int o_pos[PER];
    bool o_live[PER];
    // (scale, bias and shortcut are asked for before the partial sums meet: behind that they would be a wait of their own, from
    // memory no one has touched yet)
    EpiResidual<TO, RUN> shortcut[PER];
    float scale[PER][RUN], bias[PER][RUN];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int item = tid + 256 * i, q = item & 3, n = (item >> 2) & 15, g = (item >> 6) % GROUPS, j = (item >> 6) / GROUPS;
        const int f = f0 + g * RUNT;                    // its first tile: tile f % MT of slice f / MT
        o_co[i] = (f / MT) * (16 * MT) + 4 * MT * q + 4 * (f % MT);
        o_pos[i] = p0 + 16 * j + n;
        o_live[i] = item < ITEMS && o_pos[i] < P && o_co[i] < Co;  // (Co is a multiple of 16: a run is all in or all out)
        if (!o_live[i]) continue;
        if (ep.residual) shortcut[i].load(ep, o_pos[i], o_co[i]);
        if (ep.scale)
#pragma unroll
            for (int g4 = 0; g4 < RUNT; ++g4) *(f32x4*)(scale[i] + 4 * g4) = *(const f32x4*)(ep.scale + o_co[i] + 4 * g4);
        if (ep.bias)
#pragma unroll
            for (int g4 = 0; g4 < RUNT; ++g4) *(f32x4*)(bias[i] + 4 * g4) = *(const f32x4*)(ep.bias + o_co[i] + 4 * g4);
    }
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int j = 0; j < TN; ++j) *(f32x4*)(part + ((wave * TM + m) * TN + j) * 1024 + lane * 16) = acc[m][j];
    __syncthreads();
    epi_by_form(ep, [&](auto form) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            if (!o_live[i]) continue;
            const int item = tid + 256 * i, q = item & 3, n = (item >> 2) & 15, g = (item >> 6) % GROUPS, j = (item >> 6) / GROUPS;
            float v[RUN];
#pragma unroll
            for (int m = 0; m < RUNT; ++m) {
                const char* at = part + ((g * RUNT + m) * TN + j) * 1024 + (q * 16 + n) * 16;
                f32x4 sum = *(const f32x4*)at;
#pragma unroll
                for (int w = 1; w < 4; ++w) sum += *(const f32x4*)(at + w * TM * TN * 1024);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[4 * m + e] = sum[e];
            }
            epi_scale_bias_act_of<decltype(form)::value, RUN>(v, ep, scale[i], bias[i]);
            if (ep.residual) shortcut[i].add(v);
            TO* yp = y + (int64_t)o_pos[i] * ep.ldy + o_co[i];
            if constexpr (sizeof(TO) == 4) {
#pragma unroll
                for (int g4 = 0; g4 < RUNT; ++g4) *(f32x4*)(yp + 4 * g4) = f32x4{v[4 * g4], v[4 * g4 + 1], v[4 * g4 + 2], v[4 * g4 + 3]};
            } else if constexpr (RUNT == 1) {
                uint2 o;
                o.x = pack2_from_f32<TO>(v[0], v[1]);
                o.y = pack2_from_f32<TO>(v[2], v[3]);
                *(uint2*)yp = o;
            } else {
#pragma unroll
                for (int g8 = 0; g8 < RUNT / 2; ++g8) {
                    *(u32x4*)(yp + 8 * g8) = pack8_from_f32<TO>(v + 8 * g8);
                }
            }
        }
    });
}

// Channel tiles of the packed section that hold rows of the layer (the section is padded to whole slices).
inline int section_tiles(int KS, int Co)
{
    const int MT = stream_mt_of(KS);
    return (Co + 16 * MT - 1) / (16 * MT) * MT;
}

template <typename T, typename TO, int KS, int TM, int TN>
rtoss_status launch_variant(const rtoss_wdesc& d, const ConvParams& c, const char* wf, const void* x, void* y, hipStream_t s)
{
    const int64_t P = (int64_t)c.N * c.H * c.W;
    const int co_blocks = (section_tiles(KS, d.Co) + TM - 1) / TM;
    const int64_t total = (P + 16 * TN - 1) / (16 * TN) * co_blocks;
    if (P > 0x7fffff00 || total > 0x3fffffff) return fail(RTOSS_ESHAPE, "conv1x1: too many positions");
    const int work_per_xcd = (int)((total + 7) / 8);
    dim3 grid((unsigned)(work_per_xcd * 8)), block(256);
    conv1x1_ksplit_kernel<T, TO, KS, TM, TN><<<grid, block, 0, s>>>((const T*)x, (TO*)y, wf, (int)P, d.Co, Divisor(co_blocks), (int)total,
                                                                    work_per_xcd, c.ep);
    return check_hip(hipGetLastError(), "conv1x1 K-split launch");
}

// Variants by number: tile of a workgroup in channels x positions.
enum Variant { kNone = 0, k32x16, k32x32, k64x32 };

template <typename T, typename TO, int KS>
rtoss_status launch_ks(const rtoss_wdesc& d, const ConvParams& c, int plan, const char* wf, const void* x, void* y, hipStream_t s)
{
    switch (plan) {
    case k32x16: return launch_variant<T, TO, KS, 2, 1>(d, c, wf, x, y, s);
    case k32x32: if constexpr (sizeof(T) == 2) return launch_variant<T, TO, KS, 2, 2>(d, c, wf, x, y, s); else break;
    case k64x32: if constexpr (sizeof(T) == 2) return launch_variant<T, TO, KS, 4, 2>(d, c, wf, x, y, s); else break;
    }
    return fail(RTOSS_EINVAL, "conv1x1: unknown K-split plan %d", plan);
}

template <typename T, typename TO>
rtoss_status launch_typed(const rtoss_wdesc& d, const ConvParams& c, int plan, const char* wf, const void* x, void* y, hipStream_t s)
{
    switch (stage_count(d)) {
    case 4: return launch_ks<T, TO, 4>(d, c, plan, wf, x, y, s);
    case 8: return launch_ks<T, TO, 8>(d, c, plan, wf, x, y, s);
    case 16: return launch_ks<T, TO, 16>(d, c, plan, wf, x, y, s);
    case 32: return launch_ks<T, TO, 32>(d, c, plan, wf, x, y, s);
    }
    return fail(RTOSS_ESHAPE, "conv1x1: unsupported depth for the K split");
}

}  // namespace

// When a launch belongs here: while its workgroups fit the chip in a round or two; beyond that rereading the weights per
// tile costs more than the streaming kernel's start (us, this kernel and the streaming one; positions in brackets):
//     512 -> 256 (400)  3.0  4.8      256 -> 128 (6400)  4.5  5.3      512 -> 128 (6400)   5.7  5.2  stays
//     128 -> 128 (6400) 3.8  4.4      1024 -> 512 (400)  4.6  5.2      128 -> 128 (25600)  7.7  6.1  stays
// The smallest tile that leaves about one workgroup per compute unit.
// fp32 (the matrix instruction takes 16 times as long, so a small tile per workgroup rereads its weights at little cost):
// workgroups of 32 channels x 16 positions per compute unit up to which this kernel is not the slower one (us, this kernel
// and the streaming one, which has its products on the bf16 instruction; positions in brackets):
//     64 ->  64 (6400)      3.4   3.4      64 -> 256 (3192)    4.2   3.9  stays    64 ->  64 (12 769)    4.2  4.0  stays
//    128 ->  64 (6400)      4.0   4.2     128 -> 256 (1600)    4.0   4.2          128 ->  64 (12 769)    5.4  5.2  stays
//    128 -> 256 (3192)      5.5   5.2 stays
//    256 ->  64 (3192)      4.0   5.1     256 -> 256 (812)     4.0   5.1          256 ->  64 (6400)      5.8  5.4  stays
//     64 ->  16 (12 800)    3.6   3.6      64 ->  48 (25 600)  5.4   4.9  stays   128 ->  16 (25 600)    7.0  6.4  stays
//    128 ->  48 (12 800)    5.1   4.9 stays   256 -> 48 (6400) 5.5   5.1  stays   256 ->  32 (12 800)    5.5  6.7  stays: the smaller error
//    512 ->  32 (6400)      6.1   9.3     512 -> 256 (400)     4.0   6.2
int ksplit1x1_plan(const rtoss_wdesc& d, const ConvParams& c)
{
    const int KS = stage_count(d);
    if (KS < 4) return kNone;
    const DeviceInfo& dev = c.dev;
    const int64_t cus = dev.cus, P = (int64_t)c.N * c.H * c.W;
    const auto groups = [&](int tm, int tn) { return (int64_t)((section_tiles(KS, d.Co) + tm - 1) / tm) * ((P + 16 * tn - 1) / (16 * tn)); };
    if (P > 0x7fffff00 || groups(2, 1) > kMaxGridGroups) return kNone;
    if (d.dt == RTOSS_F32) {
        // (tenths of a workgroup per compute unit; one live weight per group of 64 channels: the streaming kernel's six products
        // would be less precise than the fp32 instruction here, fp32_split.h)
        if (KS == 4 && few_live_products(d)) return k32x16;
        const int64_t most = KS <= 8 ? 50 : KS == 16 ? 25 : 16;
        return 10 * groups(2, 1) <= most * cus ? k32x16 : kNone;
    }
    if (groups(2, 1) <= cus) return k32x16;
    if (groups(2, 2) <= cus) return k32x32;
    return groups(4, 2) <= (KS <= 8 ? 2 : 1) * cus ? k64x32 : kNone;
}

rtoss_status launch_conv1x1_ksplit(const rtoss_wdesc& d, const ConvParams& c, int plan, const void* section, const void* x, void* y,
                                   hipStream_t s)
{
    const char* wf = (const char*)section;
    const bool f32out = c.out_dt == RTOSS_F32;
    if (d.dt == RTOSS_F32) return launch_typed<float, float>(d, c, plan, wf, x, y, s);
    if (d.dt == RTOSS_F16)
        return f32out ? launch_typed<f16_t, float>(d, c, plan, wf, x, y, s) : launch_typed<f16_t, f16_t>(d, c, plan, wf, x, y, s);
    return f32out ? launch_typed<bf16_t, float>(d, c, plan, wf, x, y, s) : launch_typed<bf16_t, bf16_t>(d, c, plan, wf, x, y, s);
}

}  // namespace rtoss
