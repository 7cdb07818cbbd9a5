// 3x3 pattern-pruned convolution on the CDNA4 matrix cores for launches that cannot fill the chip with work: the
// input channels are split over the waves of a workgroup.  Reads the packed sections of sparse_frag.h (2-of-4 steps), of
// the dense-mode kernel (one step per tap: 16-bit dictionaries without a 2-of-4 shape, and fp32) and of the gather
// kernel (one step per tap that a block of kernels keeps).
//
// What bounds such a launch (a 20x20 or 40x40 image, one frame, a small pyramid level) is not a rate but a chain of
// latencies: the single-buffered kernel walks the stages of 32 input channels one after the other, and each stage is
// a global -> LDS copy (about a microsecond when the data is in no near cache), a barrier and a few hundred cycles of
// matrix work on a handful of compute units.  256 -> 256 channels at 20x20, one image: 8 stages, 24 workgroups, 10.5 us.
// Here
//   * wave v of a workgroup's four takes stages v, v + 4, ... for the whole output tile of the workgroup.  It copies
//     its own stages into LDS of its own, waits for its own copies and multiplies: no barrier until the end.
//   * 256 input channels arrive in two latencies.  (All of them in one, with two slots per wave: the same time, and
//     half the workgroups per compute unit.)
//   * Tiles are small (16 to 64 channels x 16 to 64 positions): four times as many workgroups from the K split's
//     smaller footprint, and the smallest launches still reach most compute units.
//   * The four partial sums meet in LDS: one write, one barrier, and each lane adds the four values of the outputs it
//     stores.  (fp32, the same products in another order.)
// Measured for that layer: 4.0 us.
//
// The dispatch (ksplit_plan) takes this kernel where the single-buffered or pipelined one would leave the chip idle;
// see the rule there.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "dtypes.h"
#include "epilogue.h"
#include "mma.h"
#include "sparse_frag.h"
#include "work_order.h"
#include "tile3x3.h"

namespace rtoss {

namespace {

// How a stage of one channel tile is multiplied: the tap layouts of sparse_frag.h, or one dense step per tap.
// (kGathered: one dense step per tap that any kernel of the block keeps, conv3x3_gather.hip.)
constexpr int kDenseTaps = 2, kGathered = 3;
constexpr int kGatherSteps = 3;  // steps of a gathered stage in LDS at a time
constexpr int steps_tile_bytes(int lay) { return lay == kGathered ? kGatherSteps * kFragBytes : lay == kDenseTaps ? 9 * kFragBytes : layout_tile_bytes(kLayouts[lay]); }

// Channel tiles that hold rows of the layer: 64 channels are dealt over the rows of four tiles (tile_row_channel).
inline int channel_tiles(int Co) { return 4 * ((Co + 63) / 64); }

// Sizes of one variant: 16*TM channels x RT x CT blocks of 4x4 positions, one stage per wave in LDS.
template <int S, int TM, int RT, int CT, int LAY> struct KSplit {
    using G = Geom<S, RT, CT>;
    static constexpr int TN = RT * CT;
    static constexpr int TILE = steps_tile_bytes(LAY);
    static constexpr int A_BYTES = TM * TILE;
    static constexpr int A_COPIES = (A_BYTES + 1023) / 1024;  // 64 lanes x 16 bytes each
    static constexpr int H_COPIES = LAY == kGathered;         // the block's step count and tap lists
    static constexpr int X_COPIES = (G::x_bytes + 1023) / 1024;
    static constexpr int COPIES = A_COPIES + X_COPIES + H_COPIES;
    static constexpr int SLOT = COPIES * 1024;                // one stage
    static constexpr int LDS = 4 * SLOT;
    static constexpr int MPT = TM * TN >= 4 ? TM * TN / 4 : 1;  // channel tiles whose outputs one lane stores
    static_assert(MPT <= TM && TM % MPT == 0, "a lane stores tiles of one position");
    static_assert(4 * TM * TN * 1024 <= LDS, "the partial sums fit");
    static_assert(LDS <= 160 * 1024, "a compute unit's LDS");
};

// Scale, bias and shortcut of a lane's 4 * M consecutive channels.
template <typename TO, int M> struct OutputOperands {
    EpiResidual<TO, 4 * M> shortcut;
    float scale[4 * M], bias[4 * M];
    static __device__ __forceinline__ bool any(const Epilogue& ep) { return (uintptr_t)ep.residual | (uintptr_t)ep.scale | (uintptr_t)ep.bias; }
    __device__ __forceinline__ void load(const Epilogue& ep, int64_t pos, int co)
    {
        if (ep.residual) shortcut.load(ep, pos, co);
        if (ep.scale)
#pragma unroll
            for (int g = 0; g < M; ++g) *(f32x4*)(scale + 4 * g) = *(const f32x4*)(ep.scale + co + 4 * g);
        if (ep.bias)
#pragma unroll
            for (int g = 0; g < M; ++g) *(f32x4*)(bias + 4 * g) = *(const f32x4*)(ep.bias + co + 4 * g);
    }
};

template <typename T, typename TO, int S, int TM, int RT, int CT, int LAY>
__global__ __launch_bounds__(256) void conv3x3_ksplit_kernel(const T* __restrict__ x, TO* __restrict__ y,
                                                             const char* __restrict__ wfrag, const char* __restrict__ zeros,
                                                             int H, int W, int Ci, int Co, int Ho, int Wo, int m_tiles_total,
                                                             WorkOrder order, const char* __restrict__ headers, Epilogue ep)
{
    using K = KSplit<S, TM, RT, CT, LAY>;
    using G = typename K::G;
    constexpr TapLayout LY = kLayouts[LAY >= kDenseTaps ? 0 : LAY];
    constexpr int NG = LY.groups, FR = layout_fragments(LY), TN = K::TN;
    constexpr int PER = 16 / (int)sizeof(T);  // channels in a lane's 16 bytes; a stage is four of them
    extern __shared__ __attribute__((aligned(16))) char smem[];  // [wave][weights | activations]; at the end the partial sums

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int work = order.item();
    if (work >= order.total) return;
    const int all_tile = order.co_blocks.quotient(work);
    const int mt0 = order.co_blocks.remainder(work, all_tile) * TM;
    const WorkOrder::Tile tile = order.tile(all_tile);
    const int n_img = tile.n_img, oh0 = tile.row * G::TH, ow0 = tile.col * G::TW;
    const int ih0 = oh0 * S - 1, iw0 = ow0 * S - 1;
    const int stages = Ci / (4 * PER);
    char* mine = smem + wave * K::SLOT;

    // ---- this wave's copies ----
    // (gathered: [stage][block of four tiles][step][tile], else [stage][tile][step])
    constexpr int FILE_TILE = LAY == kGathered ? 9 * kFragBytes : K::TILE;
    const char* a_src = wfrag + (LAY == kGathered ? (int64_t)(mt0 / 4) * (4 * FILE_TILE) + (mt0 % 4) * kFragBytes : (int64_t)mt0 * FILE_TILE) + lane * 16;
    const int64_t a_stage_stride = (int64_t)m_tiles_total * FILE_TILE;
    const char* x_ptr[K::X_COPIES];
    // gathered: the fragments of steps first .. first+kGatherSteps-1 (those past the stage's own count are not multiplied)
    auto issue_steps = [&](int stage, char* slot, int first) {
        const char* src = a_src + stage * a_stage_stride + first * (4 * kFragBytes);
#pragma unroll
        for (int st = 0; st < kGatherSteps; ++st)
#pragma unroll
            for (int m = 0; m < TM; ++m) copy16_to_lds(src + (4 * st + m) * kFragBytes, slot + (st * TM + m) * kFragBytes);
    };
    auto issue_weights = [&](int stage, char* slot) {
        if constexpr (LAY == kGathered) {
            copy16_to_lds(headers + ((int64_t)stage * (m_tiles_total / 4) + mt0 / 4) * 64 + (lane & 3) * 16, slot + (K::A_COPIES + K::X_COPIES) * 1024);
            issue_steps(stage, slot, 0);
            return;
        }
#pragma unroll
        for (int k = 0; k < K::A_COPIES; ++k) {
            const char* src = a_src + stage * a_stage_stride + k * 1024;
            if ((k + 1) * 1024 > K::A_BYTES && k * 1024 + lane * 16 >= K::A_BYTES) src = zeros;  // half a copy past an odd tile
            copy16_to_lds(src, slot + k * 1024);
        }
    };
    auto issue_activations = [&](int stage, char* slot) {
#pragma unroll
        for (int k = 0; k < K::X_COPIES; ++k) copy16_to_lds(x_ptr[k] + stage * 64, slot + (K::A_COPIES + k) * 1024);
    };
    // (the first stage's weights are under way while the lanes work out their activation sources)
    if (wave < stages) issue_weights(wave, mine);

    // outputs this lane stores: 4*MPT consecutive channels of one position
    constexpr int MG = TM / K::MPT;
    constexpr bool IDLE = MG * TN < 4;  // fewer outputs than lanes: the upper waves store nothing
    const int o_m = (tid % MG) * K::MPT, o_q = (tid / MG) & 3, o_n = (tid / (4 * MG)) & 15, o_j = tid / (64 * MG);
    const int o_h = oh0 + 4 * (o_j / CT) + (o_n >> 2), o_w = ow0 + 4 * (o_j % CT) + (o_n & 3);
    const int o_co = 64 * ((mt0 + o_m) >> 2) + 16 * o_q + 4 * ((mt0 + o_m) & 3);
    const bool o_live = (!IDLE || o_j < TN) && o_h < Ho && o_w < Wo && o_co < Co;
    const int64_t o_pos = ((int64_t)n_img * Ho + o_h) * Wo + o_w;

#pragma unroll
    for (int k = 0; k < K::X_COPIES; ++k) {
        const int c = k * 64 + lane;
        const int pos = c / G::kChunks, q = c % G::kChunks;
        const int xr = pos / G::LW, xc = pos % G::LW;
        const int ih = ih0 + xr, iw = iw0 + xc;
        const bool inside = q < 4 && xr < G::IH && xc < G::IW && ih >= 0 && ih < H && iw >= 0 && iw < W;
        const int off = ((n_img * H + ih) * W + iw) * (Ci / PER) + q;  // in 16-byte chunks (31 bits: checked by the launcher)
        x_ptr[k] = inside ? (const char*)x + (int64_t)off * 16 : zeros;
    }
    if (wave < stages) issue_activations(wave, mine);

    // Scale, bias and shortcut of this lane's outputs come with the first stage, from memory no one has touched yet (asked for behind
    // the last stage instead: 128 -> 128 @ 40 with SiLU 4.82 us, now 4.52; stride 2, 256 -> 256 @ 40 6.36, 6.00).  One branch around all
    // three: a layer without them pays for each (fp32 64 -> 64 @ 56: three branches 5.84 us, one 5.78, none here 5.79).
    // Not in the 16-bit dense mode at stride 2, where holding them through the stages costs each stage: 64 -> 64 @ 20 3.85 us early, 3.71
    // late, 512 -> 512 @ 7 8.01 and 7.40, with SiLU 8.19 and 7.51.  (fp32: 256 -> 256 @ 7 10.70 and 10.45, 64 -> 64 @ 20 with shortcut, in
    // no cache, 5.26 and 5.52)
    constexpr bool EARLY = S == 1 || LAY != kDenseTaps || sizeof(T) == 4;
    constexpr int RUN = 4 * K::MPT;
    OutputOperands<TO, K::MPT> output;
    if (EARLY && output.any(ep) && o_live) output.load(ep, o_pos, o_co);

    const int nn = lane & 15, qq = lane >> 4;
    const int pr = nn >> 2, pc = nn & 3;
    const int xb0 = (pr * S * G::LW + pc * S) * G::kPos + qq * 16;  // this lane's position of block 0, tap (0,0), its 8 channels
    f32x4 acc[TM][TN];
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[m][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    auto multiply = [&](char* slot, int stage) {
        const char* lds_a = slot + lane * 16;
        const char* lds_x = slot + K::A_COPIES * 1024 + xb0;
        auto x_at = [&](int j, int t) {
            return *(const u32x4*)(lds_x + ((4 * (j / CT) * S + t / 3) * G::LW + 4 * (j % CT) * S + t % 3) * G::kPos);
        };
        if constexpr (LAY == kGathered) {
            const char* hdr = slot + (K::A_COPIES + K::X_COPIES) * 1024;
            int steps = __builtin_amdgcn_readfirstlane(*(const int*)hdr);
            steps = steps < 0 || steps > 9 ? 9 : steps;  // (a corrupt header cannot run the loops out of bounds)
            for (int first = 0; first < steps; first += kGatherSteps) {
                int tap[kGatherSteps];
#pragma unroll
                for (int st = 0; st < kGatherSteps; ++st) tap[st] = *(const uint8_t*)(hdr + 8 + qq * 9 + first + st);
                if (first > 0) {
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // reads of the steps before
                    issue_steps(stage, slot, first);
                    __builtin_amdgcn_s_waitcnt(0x0f70);
                    asm volatile("" ::: "memory");
                }
#pragma unroll
                for (int st = 0; st < kGatherSteps; ++st) {
                    if (first + st >= steps) break;
                    const int t3 = (tap[st] * 11) >> 5;  // tap / 3
                    const char* at = lds_x + (t3 * G::LW + tap[st] - 3 * t3) * G::kPos;
                    u32x4 b[TN];
#pragma unroll
                    for (int j = 0; j < TN; ++j) b[j] = *(const u32x4*)(at + (4 * (j / CT) * S * G::LW + 4 * (j % CT) * S) * G::kPos);
#pragma unroll
                    for (int m = 0; m < TM; ++m) {
                        const u32x4 a = *(const u32x4*)(lds_a + (st * TM + m) * kFragBytes);
#pragma unroll
                        for (int j = 0; j < TN; ++j) acc[m][j] = Dense16<T>::mma(a, b[j], acc[m][j]);
                    }
                }
            }
        } else if constexpr (LAY == kDenseTaps) {
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                u32x4 b[TN];
#pragma unroll
                for (int j = 0; j < TN; ++j) b[j] = x_at(j, t);
#pragma unroll
                for (int m = 0; m < TM; ++m) {
                    const u32x4 a = *(const u32x4*)(lds_a + m * K::TILE + t * kFragBytes);
#pragma unroll
                    for (int j = 0; j < TN; ++j) acc[m][j] = Dense16<T>::mma(a, b[j], acc[m][j]);
                }
            }
        } else {
            if constexpr (LY.centre) {
                u32x4 b[TN];
#pragma unroll
                for (int j = 0; j < TN; ++j) b[j] = x_at(j, 4);
#pragma unroll
                for (int m = 0; m < TM; ++m) {
                    const u32x4 a = *(const u32x4*)(lds_a + m * K::TILE + 2 * NG * kFragBytes);
#pragma unroll
                    for (int j = 0; j < TN; ++j) acc[m][j] = Dense16<T>::mma(a, b[j], acc[m][j]);
                }
            }
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                u32x8 bf[2][TN];  // B operands of both sparse steps
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    u32x4 r[4];
#pragma unroll
                    for (int f = 0; f < 4; ++f) r[f] = x_at(j, LY.tap[g][f]);
#pragma unroll
                    for (int half = 0; half < 2; ++half) bf[half][j] = sparse_operand(r, half);
                }
#pragma unroll
                for (int m = 0; m < TM; ++m) {
                    const int idx = *(const int*)(slot + m * K::TILE + FR * kFragBytes + (g * 64 + lane) * 4);
                    const u32x4 a0 = *(const u32x4*)(lds_a + m * K::TILE + (2 * g) * kFragBytes);
                    const u32x4 a1 = *(const u32x4*)(lds_a + m * K::TILE + (2 * g + 1) * kFragBytes);
#pragma unroll
                    for (int j = 0; j < TN; ++j) acc[m][j] = Sparse64<T>::template mma<0>(a0, bf[0][j], acc[m][j], idx);
#pragma unroll
                    for (int j = 0; j < TN; ++j) acc[m][j] = Sparse64<T>::template mma<1>(a1, bf[1][j], acc[m][j], idx);
                }
            }
        }
    };
    for (int s = wave; s < stages; s += 4) {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this wave's copies have landed
        asm volatile("" ::: "memory");
        multiply(mine, s);
        if (s + 4 < stages) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // this wave's reads of the slot are complete
            issue_weights(s + 4, mine);
            issue_activations(s + 4, mine);
        }
    }

    if (!EARLY && output.any(ep) && o_live) output.load(ep, o_pos, o_co);
    __syncthreads();  // everybody is done with the slots
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int j = 0; j < TN; ++j) *(f32x4*)(smem + ((wave * TM + m) * TN + j) * 1024 + lane * 16) = acc[m][j];
    __syncthreads();
    if (!o_live) return;
    float v[RUN];
#pragma unroll
    for (int m = 0; m < K::MPT; ++m) {
        const char* at = smem + ((o_m + m) * TN + o_j) * 1024 + (o_q * 16 + o_n) * 16;
        f32x4 sum = *(const f32x4*)at;
#pragma unroll
        for (int w = 1; w < 4; ++w) sum += *(const f32x4*)(at + w * TM * TN * 1024);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[4 * m + e] = sum[e];
    }
    epi_scale_bias_act<RUN>(v, ep, output.scale, output.bias);
    if (ep.residual) output.shortcut.add(v);
    TO* yp = y + o_pos * ep.ldy + o_co;
    if constexpr (sizeof(TO) == 4) {
#pragma unroll
        for (int g = 0; g < K::MPT; ++g) *(f32x4*)(yp + 4 * g) = f32x4{v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
    } else if constexpr (K::MPT == 1) {
        uint2 o;
        o.x = pack2_from_f32<TO>(v[0], v[1]);
        o.y = pack2_from_f32<TO>(v[2], v[3]);
        *(uint2*)yp = o;
    } else {
#pragma unroll
        for (int g = 0; g < K::MPT / 2; ++g) {
            *(u32x4*)(yp + 8 * g) = pack8_from_f32<TO>(v + 8 * g);
        }
    }
}

template <typename T, typename TO, int S, int TM, int RT, int CT, int LAY>
rtoss_status launch_variant(const rtoss_wdesc& d, const ConvParams& c, const char* wfrag, const char* zeros, const void* x, void* y, hipStream_t s,
                            const char* headers = nullptr)
{
    using K = KSplit<S, TM, RT, CT, LAY>;
    using G = typename K::G;
    const int Ho = (c.H - 1) / S + 1, Wo = (c.W - 1) / S + 1;
    const int tiles_r = (Ho + G::TH - 1) / G::TH, tiles_c = (Wo + G::TW - 1) / G::TW;
    const int co_blocks = channel_tiles(d.Co) / TM;
    auto kern = conv3x3_ksplit_kernel<T, TO, S, TM, RT, CT, LAY>;
    static LaunchOnce lds_once;  // per instantiation
    if (rtoss_status st = ensure_dynamic_lds((const void*)kern, K::LDS, lds_once, c.dev.device, "conv3x3 shared memory attribute")) return st;
    const int64_t total = (int64_t)tiles_r * tiles_c * co_blocks * c.N;
    if (total > 0x3fffffff) return fail(RTOSS_ESHAPE, "conv: too many tiles");
    if ((int64_t)c.N * c.H * c.W * d.Ci * (int)sizeof(T) / 16 > 0x7fffffff) return fail(RTOSS_ESHAPE, "conv: input too large for 32-bit chunk offsets");
    const WorkOrder order(total, co_blocks, tiles_r * tiles_c, tiles_c);
    dim3 grid(order.grid()), block(256);
    kern<<<grid, block, K::LDS, s>>>((const T*)x, (TO*)y, wfrag, zeros, c.H, c.W, d.Ci, d.Co, Ho, Wo,
                                     LAY >= kDenseTaps ? channel_tiles(d.Co) : padded_m_tiles(d.Co), order, headers, c.ep);
    return check_hip(hipGetLastError(), "conv3x3 K-split launch");
}

// Variants by number, smallest tiles first: channels x positions of a workgroup's tile.
enum Variant { kNone = 0, k16x4x8, k32x4x8, k32x8x8, kS2_32x4x4, kS2_32x4x8, kS2_64x4x8 };

template <typename T, typename TO, int LAY>
rtoss_status launch_plan(const rtoss_wdesc& d, const ConvParams& c, int plan, const char* wf, const char* zeros, const void* x, void* y, hipStream_t s)
{
    switch (plan) {
    case k16x4x8: return launch_variant<T, TO, 1, 1, 1, 2, LAY>(d, c, wf, zeros, x, y, s);
    case k32x4x8: if constexpr (LAY != kDenseTaps) return launch_variant<T, TO, 1, 2, 1, 2, LAY>(d, c, wf, zeros, x, y, s); else break;
    case k32x8x8: if constexpr (LAY == 0) return launch_variant<T, TO, 1, 2, 2, 2, LAY>(d, c, wf, zeros, x, y, s); else break;
    case kS2_32x4x4: return launch_variant<T, TO, 2, 2, 1, 1, LAY>(d, c, wf, zeros, x, y, s);
    case kS2_32x4x8: if constexpr (LAY != 0) return launch_variant<T, TO, 2, 2, 1, 2, LAY>(d, c, wf, zeros, x, y, s); else break;
    case kS2_64x4x8: if constexpr (LAY == 0) return launch_variant<T, TO, 2, 4, 1, 2, LAY>(d, c, wf, zeros, x, y, s); else break;
    }
    return fail(RTOSS_EINVAL, "conv: unknown K-split plan %d", plan);
}

template <int LAY>
rtoss_status launch_layout(const rtoss_wdesc& d, const ConvParams& c, int plan, const char* wf, const char* zeros, const void* x, void* y, hipStream_t s)
{
    const bool f32out = c.out_dt == RTOSS_F32;
    if constexpr (LAY == kDenseTaps)
        if (d.dt == RTOSS_F32) return launch_plan<float, float, LAY>(d, c, plan, wf, zeros, x, y, s);
    if (d.dt == RTOSS_F16)
        return f32out ? launch_plan<f16_t, float, LAY>(d, c, plan, wf, zeros, x, y, s) : launch_plan<f16_t, f16_t, LAY>(d, c, plan, wf, zeros, x, y, s);
    return f32out ? launch_plan<bf16_t, float, LAY>(d, c, plan, wf, zeros, x, y, s) : launch_plan<bf16_t, bf16_t, LAY>(d, c, plan, wf, zeros, x, y, s);
}

}  // namespace

// When a launch belongs here.  One round of workgroups (all resident at once) costs 3 to 6 us whatever the layer, set
// by latencies; a second round doubles that, while the kernels with larger tiles pay about 0.9 us per stage once and
// then run at a rate.  So: the smallest tile whose workgroups all fit the chip at once, else none.  Lines drawn from a
// sweep over 32 to 256 channels, images from 14x30 to 112x140, batches of 1 to 4 (layout 0, bf16), e.g. 128 -> 128:
//     14x30 3.3 us (6.7 with the other kernel), 40x60 4.3 (6.9), 60x80 5.8 (7.0), 80x100 stays (8.3 against 7.1).
// A tile of 16 channels rereads the activations most often: it is taken while it leaves one workgroup per compute unit.
int ksplit3x3_plan(const rtoss_wdesc& d, const ConvParams& c, int layout)
{
    if (d.Ci * elem_bytes(d.dt) % 64 || d.Co % 16) return kNone;
    if ((int64_t)c.N * c.H * c.W * d.Ci * elem_bytes(d.dt) / 16 > kMaxChunks) return kNone;  // (the dense-mode kernel has no such limit)
    const DeviceInfo& dev = c.dev;
    const int64_t cus = dev.cus;
    const int stages = d.Ci * elem_bytes(d.dt) / 64;
    const int Ho = (c.H - 1) / c.stride + 1, Wo = (c.W - 1) / c.stride + 1;
    // workgroups of a variant with tiles of 16*tm channels x rows x cols positions
    const auto groups = [&](int tm, int rows, int cols) {
        return (int64_t)(channel_tiles(d.Co) / tm) * ((Ho + rows - 1) / rows) * ((Wo + cols - 1) / cols) * c.N;
    };
    if (layout == kGathered) {
        // 48 KB of LDS with 8 rows of 4, 60 KB with 8 of 8: three and two workgroups per compute unit.  A second round
        // is still the better choice for deep layers: the other kernel has their every stage's copy in front of it.
        // 256 -> 256 with shared patterns of 3: 14x30 4.0 us (12.2 before), 30x40 4.9 (12.5), 60x80 9.1 (12.6), 80x100
        // stays (13.6 against 14.3); 64 -> 64: 60x80 4.0 (6.1), 112x140 5.1 (6.3).  Independent patterns gain as much.
        if (c.stride != 1) return kNone;
        if (groups(1, 4, 8) <= cus) return k16x4x8;
        if (groups(2, 4, 8) <= (stages >= 4 ? 5 : 3) * cus) return k32x4x8;
        return groups(2, 8, 8) <= 2 * cus ? k32x8x8 : kNone;
    }
    if (layout == kDenseTaps) {
        // the dense-mode kernel has small tiles of its own: only the depth of the layer is left to gain here
        if (stages < 4 && c.stride == 1) return kNone;
        if (c.stride == 1) return groups(1, 4, 8) <= 2 * cus ? k16x4x8 : kNone;
        if (groups(2, 4, 4) <= cus) return kS2_32x4x4;
        return groups(2, 4, 8) <= cus ? kS2_32x4x8 : kNone;
    }
    if (c.stride == 1) {
        if (groups(1, 4, 8) <= cus) return k16x4x8;
        if (groups(2, 4, 8) <= 2 * cus) return k32x4x8;
        // (layout 1 has larger fragments: one workgroup per compute unit, and what fits in one round was taken above)
        return layout == 0 && stages >= 2 && groups(2, 8, 8) <= 2 * cus ? k32x8x8 : kNone;
    }
    if (groups(2, 4, 4) <= (layout == 0 && stages >= 2 ? 2 : 1) * cus) return kS2_32x4x4;
    if (layout == 0) return stages >= 3 && groups(4, 4, 8) <= cus ? kS2_64x4x8 : kNone;
    return groups(2, 4, 8) <= cus ? kS2_32x4x8 : kNone;
}

rtoss_status launch_conv3x3_ksplit(const rtoss_wdesc& d, const ConvParams& c, int layout, int plan, const void* section, const void* zeros,
                                   const void* x, void* y, hipStream_t s)
{
    const char *wf = (const char*)section, *z = (const char*)zeros;
    if (layout == kDenseTaps) return launch_layout<kDenseTaps>(d, c, plan, wf, z, x, y, s);
    return layout == 1 ? launch_layout<1>(d, c, plan, wf, z, x, y, s) : launch_layout<0>(d, c, plan, wf, z, x, y, s);
}

rtoss_status launch_conv3x3_ksplit_gather(const rtoss_wdesc& d, const ConvParams& c, int plan, const void* headers, const void* frags,
                                          const void* zeros, const void* x, void* y, hipStream_t s)
{
    const char *wf = (const char*)frags, *z = (const char*)zeros, *h = (const char*)headers;
    const auto launch = [&](auto t, auto to) {
        using T = decltype(t);
        using TO = decltype(to);
        if (plan == k16x4x8) return launch_variant<T, TO, 1, 1, 1, 2, kGathered>(d, c, wf, z, x, y, s, h);
        if (plan == k32x4x8) return launch_variant<T, TO, 1, 2, 1, 2, kGathered>(d, c, wf, z, x, y, s, h);
        if (plan == k32x8x8) return launch_variant<T, TO, 1, 2, 2, 2, kGathered>(d, c, wf, z, x, y, s, h);
        return fail(RTOSS_EINVAL, "conv: unknown K-split plan %d", plan);
    };
    const bool f32out = c.out_dt == RTOSS_F32;
    if (d.dt == RTOSS_F16) return f32out ? launch(f16_t{}, 0.f) : launch(f16_t{}, f16_t{});
    return f32out ? launch(bf16_t{}, 0.f) : launch(bf16_t{}, bf16_t{});
}

}  // namespace rtoss
