// 3x3 pattern-pruned convolution in dense mode on the CDNA4 matrix cores (fp32 accumulate): every tap is a dense K-step and pruned weights are explicit zeros.
//
// This is the matrix-core path for dictionaries the 2-of-4 sparse instruction cannot take: a
// pattern with three or more corners, or three or more edge midpoints (4- and 5-entry connected
// patterns include such shapes: the T, the plus), or any unfiltered dictionary.  Nothing is
// skipped, so the effective rate on non-zero multiply-adds is capped at k/9 of the dense rate
// (Section II.B: zeros cost as much as any weight unless the kernel can skip them); it is also
// the "dense convolution on the same kernels" comparator when given the all-ones pattern.
//
// Workgroup = 4 waves, output tile = 64 output channels x 16x16 positions; every wave owns all
// 64 channels x 4 blocks of 4x4 positions.  K runs over stages of 32 input channels: the stage's
// 4 x 9 weight fragments (one contiguous piece of the blob) and the activation tile with halo
// (channels-last, 64-byte position pitch at stride 1 and 80 at stride 2) are copied global -> LDS, then each of the 9 taps is
// one v_mfma_f32_16x16x32 step per (channel fragment, position block) whose B operand is a plain
// 16-byte read at the tap's offset.  The LDS is single-buffered; for stride 1 two workgroups
// share a compute unit and hide each other's copy latency.
//
// Output rows are stored straight from the accumulators: the packer assigns output channels to
// matrix rows so that a lane's 16 accumulator values are 16 consecutive channels (row 4q+i of
// fragment m is channel 16q + 4m + i of the workgroup's 64), and the four lane quarters of a
// position together write 128 contiguous bytes.
//
// Small launches use 16 channels x 4x16 positions per workgroup so that they still fill the chip.
// Those of fp32 tensors run through the same kernel on v_mfma_f32_16x16x4_f32: a stage is then 16 input
// channels (the same 64 bytes per position), a lane's 16 bytes are 4 consecutive channels, and the
// K step of 16 channels is 4 instructions, instruction s taking element s of every lane's 16 bytes
// (the K slots of an instruction are the channels 4q + s: any assignment of channels to slots is
// valid as long as both operands use it).  Larger fp32 launches take the bf16 instruction with
// every value split into three (dense3x3_f32.h).
//
// Operand layout of v_mfma_f32_16x16x32 (wave64; r = lane % 16, q = lane / 16): A lane holds
// row r, K = 8q..8q+7; B lane holds column r, K = 8q..8q+7; D lane holds column r, rows 4q..4q+3.
// v_mfma_f32_16x16x4_f32: A lane holds row r, K = q; B lane holds column r, K = q; same D.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "dense3x3_f32.h"
#include "dtypes.h"
#include "epilogue.h"
#include "mma.h"
#include "work_order.h"
#include "pack_plan.h"
#include "tile3x3.h"

namespace rtoss {

namespace {

constexpr int kFrag = 1024;            // 64 lanes x 16 bytes = 16 output channels x 32 input channels of one tap
constexpr int kTM = 4;                 // channel fragments per block of the blob (64 output channels)
constexpr int kBlockBytes = kTM * 9 * kFrag;  // weights of one (stage, channel block)

inline size_t frag_bytes(const rtoss_wdesc& d)
{
    return (size_t)stage_count(d) * dense_channel_blocks(d.Co) * kBlockBytes;
}

// TM channel fragments (of the blob's blocks of 4) and RT x CT position blocks per workgroup.
// RAG: channel counts between the stages (in; rows stay 16-byte multiples) and tiles (out): the last stage's copy
// lanes past the row end read the block of zeros, outputs are stored under a per-channel bound.
template <typename T, typename TO, int S, int TM, int RT, int CT, bool RAG>
__global__ __launch_bounds__(256) void conv3x3_dense_kernel(const T* __restrict__ x, TO* __restrict__ y,
                                                            const char* __restrict__ wfrag, const char* __restrict__ zeros,
                                                            int H, int W, int Ci, int Co, int Ho, int Wo, int cblocks,
                                                            Divisor tiles_c, Epilogue ep)
{
    using G = Geom<S, RT, CT>;
    constexpr int kTN = RT * CT / 4;                            // position blocks per wave
    static_assert(RT * CT % 4 == 0 && kTM % TM == 0, "four waves share the blocks; fragments split the blob's blocks evenly");
    constexpr int A_BYTES = TM * 9 * kFrag;
    constexpr int A_COPIES = A_BYTES / 1024;                    // copy instructions (64 lanes x 16 B)
    constexpr int A_PER_WAVE = (A_COPIES + 3) / 4;
    constexpr int EBI = (int)sizeof(T);                         // a stage is 64 bytes of channels per position
    constexpr int X_CHUNKS = G::x_bytes / 16;                   // including the pad chunk of every position
    constexpr int X_PER_WAVE = ((X_CHUNKS + 63) / 64 + 3) / 4;
    extern __shared__ __attribute__((aligned(16))) char smem[];  // [weights, rounded up][activations, rounded up to whole copies]
    char* lds_a = smem;
    char* lds_x = smem + A_PER_WAVE * 4096;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tile_r = tiles_c.quotient(blockIdx.x), tile_c = tiles_c.remainder(blockIdx.x, tile_r);
    const int cb = blockIdx.y / (kTM / TM), m_first = (blockIdx.y % (kTM / TM)) * TM, n_img = blockIdx.z;
    const int oh0 = tile_r * G::TH, ow0 = tile_c * G::TW;
    const int ih0 = oh0 * S - 1, iw0 = ow0 * S - 1;
    const int stages = RAG ? (Ci * EBI + 63) / 64 : Ci / (64 / EBI);

    // Copy sources of stage 0.  Every lane copies 16 bytes in every copy instruction; a lane whose LDS
    // slot is zero padding of the tile (or a pad chunk) reads the block of zeros behind the fragments.
    const char* x_ptr[X_PER_WAVE];
    static_assert(X_PER_WAVE <= 32, "one bit per copy");
    unsigned tail_ok = 0;  // RAG: bit k = the last stage still has channels at this lane's copy k
#pragma unroll
    for (int k = 0; k < X_PER_WAVE; ++k) {
        const int c = (k * 4 + wave) * 64 + lane;
        const int pos = c / G::kChunks, q = c % G::kChunks;
        if (RAG && (stages - 1) * 64 + 16 * q < Ci * EBI) tail_ok |= 1u << k;
        const int pr = pos / G::LW, pc = pos % G::LW;
        const int ih = ih0 + pr, iw = iw0 + pc;
        const bool inside = q < 4 && pr < G::IH && pc < G::IW && ih >= 0 && ih < H && iw >= 0 && iw < W;
        x_ptr[k] = inside ? (const char*)x + ((((int64_t)n_img * H + ih) * W + iw) * Ci + q * (16 / EBI)) * EBI : zeros;
    }
    const char* a_src = wfrag + (int64_t)cb * kBlockBytes + m_first * 9 * kFrag + lane * 16;
    const int64_t a_stage_stride = (int64_t)cblocks * kBlockBytes;

    const int nn = lane & 15, qq = lane >> 4;
    const int pr = nn >> 2, pc = nn & 3;
    int xb[kTN];  // LDS byte offset of this lane's position in each of its blocks, tap (0,0), its 8 channels
#pragma unroll
    for (int j = 0; j < kTN; ++j) {
        const int blk = wave * kTN + j;
        xb[j] = (((4 * (blk / CT) + pr) * S) * G::LW + (4 * (blk % CT) + pc) * S) * G::kPos + qq * 16;
    }

    // The accumulators are never cleared: the first tap of the first stage multiplies onto the
    // instruction's constant-zero C operand.  (Clearing them in the accumulation registers costs about
    // 18 cycles per register in front of the next matrix instruction.)
    f32x4 acc[TM][kTN];
    auto run_stage = [&](auto first_tag, int stage) {
        constexpr bool FIRST = decltype(first_tag)::value;
        __syncthreads();  // everybody is done reading the previous stage
#pragma unroll
        for (int k = 0; k < A_PER_WAVE; ++k) {  // (copy slots past the fragments read the block of zeros)
            const int kk = k * 4 + wave;
            copy16_to_lds(kk < A_COPIES ? a_src + stage * a_stage_stride + kk * 1024 : zeros, lds_a + kk * 1024);
        }
#pragma unroll
        for (int k = 0; k < X_PER_WAVE; ++k) {
            const char* src = x_ptr[k] + stage * 64;
            if (RAG && stage == stages - 1 && !(tail_ok >> k & 1u)) src = zeros;
            copy16_to_lds(src, lds_x + (k * 4 + wave) * 1024);
        }
        __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this wave's copies have landed in LDS
        __syncthreads();                     // ... and everybody's
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            u32x4 b[kTN];
#pragma unroll
            for (int j = 0; j < kTN; ++j)
                b[j] = *(const u32x4*)(lds_x + xb[j] + ((t / 3) * G::LW + (t % 3)) * G::kPos);
#pragma unroll
            for (int m = 0; m < TM; ++m) {
                const u32x4 a = *(const u32x4*)(lds_a + (m * 9 + t) * kFrag + lane * 16);
#pragma unroll
                for (int j = 0; j < kTN; ++j)
                    acc[m][j] = Dense16<T>::mma(a, b[j], FIRST && t == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[m][j]);
            }
        }
    };
    run_stage(std::true_type{}, 0);
    for (int stage = 1; stage < stages; ++stage) run_stage(std::false_type{}, stage);

    // ---- store: 4*TM consecutive channels of this lane's position in each of its blocks ----
    const int co_lane = cb * (16 * kTM) + 16 * qq + 4 * m_first;
    constexpr int EB = (int)sizeof(TO);
    constexpr int RUN = 4 * TM;
#pragma unroll
    for (int j = 0; j < kTN; ++j) {
        const int blk = wave * kTN + j;
        const int oh = oh0 + 4 * (blk / CT) + pr, ow = ow0 + 4 * (blk % CT) + pc;
        if (oh >= Ho || ow >= Wo || co_lane >= Co) continue;  // (not RAG: Co is a multiple of 16, a run is all in or all out)
        const int64_t pos = ((int64_t)n_img * Ho + oh) * Wo + ow;
        TO* yp = y + pos * ep.ldy + co_lane;
        float v[RUN];
#pragma unroll
        for (int m = 0; m < TM; ++m)
#pragma unroll
            for (int e = 0; e < 4; ++e) v[4 * m + e] = acc[m][j][e];
        if constexpr (RAG) {
            epi_ragged<TO, RUN>(v, ep, pos, co_lane, Co);
            store_ragged<TO, RUN>(yp - co_lane, v, co_lane, Co, ep.ldy);
            continue;
        }
        epi_scale_bias_act<RUN>(v, ep, co_lane);
        epi_residual<TO, RUN>(v, ep, pos, co_lane);
        if constexpr (EB == 4) {
#pragma unroll
            for (int g = 0; g < TM; ++g) *(f32x4*)(yp + 4 * g) = f32x4{v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
        } else if constexpr (TM == 1) {
            uint2 o;
            o.x = pack2_from_f32<TO>(v[0], v[1]);
            o.y = pack2_from_f32<TO>(v[2], v[3]);
            *(uint2*)yp = o;
        } else {
#pragma unroll
            for (int g = 0; g < TM / 2; ++g) {
                *(u32x4*)(yp + 8 * g) = pack8_from_f32<TO>(v + 8 * g);
            }
        }
    }
}

template <typename T, typename TO, int S, int TM, int RT, int CT, bool RAG = false>
rtoss_status launch_shape(const rtoss_wdesc& d, const ConvParams& c, const char* wfrag, const void* x, void* y, hipStream_t s)
{
    using G = Geom<S, RT, CT>;
    const int Ho = (c.H + 2 - 3) / S + 1, Wo = (c.W + 2 - 3) / S + 1;
    const int tiles_r = (Ho + G::TH - 1) / G::TH, tiles_c = (Wo + G::TW - 1) / G::TW;
    const int cblocks = dense_channel_blocks(d.Co);
    constexpr int x_copies_per_wave = ((G::x_bytes / 16 + 63) / 64 + 3) / 4;
    constexpr int a_copies_per_wave = (TM * 9 + 3) / 4;
    const size_t smem = (size_t)(a_copies_per_wave + x_copies_per_wave) * 4096;
    auto kern = conv3x3_dense_kernel<T, TO, S, TM, RT, CT, RAG>;
    static LaunchOnce lds_once;  // per instantiation
    if (rtoss_status st = ensure_dynamic_lds((const void*)kern, smem, lds_once, c.dev.device, "conv3x3 dense shared memory attribute")) return st;
    const int ygrid = cblocks * (kTM / TM);
    if (c.N > 65535 || ygrid > 65535) return fail(RTOSS_ESHAPE, "conv: batch or channel count too large");
    dim3 grid((unsigned)(tiles_r * tiles_c), (unsigned)ygrid, (unsigned)c.N), block(256);
    kern<<<grid, block, smem, s>>>((const T*)x, (TO*)y, wfrag, wfrag + frag_bytes(d), c.H, c.W, d.Ci, d.Co, Ho, Wo, cblocks,
                                   Divisor(tiles_c), c.ep);
    return check_hip(hipGetLastError(), "conv3x3 dense launch");
}

// fp32: dense3x3_f32.h
template <typename T, typename TO, int S, int R, bool RAG>
__global__ __launch_bounds__(256, 2) void conv3x3_dense_kernel(const T* __restrict__ x, TO* __restrict__ y,
                                                               const char* __restrict__ wfrag, const char* __restrict__ zeros,
                                                               int H, int W, int Ci, int Co, int Ho, int Wo, WorkOrder order, Epilogue ep)
{
    static_assert(sizeof(T) == 4 && sizeof(TO) == 4, "fp32");
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int work = order.item();
    if (work >= order.total) return;
    const int all_tile = order.co_blocks.quotient(work), cblocks = order.co_blocks.by, cb = order.co_blocks.remainder(work, all_tile);
    const WorkOrder::Tile tile = order.tile(all_tile);
    dense3x3_f32_tile<S, R, RAG>(x, y, wfrag, zeros, H, W, Ci, Co, Ho, Wo, cblocks, cb, tile.n_img, tile.row * R, tile.col * 16, ep, smem);
}

template <int S, int R, bool RAG>
rtoss_status launch_f32_rows(const rtoss_wdesc& d, const ConvParams& c, const char* wfrag, const void* x, void* y, hipStream_t s)
{
    const int Ho = (c.H - 1) / S + 1, Wo = (c.W - 1) / S + 1;
    const int tiles_r = (Ho + R - 1) / R, tiles_c = (Wo + 15) / 16, cblocks = dense_channel_blocks(d.Co);
    auto kern = conv3x3_dense_kernel<float, float, S, R, RAG>;
    constexpr int lds = F32Tile<S, R>::LDS;
    static LaunchOnce lds_once;  // per instantiation
    if (rtoss_status st = ensure_dynamic_lds((const void*)kern, lds, lds_once, c.dev.device, "conv3x3 dense shared memory attribute")) return st;
    if (c.N > 65535 || cblocks * kTM > 65535) return fail(RTOSS_ESHAPE, "conv: batch or channel count too large");  // (as above)
    const int64_t total = (int64_t)tiles_r * tiles_c * cblocks * c.N;  // (at most kMaxGridGroups: dense3x3_launch_ok)
    const WorkOrder order(total, cblocks, tiles_r * tiles_c, tiles_c);
    kern<<<dim3(order.grid()), dim3(256), lds, s>>>((const float*)x, (float*)y, wfrag, wfrag + frag_bytes(d), c.H, c.W, d.Ci, d.Co, Ho, Wo, order, c.ep);
    return check_hip(hipGetLastError(), "conv3x3 dense launch");
}

inline bool ragged(const rtoss_wdesc& d) { return d.Ci % stage_channels(d.dt) || d.Co % 16; }

template <typename T, typename TO, int S>
rtoss_status launch_stride(const rtoss_wdesc& d, const ConvParams& c, const char* wfrag, const void* x, void* y, hipStream_t s)
{
    // 64 channels x 16x16 positions per workgroup; launches that would not fill the chip that way take
    // 16 channels x 4x16 positions (16 times as many workgroups).
    const int Ho = (c.H + 2 - 3) / S + 1, Wo = (c.W + 2 - 3) / S + 1;
    const int64_t big = (int64_t)((Ho + 15) / 16) * ((Wo + 15) / 16) * dense_channel_blocks(d.Co) * c.N;
    if (ragged(d)) return launch_shape<T, TO, S, 1, 1, 4, true>(d, c, wfrag, x, y, s);
    if (big < 256) return launch_shape<T, TO, S, 1, 1, 4>(d, c, wfrag, x, y, s);
    return launch_shape<T, TO, S, 4, 4, 4>(d, c, wfrag, x, y, s);
}

// Workgroups of an fp32 launch with R output rows each.
inline int64_t f32_groups(const rtoss_wdesc& d, const ConvParams& c, int rows)
{
    const int Ho = (c.H - 1) / c.stride + 1, Wo = (c.W - 1) / c.stride + 1;
    return (int64_t)((Ho + rows - 1) / rows) * ((Wo + 15) / 16) * dense_channel_blocks(d.Co) * c.N;
}

// fp32.  Rows of a workgroup's tile on the bf16 instruction, or 0: too few workgroups for it, the small tile above on the fp32
// instruction is faster (a launch waits for the split of 64 channels' weights, and ragged channel counts pad the larger tiles).
// us on the small tile / with 2 / 4 / 8 rows (eight: conv3x3_strip.hip), workgroups with 2 rows in brackets:
//      32 ->  32 1x40x50 (80)    4.2  5.1  6.7           64 ->  64 4x80x80 (800)    24.0  18.7  15.0  16.1
//      96 ->  96 1x40x50 (160)  10.2  9.3 11.7           96 ->  96 2x80x100 (1120)  40.7  26.2  26.4  27.4
//     128 -> 128 1x56x60 (224)  13.5 11.8 15.3           32 ->  32 4x112x140 (2016) 25.0  17.5  15.4  13.4
//      64 ->  64 2x60x70 (300)  11.9  9.6  9.7          256 -> 256 4x80x80 (3200)   274   164   141   135
//     ragged: 40 -> 72 2x40x60 (320) 8.8 9.9 9.9; 80 -> 80 1x100x120 (800) 25.6 22.4 18.4; 48 -> 72 4x77x91 (1872) 33.1 29.8 24.0
//     stride 2, two rows (four would leave one workgroup per compute unit): 64 -> 128 2x80x100 13.5 10.6, 32 -> 64 4x112x140 15.4 10.7
// Layers of up to 16 input channels, half of whose stage is zeros, would be faster on the small tile in launches of up to three
// workgroups per compute unit (16 -> 16 4x56x56 6.7 us, 5.2 there; 16 -> 64 2x126x83 8.8 and 7.5; stride 2 16 -> 16 1x320x320 11.3 and 10.4), with the
// fp32 instruction's larger error: not taken.
// Sums of few live products stay on the fp32 instruction, for their precision (8 -> 72 4x77x91, k = 2: 14.7 us, split 13.9; stride 2 8.5, 7.0).
int f32_rows(const rtoss_wdesc& d, const ConvParams& c, int64_t cus)
{
    if (few_live_products(d) || (!ragged(d) && !stores_in_reach(c))) return 0;
    const int64_t g2 = f32_groups(d, c, 2);
    if (c.stride == 2) return g2 > cus / 2 ? 2 : 0;
    if (ragged(d) ? 2 * g2 < 3 * cus : 8 * g2 < 5 * cus) return 0;
    return 2 * f32_groups(d, c, 4) >= cus ? 4 : 2;
}

template <bool RAG> rtoss_status launch_f32(const rtoss_wdesc& d, const ConvParams& c, const char* wfrag, const void* x, void* y, hipStream_t s)
{
    const DeviceInfo& dev = c.dev;
    const int rows = f32_rows(d, c, dev.cus);
    if (c.stride == 2) {
        if (rows == 0) return launch_shape<float, float, 2, 1, 1, 4, RAG>(d, c, wfrag, x, y, s);
        return launch_f32_rows<2, 2, RAG>(d, c, wfrag, x, y, s);
    }
    if (rows == 0) return launch_shape<float, float, 1, 1, 1, 4, RAG>(d, c, wfrag, x, y, s);
    if constexpr (!RAG)  // (ragged launches that small take the tile above)
        if (rows == 2) return launch_f32_rows<1, 2, false>(d, c, wfrag, x, y, s);
    return launch_f32_rows<1, 4, RAG>(d, c, wfrag, x, y, s);
}

template <typename T, typename TO>
rtoss_status launch_typed(const rtoss_wdesc& d, const ConvParams& c, const char* wfrag, const void* x, void* y, hipStream_t s)
{
    if (c.stride == 1) return launch_stride<T, TO, 1>(d, c, wfrag, x, y, s);
    return launch_stride<T, TO, 2>(d, c, wfrag, x, y, s);
}

}  // namespace

// ---- host-visible entry points of this file ----

bool dense3x3_shape_ok(const rtoss_wdesc& d)
{
    return d.ksize == 3 && d.Ci * elem_bytes(d.dt) % 16 == 0;  // rows of whole 16-byte copies
}

bool dense3x3_launch_ok(const rtoss_wdesc& d, const ConvParams& c)
{
    if (d.dt == RTOSS_F32 && f32_groups(d, c, c.stride == 1 ? 4 : 2) > kMaxGridGroups) return false;
    if (!ragged(d)) return true;
    const int Ho = (c.H - 1) / c.stride + 1, Wo = (c.W - 1) / c.stride + 1;  // tiles of 4x16 positions x 16 channels
    return (int64_t)((Ho + 3) / 4) * ((Wo + 15) / 16) <= kMaxGridGroups && dense_channel_blocks(d.Co) * kTM <= 65535;
}

size_t dense3x3_section_bytes(const rtoss_wdesc& d) { return frag_bytes(d) + zero_section_bytes(stage_count(d)); }

rtoss_status launch_conv3x3_dense(const rtoss_wdesc& d, const ConvParams& c, const void* section, const void* x, void* y,
                                  hipStream_t s)
{
    const char* wf = (const char*)section;
    const bool f32out = c.out_dt == RTOSS_F32;
    if (const int plan = ksplit3x3_plan(d, c, 2)) return launch_conv3x3_ksplit(d, c, 2, plan, section, wf + frag_bytes(d), x, y, s);
    if (const int plan = strip3x3_plan(d, c, 2)) return launch_conv3x3_strip(d, c, 2, plan, section, wf + frag_bytes(d), x, y, s);
    if (d.dt == RTOSS_F32) return ragged(d) ? launch_f32<true>(d, c, wf, x, y, s) : launch_f32<false>(d, c, wf, x, y, s);
    if (d.dt == RTOSS_F16)
        return f32out ? launch_typed<f16_t, float>(d, c, wf, x, y, s) : launch_typed<f16_t, f16_t>(d, c, wf, x, y, s);
    return f32out ? launch_typed<bf16_t, float>(d, c, wf, x, y, s) : launch_typed<bf16_t, bf16_t>(d, c, wf, x, y, s);
}

}  // namespace rtoss
