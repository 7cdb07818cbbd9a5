// 3x3 pattern-pruned convolution, stride 1, over strips of output rows: the kernel for launches between the ones that
// cannot fill the chip (conv3x3_ksplit.hip) and the ones large enough for the persistent pipeline (conv3x3_rows.hip).
// Reads the packed sections of sparse_frag.h (2-of-4 steps) and of the dense mode (one step per tap: dictionaries without a
// 2-of-4 shape).  Large fp32 launches use the same operand scheme with every value split into three (dense3x3_f32.h).
//
// With the 16 columns of a matrix instruction as a 4x4 block of positions every tap of every block is an operand read of
// its own, nine per block, and LDS bandwidth bounds these layers: a 16-byte read per lane is 8 cycles of the compute
// unit's LDS, a matrix instruction 16 cycles of one of its four SIMDs.  Here the 16 columns are 16 consecutive
// positions of one output row, so the operands of the nine taps are overlapping windows of the same input rows: with
// R[i][kw] = the read of input row i at column shift kw, output row j takes tap (kh, kw) from R[j + kh][kw].  A wave owns
// TN rows and all 64 channels of the workgroup and reads 3*(TN + 2) activation vectors per stage of input channels
// instead of 9*TN; with the weight fragments, TN = 5: 49 reads for 100 matrix instructions (92 with 4x4 blocks).
//
// Two workgroups per compute unit cover each other's copies and barriers.  TN is chosen per launch (strip3x3_plan).  Where
// two buffers of a workgroup fit LDS twice, the next stage's copies are issued behind the barrier that opens a stage (DB).
//
// The dense mode has no operands to transpose, so a wave can take all its weights from memory and half the tiles (the second
// kernel here): LDS then carries the activations only, through registers -- a wave with copies into LDS under way waits for
// all of its LDS reads at once, the compiler cannot count them apart.
//
// What bounds it now, by counters: dense mode with 20 rows keeps the matrix pipes busy 60 % of the time where a compute unit
// has one or two tiles (256 -> 256 at 100x168, two images; 53 % with the weights in LDS), 77 % where it has two; the 2-of-4
// layout with TN = 3 35 %, LDS 32 % (one image): neither rate, but what a stage spends around its matrix instructions, the copies'
// issue and latency and the barriers, with two workgroups to hide it; and with one round of workgroups nothing hides the
// first stage and the stores.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "dense3x3_f32.h"
#include "dtypes.h"
#include "epilogue.h"
#include "mma.h"
#include "pack_plan.h"
#include "sparse_frag.h"
#include "work_order.h"
#include "strip_output.h"

namespace rtoss {

namespace {

constexpr int kTM = kStripTM, kCols = kStripCols, kLW = kStripLW;
constexpr int kDenseTaps = kNumLayouts;
constexpr int kTwoBuffers = 8; // in a plan: rows per wave + kTwoBuffers
constexpr int kDenseRows = 16; // in a plan of the dense mode without weights in LDS: rows of a workgroup + kDenseRows
constexpr int strip_tile_bytes(int lay) { return lay == kDenseTaps ? kDenseTileBytes : layout_tile_bytes(kLayouts[lay]); }

// The phase of a 2-of-4 layout (the centre's, then one per group) that reads input row i at column shift kw first.
constexpr int first_phase(const TapLayout& l, int tn, int i, int kw)
{
    const auto reads = [&](int t) { return kw == t % 3 && i >= t / 3 && i < t / 3 + tn; };
    if (l.centre && reads(4)) return 0;
    for (int g = 0; g < l.groups; ++g)
        for (int f = 0; f < 4; ++f)
            if (reads(l.tap[g][f])) return g + l.centre;
    return -1;
}

template <int TN, int LAY, bool DB> struct Strip {
    static constexpr int ROWS = 4 * TN;                      // output rows of a workgroup
    static constexpr int TILE = strip_tile_bytes(LAY);
    static constexpr int A_BYTES = kTM * TILE;
    static constexpr int A_COPIES = A_BYTES / 1024;          // 64 lanes x 16 bytes each
    static constexpr int X_CHUNKS = (ROWS + 2) * kLW * 4;
    static constexpr int X_COPIES = (X_CHUNKS + 63) / 64;
    static constexpr int A_PER_WAVE = (A_COPIES + 3) / 4, X_PER_WAVE = (X_COPIES + 3) / 4;
    static constexpr int X_AREA = X_PER_WAVE * 4096;
    static constexpr int BUF = A_BYTES + X_AREA;             // one stage
    static constexpr int LDS = (DB ? 2 : 1) * BUF + EpiScaleBias<16 * kTM>::kBytes;
    static constexpr bool AHEAD = DB && LAY == 0;            // operands a phase ahead (run_stage)
    static_assert(A_BYTES % 1024 == 0, "weight fragments are whole copy instructions");
};

template <typename T, typename TO, int TN, int LAY, bool DB, bool ROWS_OUT>
__device__ __forceinline__ void strip_tile(const T* __restrict__ x, TO* __restrict__ y, const char* __restrict__ wfrag, const char* __restrict__ zeros,
                                           int H, int W, int Ci, int Co, int m_tiles_total, WorkOrder order, const Epilogue& ep)
{
    using P = Strip<TN, LAY, DB>;
    constexpr TapLayout LY = kLayouts[LAY == kDenseTaps ? 0 : LAY];
    constexpr int NG = LY.groups, FR = layout_fragments(LY);
    constexpr int PER = 16 / (int)sizeof(T);  // channels in a lane's 16 bytes; a stage is four of them
    extern __shared__ __attribute__((aligned(16))) char smem[];  // [weights][activations][scale, bias]
    float* const lds_ep = (float*)(smem + (DB ? 2 : 1) * P::BUF);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int work = order.item();
    if (work >= order.total) return;
    const int all_tile = order.co_blocks.quotient(work), cb = order.co_blocks.remainder(work, all_tile);
    const WorkOrder::Tile tile = order.tile(all_tile);
    const int n_img = tile.n_img, oh0 = tile.row * P::ROWS, ow0 = tile.col * kCols;
    const int stages = Ci / (4 * PER);

    EpiScaleBias<16 * kTM> scale_bias;
    scale_bias.load(ep, 64 * cb, Co, tid);

    const char* a_src = wfrag + (int64_t)cb * P::A_BYTES + lane * 16;
    const int64_t a_stage_stride = (int64_t)m_tiles_total * P::TILE;
    const char* x_ptr[P::X_PER_WAVE];
#pragma unroll
    for (int k = 0; k < P::X_PER_WAVE; ++k) {
        const int pos = (k * 4 + wave) * 16 + (lane >> 2);
        const int xr = pos / kLW, xc = pos % kLW;
        const int ih = oh0 - 1 + xr, iw = ow0 - 1 + xc;
        const bool inside = xr < P::ROWS + 2 && (unsigned)ih < (unsigned)H && (unsigned)iw < (unsigned)W;
        const int off = ((n_img * H + ih) * W + iw) * (Ci / PER) + (lane & 3);  // in 16-byte chunks (31 bits: checked by the launcher)
        x_ptr[k] = inside ? (const char*)x + (int64_t)off * 16 : zeros;
    }

    const int nn = lane & 15, qq = lane >> 4;
    const int xoff = (wave * TN * kLW + nn) * 64 + qq * 16;
    f32x4 acc[kTM][TN];
    auto issue_copies = [&](int stage, char* buf) {
#pragma unroll
        for (int k = 0; k < P::A_PER_WAVE; ++k) {
            const int kk = k * 4 + wave;  // wave-uniform
            if (kk < P::A_COPIES) copy16_to_lds(a_src + stage * a_stage_stride + kk * 1024, buf + kk * 1024);
        }
#pragma unroll
        for (int k = 0; k < P::X_PER_WAVE; ++k) copy16_to_lds(x_ptr[k] + stage * 64, buf + P::A_BYTES + (k * 4 + wave) * 1024);
    };
    issue_copies(0, smem);
    auto run_stage = [&](auto first_tag, int stage) {
        constexpr bool FIRST = decltype(first_tag)::value;
        const f32x4 none = {0.f, 0.f, 0.f, 0.f};
        const char* lds_a = smem + (DB ? (stage & 1) * P::BUF : 0);
        const char* lds_x = lds_a + P::A_BYTES;
        if constexpr (DB) {
            __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this wave's copies of this stage have landed in LDS
            if constexpr (FIRST) scale_bias.store(lds_ep, ep, tid);
            __syncthreads();  // ... and everybody's; and everybody is done reading the other buffer
            if (stage + 1 < stages) issue_copies(stage + 1, smem + ((stage & 1) ^ 1) * P::BUF);
        } else {
            if constexpr (!FIRST) {
                __syncthreads();  // everybody is done reading the previous stage
                issue_copies(stage, smem);
            }
            __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this wave's copies have landed in LDS
            if constexpr (FIRST) scale_bias.store(lds_ep, ep, tid);
            __syncthreads();                     // ... and everybody's
        }
        u32x4 R[TN + 2][3];
        const char* A = lds_a + lane * 16;
        if constexpr (LAY == kDenseTaps) {
#pragma unroll
            for (int i = 0; i < TN + 2; ++i)
#pragma unroll
                for (int kw = 0; kw < 3; ++kw) R[i][kw] = *(const u32x4*)(lds_x + xoff + (i * kLW + kw) * 64);
#pragma unroll
            for (int t = 0; t < 9; ++t)
#pragma unroll
                for (int m = 0; m < kTM; ++m) {
                    const u32x4 a = *(const u32x4*)(A + m * P::TILE + t * kFragBytes);
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[m][j] = Dense16<T>::mma(a, R[j + t / 3][t % 3], FIRST && t == 0 ? none : acc[m][j]);
                }
        } else {
            // Phases: the centre, then the groups of four taps.  With copies into LDS under way a wave cannot wait for some of its
            // reads, only for all it has asked for: 26 of the stage's 35 stood in front of the first product.  With two buffers a
            // phase's operands are asked for in front of the products of the phase before, so the first product waits for 7.
            // (256 -> 256 on 1x50x84 10.5 -> 10.0 us, 512 -> 512 on 2x40x40 18.1 -> 16.9; TN = 3, whose two workgroups per compute
            // unit cover each other, gains less: 4x50x84 18.1 -> 17.6, 1x100x168 19.4 -> 18.9, 512 -> 256 on 1x100x160 30.8 -> 29.6.
            // Layout 1 and one buffer gained nothing from it.)
            constexpr int PHASES = NG + LY.centre;
            u32x4 a[2][kTM][2];
            int idx[2][kTM];
            auto fetch = [&](auto phase_tag) {
                constexpr int phase = decltype(phase_tag)::value, g = phase - LY.centre, at = P::AHEAD ? phase % 2 : 0;
                static_for<3 * (TN + 2)>([&](auto window) {
                    constexpr int i = decltype(window)::value / 3, kw = decltype(window)::value % 3;
                    if constexpr ((P::AHEAD ? first_phase(LY, TN, i, kw) : 0) == phase) R[i][kw] = *(const u32x4*)(lds_x + xoff + (i * kLW + kw) * 64);
                });
#pragma unroll
                for (int m = 0; m < kTM; ++m) {
                    a[at][m][0] = *(const u32x4*)(A + m * P::TILE + (g < 0 ? 2 * NG : 2 * g) * kFragBytes);
                    if constexpr (g >= 0) {
                        a[at][m][1] = *(const u32x4*)(A + m * P::TILE + (2 * g + 1) * kFragBytes);
                        idx[at][m] = *(const int*)(lds_a + m * P::TILE + FR * kFragBytes + (g * 64 + lane) * 4);
                    }
                }
            };
            fetch(std::integral_constant<int, 0>{});
            static_for<PHASES>([&](auto phase_tag) {
                constexpr int phase = decltype(phase_tag)::value, g = phase - LY.centre, at = P::AHEAD ? phase % 2 : 0;
                if constexpr (P::AHEAD) {
                    __builtin_amdgcn_sched_barrier(0);
                    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
                    if constexpr (phase + 1 < PHASES) fetch(std::integral_constant<int, phase + 1>{});
                    __builtin_amdgcn_sched_barrier(0);
                } else if constexpr (phase > 0) {
                    fetch(phase_tag);
                }
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    if constexpr (g < 0) {
#pragma unroll
                        for (int m = 0; m < kTM; ++m) acc[m][j] = Dense16<T>::mma(a[at][m][0], R[j + 1][1], FIRST ? none : acc[m][j]);
                    } else {
                        u32x4 r[4];
#pragma unroll
                        for (int f = 0; f < 4; ++f) {
                            const int t = LY.tap[g][f];
                            r[f] = R[j + t / 3][t % 3];
                        }
                        const u32x8 b[2] = {sparse_operand(r, 0), sparse_operand(r, 1)};
#pragma unroll
                        for (int m = 0; m < kTM; ++m)
                            acc[m][j] = Sparse64<T>::template mma<0>(a[at][m][0], b[0], FIRST && phase == 0 ? none : acc[m][j], idx[at][m]);
#pragma unroll
                        for (int m = 0; m < kTM; ++m) acc[m][j] = Sparse64<T>::template mma<1>(a[at][m][1], b[1], acc[m][j], idx[at][m]);
                    }
                }
            });
        }
    };
    run_stage(std::true_type{}, 0);
    for (int stage = 1; stage < stages; ++stage) run_stage(std::false_type{}, stage);

    // ---- store: a lane holds column nn (position) and 16 consecutive channels of each of its rows ----
    // ROWS_OUT: in rows of 128 bytes, past the L2's write-back (RowTile, through the LDS buffer that the last stage does not read; the one
    // buffer behind a barrier).  Stores of 16 bytes from the registers, written back when the launch ends, took 64 -> 64 channels on 16x80x80 with
    // SiLU and shortcut from 12.3 to 14.3 us, 128 -> 128 on 16x40x40 10.6 to 11.3, 256 -> 256 on 1x100x168 18.0 to 18.8, 1x50x84 10.2 to 10.4.
    if (ROWS_OUT && !DB) __syncthreads();  // everybody is done reading the last stage
    char* const area = smem + (DB ? (stages & 1) * P::BUF : 0) + wave * (TN * RowTile<TO>::kBytes);
    static_assert(4 * TN * RowTile<TO>::kBytes <= P::BUF, "the tiles of all waves fit a buffer");
    strip_output<TO, TN, ROWS_OUT>(acc, area, lds_ep, y, H, W, Co, cb, n_img, oh0 + wave * TN, ow0, lane, ep);
}

// (ROWS: whether 16-bit outputs leave in rows, where both are there; two buffers and fp32 results know one way)
template <typename T, typename TO, int TN, int LAY, bool DB>
__global__ __launch_bounds__(256, 2) void conv3x3_strip_kernel(const T* __restrict__ x, TO* __restrict__ y, const char* __restrict__ wfrag,
                                                               const char* __restrict__ zeros, int H, int W, int Ci, int Co, int m_tiles_total,
                                                               WorkOrder order, Epilogue ep)
{
    strip_tile<T, TO, TN, LAY, DB, DB && sizeof(TO) == 2>(x, y, wfrag, zeros, H, W, Ci, Co, m_tiles_total, order, ep);
}
template <typename T, typename TO, int TN, int LAY, bool DB, bool ROWS>
__global__ __launch_bounds__(256, 2) void conv3x3_strip_kernel(const T* __restrict__ x, TO* __restrict__ y, const char* __restrict__ wfrag,
                                                               const char* __restrict__ zeros, int H, int W, int Ci, int Co, int m_tiles_total,
                                                               WorkOrder order, Epilogue ep)
{
    strip_tile<T, TO, TN, LAY, DB, ROWS>(x, y, wfrag, zeros, H, W, Ci, Co, m_tiles_total, order, ep);
}

// Dense mode.  A tap's fragment is used for one product per row and tile and needs no transposition, so here the weights stay out
// of LDS: wave (p, h) owns channel tiles 2p and 2p+1 and the rows of half h, and loads its fragments straight into registers,
// the next column of taps' while the current one is multiplied.
template <int ROWS> struct DenseStrip {
    static constexpr int RW = ROWS / 2;                          // rows of a wave
    static constexpr int CHUNKS = (ROWS + 2) * kLW * 4;
    static constexpr int PER_WAVE = (CHUNKS + 255) / 256;        // copy instructions
    static constexpr int BUF = PER_WAVE * 4096;
    static constexpr int LDS = 2 * BUF + EpiScaleBias<64>::kBytes;
};

template <typename T, typename TO, int ROWS, bool ROWS_OUT>
__device__ __forceinline__ void dense_strip_tile(const T* __restrict__ x, TO* __restrict__ y, const char* __restrict__ wfrag,
                                                 const char* __restrict__ zeros, int H, int W, int Ci, int Co, int co_blocks, int cb,
                                                 int n_img, int oh0, int ow0, const Epilogue& ep, char* smem)
{
    using P = DenseStrip<ROWS>;
    constexpr int RW = P::RW;
    float* const lds_ep = (float*)(smem + 2 * P::BUF);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), pair = wave >> 1, half = wave & 1;
    const int stages = Ci / 32;
    EpiScaleBias<64> scale_bias;
    scale_bias.load(ep, 64 * cb, Co, tid);

    const char* a_src = wfrag + (int64_t)(4 * cb + 2 * pair) * kDenseTileBytes + lane * 16;
    const int64_t a_stage = (int64_t)co_blocks * (4 * kDenseTileBytes);
    struct Column {
        u32x4 a[2][3];  // [tile][kh]
    };
    auto load_column = [&](Column& c, int stage, int kw) {
        const char* p = a_src + stage * a_stage + kw * kFragBytes;
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int kh = 0; kh < 3; ++kh) c.a[m][kh] = *(const u32x4*)(p + m * kDenseTileBytes + 3 * kh * kFragBytes);
    };
    Column column[3];  // of the stage; each is replaced by the next stage's behind its products
#pragma unroll
    for (int kw = 0; kw < 3; ++kw) load_column(column[kw], 0, kw);
    const char* x_ptr[P::PER_WAVE];
#pragma unroll
    for (int k = 0; k < P::PER_WAVE; ++k) {
        const int pos = (k * 4 + wave) * 16 + (lane >> 2);
        const int xr = pos / kLW, xc = pos % kLW;
        const int ih = oh0 - 1 + xr, iw = ow0 - 1 + xc;
        const bool inside = xr < ROWS + 2 && (unsigned)ih < (unsigned)H && (unsigned)iw < (unsigned)W;
        const int off = ((n_img * H + ih) * W + iw) * (Ci / 8) + (lane & 3);  // in 16-byte chunks (31 bits: strip3x3_plan)
        x_ptr[k] = inside ? (const char*)x + (int64_t)off * 16 : zeros;
    }
    u32x4 raw[P::PER_WAVE];
    auto load_activations = [&](int stage) {
#pragma unroll
        for (int k = 0; k < P::PER_WAVE; ++k) raw[k] = *(const u32x4*)(x_ptr[k] + stage * 64);
    };
    auto store_activations = [&](char* buf) {
#pragma unroll
        for (int k = 0; k < P::PER_WAVE; ++k) *(u32x4*)(buf + (k * 4 + wave) * 1024 + lane * 16) = raw[k];
    };
    load_activations(0);
    const int nn = lane & 15, qq = lane >> 4;
    f32x4 acc[2][RW];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int j = 0; j < RW; ++j) acc[m][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    store_activations(smem);
    scale_bias.store(lds_ep, ep, tid);
    for (int stage = 0; stage < stages; ++stage) {
        const int next = min(stage + 1, stages - 1);  // (behind the last stage: again, not used; a branch would make the waits coarser)
        char* const other = smem + ((stage & 1) ^ 1) * P::BUF;
        const char* X = smem + (stage & 1) * P::BUF + (half * RW * kLW + nn) * 64 + qq * 16;
        __syncthreads();  // the stage is in LDS; everybody is done with the other buffer
        static_for<3>([&](auto kw_tag) {
            constexpr int kw = decltype(kw_tag)::value;
            if constexpr (kw == 0) load_activations(next);
            auto row = [&](int i) { return *(const u32x4*)(X + (i * kLW + kw) * 64); };
            u32x4 b[3] = {row(0), row(1), row(2)};
            __builtin_amdgcn_sched_barrier(0);  // (the scheduler would move the loads down to where they are used)
#pragma unroll
            for (int i = 0; i < RW + 2; ++i) {
                const u32x4 r = b[i % 3];
#pragma unroll
                for (int kh = 0; kh < 3; ++kh) {
                    if (i < kh || i - kh >= RW) continue;
#pragma unroll
                    for (int m = 0; m < 2; ++m) acc[m][i - kh] = Dense16<T>::mma(column[kw].a[m][kh], r, acc[m][i - kh]);
                }
                if (i + 3 < RW + 2) b[i % 3] = row(i + 3);
                __builtin_amdgcn_sched_barrier(0);
            }
            load_column(column[kw], next, kw);
            if constexpr (kw == 2) store_activations(other);
            __builtin_amdgcn_sched_barrier(0);
        });
    }

    // ---- store: a lane holds 8 consecutive channels of one position per row ----
    const int co = 64 * cb + 16 * qq + 8 * pair, ow = ow0 + nn, oh = oh0 + half * RW;
    const bool live = co < Co && ow < W;  // (Co is a multiple of 16)
    // (ROWS_OUT: whole rows past the L2's write-back, as above, where the tiles are tall: 20 rows 2x256@100x168 34.2 -> 33.9 us,
    // 1x256@100x168 20.8 -> 20.4; 12 rows 4x128@60x80 9.4 -> 9.5)
    if (!ROWS_OUT && !live) return;
    if constexpr (ROWS_OUT) __syncthreads();  // everybody is done reading the last stage
    static_assert(ROWS * RowTile<TO>::kBytes <= 2 * P::BUF, "the outputs fit the buffers");
    const int64_t pos0 = ((int64_t)n_img * H + oh) * W + ow;
    auto finish = [&](auto shortcut_tag, auto form) {
        constexpr bool SHORTCUT = decltype(shortcut_tag)::value;
        EpiResidual<TO, 8> shortcut[RW];
        if constexpr (SHORTCUT) {
#pragma unroll
            for (int j = 0; j < RW; ++j)
                if (live && oh + j < H) shortcut[j].load(ep, pos0 + (int64_t)j * W, co);
        }
#pragma unroll
        for (int j = 0; j < RW; ++j) {
            if (oh + j >= H) break;
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = acc[e / 4][j][e % 4];
            epi_scale_bias_act_of<decltype(form)::value, 8>(v, ep, lds_ep + 16 * qq + 8 * pair, lds_ep + 64 + 16 * qq + 8 * pair);
            if constexpr (SHORTCUT) shortcut[j].add(v);
            TO* yp = y + (pos0 + (int64_t)j * W) * ep.ldy + co;
            if constexpr (sizeof(TO) == 4) {
#pragma unroll
                for (int g = 0; g < 2; ++g) *(f32x4*)(yp + 4 * g) = f32x4{v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
            } else {
                const u32x4 o = pack8_from_f32<TO>(v);
                if constexpr (ROWS_OUT) *(u32x4*)(smem + (half * RW + j) * RowTile<TO>::kBytes + RowTile<TO>::chunk_at(nn, 2 * qq + pair)) = o;
                else *(u32x4*)yp = o;
            }
        }
    };
    if (ep.residual) epi_by_form<false>(ep, [&](auto form) { finish(std::true_type{}, form); });
    else epi_by_form<false>(ep, [&](auto form) { finish(std::false_type{}, form); });
    if constexpr (ROWS_OUT) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < ROWS / 4; ++i) {
            const int r = wave + 4 * i;
            if (oh0 + r >= H) break;
            const auto base = store_base(y + (((int64_t)n_img * H + oh0 + r) * W + ow0) * ep.ldy + 64 * cb);
            RowTile<TO>::store(smem + r * RowTile<TO>::kBytes, lane, base, [&](int row, int c) {
                return ow0 + row < W && 64 * cb + 8 * c < Co ? (uint32_t)row * ep.ldy * 2 + c * 16 : kNoStore;
            });
        }
    }
}

// (fp32: dense3x3_f32.h, eight rows)
template <typename T, int ROWS> constexpr int dense_strip_lds = sizeof(T) == 4 ? F32Tile<1, ROWS>::LDS : DenseStrip<ROWS>::LDS;
template <typename T, typename TO, int ROWS, bool ROWS_OUT>
__device__ __forceinline__ void dense_strip_work(const T* __restrict__ x, TO* __restrict__ y, const char* __restrict__ wfrag,
                                                 const char* __restrict__ zeros, int H, int W, int Ci, int Co, WorkOrder order, const Epilogue& ep)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int work = order.item();
    if (work >= order.total) return;
    const int all_tile = order.co_blocks.quotient(work), co_blocks = order.co_blocks.by, cb = order.co_blocks.remainder(work, all_tile);
    const WorkOrder::Tile tile = order.tile(all_tile);
    const int n_img = tile.n_img, oh0 = tile.row * ROWS, ow0 = tile.col * kCols;
    if constexpr (sizeof(T) == 4) dense3x3_f32_tile<1, ROWS, false>(x, y, wfrag, zeros, H, W, Ci, Co, H, W, co_blocks, cb, n_img, oh0, ow0, ep, smem);
    else dense_strip_tile<T, TO, ROWS, ROWS_OUT>(x, y, wfrag, zeros, H, W, Ci, Co, co_blocks, cb, n_img, oh0, ow0, ep, smem);
}
template <typename T, typename TO, int ROWS>
__global__ __launch_bounds__(256, 2) void conv3x3_strip_kernel(const T* __restrict__ x, TO* __restrict__ y,
                                                               const char* __restrict__ wfrag, const char* __restrict__ zeros,
                                                               int H, int W, int Ci, int Co, WorkOrder order, Epilogue ep)
{
    dense_strip_work<T, TO, ROWS, false>(x, y, wfrag, zeros, H, W, Ci, Co, order, ep);
}
template <typename T, typename TO, int ROWS, bool ROWS_OUT>
__global__ __launch_bounds__(256, 2) void conv3x3_strip_kernel(const T* __restrict__ x, TO* __restrict__ y,
                                                               const char* __restrict__ wfrag, const char* __restrict__ zeros,
                                                               int H, int W, int Ci, int Co, WorkOrder order, Epilogue ep)
{
    dense_strip_work<T, TO, ROWS, ROWS_OUT>(x, y, wfrag, zeros, H, W, Ci, Co, order, ep);
}

template <typename T, typename TO, int ROWS, bool... ROWS_OUT>
rtoss_status launch_dense_rows(const rtoss_wdesc& d, const ConvParams& c, const char* wf, const char* zeros, const void* x, void* y, hipStream_t s)
{
    const int strips = (c.W + kCols - 1) / kCols, rows = (c.H + ROWS - 1) / ROWS, co_blocks = (d.Co + 63) / 64;
    auto kern = conv3x3_strip_kernel<T, TO, ROWS, ROWS_OUT...>;
    constexpr int lds = dense_strip_lds<T, ROWS>;
    static LaunchOnce lds_once;  // per instantiation
    if (rtoss_status st = ensure_dynamic_lds((const void*)kern, lds, lds_once, c.dev.device, "conv3x3 shared memory attribute")) return st;
    const int64_t total = (int64_t)strips * rows * co_blocks * c.N;  // (at most kMaxGridGroups: strip3x3_plan)
    const WorkOrder order(total, co_blocks, strips * rows, strips);
    kern<<<dim3(order.grid()), dim3(256), lds, s>>>((const T*)x, (TO*)y, wf, zeros, c.H, c.W, d.Ci, d.Co, order, c.ep);
    return check_hip(hipGetLastError(), "conv3x3 strip launch");
}

template <typename T, typename TO, int TN, int LAY, bool DB, bool... ROWS>
rtoss_status launch_rows(const rtoss_wdesc& d, const ConvParams& c, const char* wf, const char* zeros, const void* x, void* y, hipStream_t s)
{
    using P = Strip<TN, LAY, DB>;
    const int strips = (c.W + kCols - 1) / kCols, rows = (c.H + P::ROWS - 1) / P::ROWS;
    const int co_blocks = (d.Co + 63) / 64;
    auto kern = conv3x3_strip_kernel<T, TO, TN, LAY, DB, ROWS...>;
    static LaunchOnce lds_once;  // per instantiation
    if (rtoss_status st = ensure_dynamic_lds((const void*)kern, P::LDS, lds_once, c.dev.device, "conv3x3 shared memory attribute")) return st;
    const int64_t total = (int64_t)strips * rows * co_blocks * c.N;
    if (total > 0x3fffffff) return fail(RTOSS_ESHAPE, "conv: too many tiles");
    if ((int64_t)c.N * c.H * c.W * d.Ci * (int)sizeof(T) / 16 > 0x7fffffff) return fail(RTOSS_ESHAPE, "conv: input too large for 32-bit chunk offsets");
    const WorkOrder order(total, co_blocks, strips * rows, strips);
    dim3 grid(order.grid()), block(256);
    kern<<<grid, block, P::LDS, s>>>((const T*)x, (TO*)y, wf, zeros, c.H, c.W, d.Ci, d.Co,
                                     LAY == kDenseTaps ? kTM * co_blocks : padded_m_tiles(d.Co), order, c.ep);
    return check_hip(hipGetLastError(), "conv3x3 strip launch");
}

// Whether 16-bit outputs leave in rows past the L2's write-back, where a kernel has both ways: not where blocks of channels share
// sectors of memory (row_pieces.h; the dense mode, which gains least, by the pitch of a slice too), nor half-empty rows of up to 2 MB
// behind a single stage, where the detour through LDS costs more than it saves.  us from the registers, in rows, of tensors in caches,
// then of tensors in none:
//     64 -> 208, 4 taps, on 16x80x80               31.3 30.2   34.6 40.7     64 -> 64, 4 taps, on 16x80x80                11.5 10.4   15.4 14.0
//     128 -> 208, 5 taps, on 16x80x80              48.4 48.9   52.2 56.2     128 -> 128, 5 taps, on 16x80x80              31.1 30.3   33.7 33.6
//     ... slice of 128 of 144, SiLU, on 16x80x80   31.9 32.9   37.2 40.6     128 -> 128, 4 taps, slice of 144, 4x100x168  22.9 21.4   27.1 26.3
//     32 -> 32, 3 taps, on 16x28x28 (0.8 MB)       3.59 3.84   4.54 4.79     32 -> 32, slice of 48, SiLU, 4x100x168       6.83 6.38   9.27 7.95
inline bool rows_out(const rtoss_wdesc& d, const ConvParams& c, bool dense, const void* y)
{
    if (!stores_in_reach(c)) return false;
    if (d.Co <= 64) return d.Co == 64 || stage_count(d) > 1 || (int64_t)c.N * c.H * c.W * d.Co * 2 > 2 << 20;
    return dense ? whole_sectors(y, d.Co, c.ep.ldy, 2) : d.Co * 2 % kSector == 0;
}

template <typename T, typename TO, int TN, int LAY>
rtoss_status launch_one_buffer(const rtoss_wdesc& d, const ConvParams& c, const char* wf, const char* zeros, const void* x, void* y, hipStream_t s)
{
    if constexpr (sizeof(TO) == 2)
        if (rows_out(d, c, false, y)) return launch_rows<T, TO, TN, LAY, false, true>(d, c, wf, zeros, x, y, s);
    return launch_rows<T, TO, TN, LAY, false>(d, c, wf, zeros, x, y, s);
}

template <typename T, typename TO, int LAY>
rtoss_status launch_typed(const rtoss_wdesc& d, const ConvParams& c, int plan, const char* wf, const char* zeros, const void* x, void* y, hipStream_t s)
{
    switch (plan) {
    case 2: return launch_one_buffer<T, TO, 2, LAY>(d, c, wf, zeros, x, y, s);
    case 3: if constexpr (LAY != 0) return launch_one_buffer<T, TO, 3, LAY>(d, c, wf, zeros, x, y, s); else break;
    case 4: return launch_one_buffer<T, TO, 4, LAY>(d, c, wf, zeros, x, y, s);
    case 5: if constexpr (LAY != 0) return launch_one_buffer<T, TO, 5, LAY>(d, c, wf, zeros, x, y, s); else break;
    case 2 + kTwoBuffers: if constexpr (LAY != kDenseTaps) return launch_rows<T, TO, 2, LAY, true>(d, c, wf, zeros, x, y, s); else break;
    case 3 + kTwoBuffers: if constexpr (LAY == 0) return launch_rows<T, TO, 3, LAY, true>(d, c, wf, zeros, x, y, s); else break;
    }
    return fail(RTOSS_EINVAL, "conv: unknown strip plan %d", plan);
}

template <typename T, typename TO>
rtoss_status launch_dense(const rtoss_wdesc& d, const ConvParams& c, int rows, const char* wf, const char* zeros, const void* x, void* y, hipStream_t s)
{
    if constexpr (sizeof(T) == 2 && sizeof(TO) == 2) {
        if (rows == 16 && rows_out(d, c, true, y)) return launch_dense_rows<T, TO, 16, true>(d, c, wf, zeros, x, y, s);
        if (rows == 20 && rows_out(d, c, true, y)) return launch_dense_rows<T, TO, 20, true>(d, c, wf, zeros, x, y, s);
    }
    switch (rows) {
    case 8: return launch_dense_rows<T, TO, 8>(d, c, wf, zeros, x, y, s);
    case 12: if constexpr (sizeof(T) == 2) return launch_dense_rows<T, TO, 12>(d, c, wf, zeros, x, y, s); else break;
    case 16: if constexpr (sizeof(T) == 2) return launch_dense_rows<T, TO, 16>(d, c, wf, zeros, x, y, s); else break;
    case 20: if constexpr (sizeof(T) == 2) return launch_dense_rows<T, TO, 20>(d, c, wf, zeros, x, y, s); else break;
    }
    return fail(RTOSS_EINVAL, "conv: unknown strip plan of %d rows", rows);
}

template <int LAY>
rtoss_status launch_layout(const rtoss_wdesc& d, const ConvParams& c, int plan, const char* wf, const char* zeros, const void* x, void* y, hipStream_t s)
{
    const bool f32out = c.out_dt == RTOSS_F32;
    if constexpr (LAY == kDenseTaps)
        if (plan > kDenseRows) {
            const int rows = plan - kDenseRows;
            if (d.dt == RTOSS_F32) return launch_dense<float, float>(d, c, rows, wf, zeros, x, y, s);
            if (d.dt == RTOSS_F16) return f32out ? launch_dense<f16_t, float>(d, c, rows, wf, zeros, x, y, s) : launch_dense<f16_t, f16_t>(d, c, rows, wf, zeros, x, y, s);
            return f32out ? launch_dense<bf16_t, float>(d, c, rows, wf, zeros, x, y, s) : launch_dense<bf16_t, bf16_t>(d, c, rows, wf, zeros, x, y, s);
        }
    if (d.dt == RTOSS_F16)
        return f32out ? launch_typed<f16_t, float, LAY>(d, c, plan, wf, zeros, x, y, s) : launch_typed<f16_t, f16_t, LAY>(d, c, plan, wf, zeros, x, y, s);
    return f32out ? launch_typed<bf16_t, float, LAY>(d, c, plan, wf, zeros, x, y, s) : launch_typed<bf16_t, bf16_t, LAY>(d, c, plan, wf, zeros, x, y, s);
}

}  // namespace

// When a launch belongs here, and with how many rows per wave.  The time of a launch is set by how many rounds of
// workgroups it takes (two per compute unit at once) and the depth of the layer; measured per stage with the chip filled
// once / twice: TN = 2 0.88 / 1.45 us, 3 1.12 / 1.85, 4 1.6 / 3.1, plus 3 us.  So: the smallest TN whose workgroups fit
// one round.  (bf16, layout 0, batch x channels @ image: 1x256@100x168 18.0 us with TN = 3, 23.2 with the single-buffered
// kernel; 4x128@60x70 8.0 and 9.6; 16x128@40x40 9.2 and 10.3; 4x64@112x130 7.3 and 8.0.  Layout 1: 2x256@100x168 33.6 and
// 40.3.  Dense mode: below.)
static int plan_within_limits(const rtoss_wdesc& d, const ConvParams& c, int layout);

int strip3x3_rows(int plan) { return plan > kDenseRows ? plan - kDenseRows : 4 * (plan % kTwoBuffers); }

int strip3x3_plan(const rtoss_wdesc& d, const ConvParams& c, int layout)
{
    if (c.stride != 1 || d.Ci * elem_bytes(d.dt) % 64 || d.Co % 16) return 0;
    // (the dense-mode kernel has neither limit)
    const int plan = plan_within_limits(d, c, layout);
    const int rows = strip3x3_rows(plan);
    if (plan == 0 || (int64_t)c.N * c.H * c.W * d.Ci * elem_bytes(d.dt) / 16 > kMaxChunks) return 0;
    // (fp32, and 16-bit results of two buffers, know rows only)
    const bool two_buffers = plan < kDenseRows && plan > kTwoBuffers;
    if (!stores_in_reach(c) && (d.dt == RTOSS_F32 || (two_buffers && c.out_dt != RTOSS_F32))) return 0;
    return (int64_t)((c.W + kCols - 1) / kCols) * ((c.H + rows - 1) / rows) * ((d.Co + 63) / 64) * c.N <= kMaxGridGroups ? plan : 0;
}

static int plan_within_limits(const rtoss_wdesc& d, const ConvParams& c, int layout)
{
    const DeviceInfo& dev = c.dev;
    const int64_t cus = dev.cus;
    const int stages = stage_count(d);
    const auto groups = [&](int tn) {
        return (int64_t)((c.W + kCols - 1) / kCols) * ((c.H + 4 * tn - 1) / (4 * tn)) * ((d.Co + 63) / 64) * c.N;
    };
    if (d.dt == RTOSS_F32) {
        // Eight rows from six workgroups per four compute units on; below that the dense-mode kernel's shorter tiles spread the
        // work better (timings, and why sums of few products stay out: f32_rows there).
        if (few_live_products(d)) return 0;
        return 2 * groups(2) >= 3 * cus ? kDenseRows + 8 : 0;
    }
    // shallow narrow launches of the dense mode: its own 16-channel tiles
    if (layout == kDenseTaps && groups(2) <= cus / 2) return 0;
    if (layout == kDenseTaps && (stages > 2 || (stages == 2 && groups(2) <= cus))) {
        // Weights past LDS: the height with the fewest rows per compute unit, three more counted for a tile's start and end
        // (us, weights through LDS and past it with 8 / 12 / 16 / 20 rows, bf16):
        //     1x256@100x168 25.7  25.4 24.6 28.6 22.6    1x128@80x100 8.5   7.3  8.5 10.3 11.6    3x96@100x140 11.9  12.5 11.9 14.0 16.1
        //     2x256@100x168 40.5  44.5 43.5 43.6 39.0    4x128@60x80 10.7  10.9  9.0 11.1 12.4    1x256@50x84  13.7  10.4 12.8 16.3 18.8
        //     4x256@100x168 72.4  77.6 73.6 73.0 67.0    2x192@70x90 15.3  13.5 11.4 14.2 16.2
        // Shallow launches of several tiles per compute unit keep the smaller registers (4x64@112x140 8.3  8.7 9.5 8.7 9.5).
        int best = 0;
        int64_t cost = 0;
        for (const int rows : {20, 16, 12, 8}) {
            const int64_t tiles = (int64_t)((c.W + kCols - 1) / kCols) * ((c.H + rows - 1) / rows) * ((d.Co + 63) / 64) * c.N;
            const int64_t rounds = (tiles + cus - 1) / cus * (rows + 3);
            if (best == 0 || rounds < cost) best = rows, cost = rounds;
        }
        return kDenseRows + best;
    }
    if (stages == 1) return groups(2) <= 4 * cus ? 2 : 0;  // (nothing to fetch ahead: four workgroups per compute unit)
    if (groups(2) <= 2 * cus) {
        if (layout == 0 && groups(2) > cus && groups(3) <= cus) return 3 + kTwoBuffers;
        return layout != kDenseTaps ? 2 + kTwoBuffers : 2;  // (dense mode: two buffers fit once)
    }
    if (groups(3) <= 2 * cus) return layout == 0 ? 3 + kTwoBuffers : 3;
    if (groups(4) <= 2 * cus) return 4;
    if (layout == 0) return 0;  // several rounds: the single-buffered kernel's four workgroups per compute unit
    // several rounds: the height that pads the image least, the taller one on a tie
    return (c.H + 19) / 20 * 20 <= (c.H + 15) / 16 * 16 || groups(5) <= 2 * cus ? 5 : 4;
}

rtoss_status launch_conv3x3_strip(const rtoss_wdesc& d, const ConvParams& c, int layout, int plan, const void* section, const void* zeros,
                                  const void* x, void* y, hipStream_t s)
{
    const char *wf = (const char*)section, *z = (const char*)zeros;
    if (layout == kDenseTaps) return launch_layout<kDenseTaps>(d, c, plan, wf, z, x, y, s);
    return layout == 1 ? launch_layout<1>(d, c, plan, wf, z, x, y, s) : launch_layout<0>(d, c, plan, wf, z, x, y, s);
}

}  // namespace rtoss
