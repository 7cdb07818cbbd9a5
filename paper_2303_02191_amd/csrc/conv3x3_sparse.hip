// 3x3 pattern-sparse convolution on the CDNA4 matrix cores (fp16 / bf16, fp32 accumulate).
//
// Why 2-of-4 structured sparsity fits pattern pruning (Section IV.B / IV.C): every kernel
// keeps k taps chosen per kernel, so at matrix-tile granularity the zeros are unstructured
// and a dense contraction cannot skip them.  The sparse matrix instruction
// (v_smfmac_f32_16x16x64) accepts a per-row choice of 2 live values in every 4 K-slots.
// For one input channel the 9 taps are split into the 4 corners {0,2,6,8}, the 4 edge
// midpoints {1,3,5,7} and the centre {4}.  Whenever every dictionary pattern has at most
// 2 corners and at most 2 edge midpoints (true for all edge-connected 2- and 3-entry
// patterns: a connected path alternates between the two classes), the corner slots and
// the edge slots of a channel are each one legal 2-of-4 group, and the centre tap is a
// plain dense K-slot.  Per 32 input channels this costs 2+2 sparse steps and 1 dense step
// instead of 9 dense steps.
//
// Instruction operand layout (wave64; r = lane % 16, q = lane / 16):
//   dense  v_mfma_f32_16x16x32:  A lane holds row r, K = 8q .. 8q+7; B lane holds column r,
//          K = 8q .. 8q+7; D lane holds column r, rows 4q .. 4q+3.
//   sparse v_smfmac_f32_16x16x64: A lane holds 8 compressed values of row r in 4 pairs;
//          pair g refers to the 4 B-values (column = any, B lane group 2*(q&1) + (g>>1),
//          B elements 8*(q>>1) + 4*(g&1) .. +3); the two 2-bit fields at bits 4g and 4g+2
//          of the 16-bit index say which of the 4 each compressed value multiplies.
//          ABID selects the low (0) or high (1) half of the index register.
//
// Data flow of one workgroup (256 lanes = 4 waves): output tile = 16*TM output channels x
// (RT x CT) blocks of 4x4 output positions; every wave owns all 16*TM channels and TN of
// the position blocks.  K runs over stages of 32 input channels: the stage's weight
// fragments (one contiguous chunk of the packed blob) and its activation tile with halo
// (channels-last, 32 channels per position, 64 bytes) are copied global ->
// LDS without passing through registers.  B operands are read from LDS as 16-byte vectors
// (8 channels of one tap) and the 4x4 (tap, channel) blocks are transposed in registers
// with byte permutes so that one lane holds, for 4 channels, the 4 taps of a group.
//
// This file holds the single-buffered kernel (stride 2, but for shallow layers in large launches, which have one of their own
// here; ragged channel counts, and stride-1 layers of up to 64 input or output channels in launches of many rounds): a plain
// loop nest with small tiles, several workgroups per compute unit.
// Large stride-1 layers take the pipelined kernel of conv3x3_rows.hip, launches of medium size the strips of conv3x3_ring.hip and
// conv3x3_strip.hip, and those that cannot fill the chip conv3x3_ksplit.hip; all read the same packed section.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "dtypes.h"
#include "epilogue.h"
#include "mma.h"
#include "rows_plan.h"
#include "sparse_frag.h"
#include "work_order.h"
#include "tile3x3.h"

namespace rtoss {

namespace {

// Stride 2.  An output position needs four input positions, so blocks of 4x4 output positions share little: a wave takes its TN
// blocks from the list of all blocks of the launch, wherever they lie, and copies 9x9 input positions for each.  A tile of
// 8x8 or 4x16 positions for the workgroup copies 5 to 12 % less, but pads the image: 20x20 outputs are 25 blocks, or 9 tiles of four
// (256 -> 256 channels at 40x40, 16 images: 18.6 us with tiles, now 12.7; the tile's pitch of 80 bytes against bank conflicts
// was 25 % more copies besides: 32 -> 64 at 112x140 4.4 us, now 3.8).
// In LDS the even input columns of a row come first, so that a tap's reads are contiguous, and the 16-byte chunks of a
// position are in reverse order in every other pair of rows.  A 16-byte read is served in passes of 16 lanes -- 0-3, 12-15,
// 20-27, then 4-11, 16-19, 28-31, ... -- and so no two lanes of a pass meet in a bank.
constexpr int kPatch = 81 * 64;
constexpr int patch_copies(int TN) { return (TN * kPatch + 1023) / 1024; }

// Single-buffered kernel: one LDS buffer, two barriers per stage, plain loop nest scheduled by the
// compiler.  It needs half the LDS of the pipelined kernel (conv3x3_rows.hip) and few registers, so several
// workgroups share a compute unit and hide each other's copy latency and epilogue.  Used for stride 2, for ragged channel
// counts and for layers too shallow or narrow for the pipelined kernel's 128-channel, 8-stage appetite: TM = 4 covers 64
// output channels per workgroup.
// LAY: tap layout (sparse_frag.h).  Layout 1 (4 and 5 entries) has three tap groups and no dense centre
// step; it always takes the one-group-at-a-time schedule.
// DB: two LDS buffers; the copies of the next stage are issued right after the barrier that opens a stage and land
// while it is multiplied (one barrier per stage).  For deep stride-1 layers, whose schedule with operand reads ahead
// is held to two workgroups per compute unit by its registers anyway: two buffers of 38 KB each still fit twice.
// RAG: channel counts that are no multiples of 32 (in; a multiple of 8, so that rows stay 16-byte aligned) or 16
// (out): the last stage's copy lanes past the row end read the block of zeros, and outputs are stored under a
// per-channel bound.
template <typename T, typename TO, int S, int TM, int TN, int RT, int CT, bool AHEAD, int LAY = 0, bool DB = false, bool RAG = false>
__global__ __launch_bounds__(256) void conv3x3_sparse_sb_kernel(const T* __restrict__ x, TO* __restrict__ y,
                                                                const char* __restrict__ wfrag,
                                                                const char* __restrict__ zeros, int H, int W, int Ci,
                                                                int Co, int Ho, int Wo, int m_tiles_total,
                                                                WorkOrder order, int blocks, Epilogue ep)
{
    using G = Geom<S, RT, CT>;
    static_assert(RT * CT == 4 * TN, "four waves share the position blocks of a workgroup");
    constexpr bool PATCH = S == 2;
    constexpr TapLayout LY = kLayouts[LAY];
    constexpr int NG = LY.groups, FR = layout_fragments(LY), TILE = layout_tile_bytes(LY);
    constexpr int A_BYTES = TM * TILE;
    constexpr int A_WAVE_COPIES = A_BYTES / 1024;            // 64 lanes x 16 B per copy instruction
    constexpr int A_PER_WAVE = (A_WAVE_COPIES + 3) / 4;
    constexpr int X_CHUNKS = G::x_bytes / 16;                // (stride 1)
    constexpr int X_PER_WAVE = PATCH ? patch_copies(TN) : ((X_CHUNKS + 63) / 64 + 3) / 4;
    static_assert(A_BYTES % 1024 == 0, "weight fragments are whole copy instructions");
    extern __shared__ __attribute__((aligned(16))) char smem[];  // [weights][activations, rounded up to whole copies] (x2 with DB)
    constexpr int BUF = A_BYTES + X_PER_WAVE * 4096;
    char* lds_a = smem;
    char* lds_x = smem + A_BYTES;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int work = order.item();
    if (work >= order.total) return;
    const int all_tile = order.co_blocks.quotient(work), mt0 = order.co_blocks.remainder(work, all_tile) * TM;
    // this wave's blocks of 4x4 output positions
    int n_of[TN], oh_of[TN], ow_of[TN];
    bool live[TN];
    const WorkOrder::Tile tile = order.tile(all_tile);  // (stride 1)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        if constexpr (PATCH) {  // (the order's tiles are blocks)
            const int blk = all_tile * (4 * TN) + wave * TN + j;
            const WorkOrder::Tile at = order.tile(blk);
            live[j] = blk < blocks;
            n_of[j] = at.n_img;
            oh_of[j] = 4 * at.row;
            ow_of[j] = 4 * at.col;
        } else {
            const int blk = wave * TN + j;
            live[j] = true;
            n_of[j] = tile.n_img;
            oh_of[j] = tile.row * G::TH + 4 * (blk / CT);
            ow_of[j] = tile.col * G::TW + 4 * (blk % CT);
        }
    }
    const int stages = RAG ? (Ci + 31) / 32 : Ci / 32;

    const char* a_src = wfrag + (int64_t)mt0 * TILE + lane * 16;
    const int64_t a_stage_stride = (int64_t)m_tiles_total * TILE;
    auto issue_weight_copies = [&](int stage, char* buf) {
#pragma unroll
        for (int k = 0; k < A_PER_WAVE; ++k)
            if (k * 4 + wave < A_WAVE_COPIES)  // wave-uniform
                copy16_to_lds(a_src + stage * a_stage_stride + (k * 4 + wave) * 1024, buf + (k * 4 + wave) * 1024);
    };
    // (the weight fragments of stage 0 need only the channel block: they are under way while the lanes work out
    // their activation sources)
    float* lds_ep = (float*)(smem + (DB ? 2 : 1) * BUF);  // scale and bias of the workgroup's channels
    EpiScaleBias<16 * TM> scale_bias;
    scale_bias.load(ep, 16 * mt0, Co, tid);
    issue_weight_copies(0, smem);

    // Copy sources of stage 0.  Every lane copies 16 bytes in every copy instruction; a lane whose LDS
    // slot is zero padding of the tile (or a pad chunk) reads the block of zeros behind the fragments.
    const char* x_ptr[X_PER_WAVE];
    static_assert(X_PER_WAVE <= 32, "one bit per copy");
    unsigned tail_ok = 0;  // RAG: bit k = the last stage still has channels at this lane's copy k
#pragma unroll
    for (int k = 0; k < X_PER_WAVE; ++k) {
        int n, ih, iw, q;
        bool inside;
        if constexpr (PATCH) {
            const int c = k * 64 + lane, pos = c / 4 % 81, r = pos / 9, i = pos % 9;
            const bool second = TN == 2 && c >= kPatch / 16;
            q = (c & 3) ^ (r & 2 ? 3 : 0);
            n = second ? n_of[TN - 1] : n_of[0];
            ih = (second ? oh_of[TN - 1] : oh_of[0]) * 2 - 1 + r;
            iw = (second ? ow_of[TN - 1] : ow_of[0]) * 2 - 1 + (i < 5 ? 2 * i : 2 * i - 9);  // even columns first
            inside = c < TN * kPatch / 16 && (second ? live[TN - 1] : live[0]);
        } else {
            const int c = (k * 4 + wave) * 64 + lane, pos = c / G::kChunks;
            q = c % G::kChunks;
            n = n_of[0];
            ih = tile.row * G::TH - 1 + pos / G::LW;
            iw = tile.col * G::TW - 1 + pos % G::LW;
            inside = pos / G::LW < G::IH && pos % G::LW < G::IW;
        }
        if (RAG && (stages - 1) * 32 + 8 * q < Ci) tail_ok |= 1u << k;
        inside = inside && (unsigned)ih < (unsigned)H && (unsigned)iw < (unsigned)W;
        // offset in 16-byte chunks: fits 31 bits (checked by the launcher)
        const int off = ((n * H + ih) * W + iw) * (Ci >> 3) + q;
        x_ptr[k] = inside ? (const char*)x + (int64_t)off * 16 : zeros;
    }

    // ---- per-lane read addresses of the B operand ----
    const int nn = lane & 15, qq = lane >> 4;
    const int pr = nn >> 2, pc = nn & 3;
    // byte offset in lds_x of this lane's output position for each of its blocks, tap (0,0) (stride 2: kernel rows 0 and 1, row 2)
    int xb[TN][PATCH ? 2 : 1];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        if constexpr (PATCH) {
            const int at = wave * (X_PER_WAVE * 1024) + j * kPatch + (2 * pr * 9 + pc) * 64;
            xb[j][0] = at + (pr & 1 ? 3 - qq : qq) * 16;
            xb[j][1] = at + (pr & 1 ? qq : 3 - qq) * 16;
        } else {
            const int blk = wave * TN + j;
            xb[j][0] = ((4 * (blk / CT) + pr) * G::LW + 4 * (blk % CT) + pc) * G::kPos + qq * 16;
        }
    }
    auto read_tap = [&](int j, int t) {
        const int kh = t / 3, kw = t % 3;
        if constexpr (PATCH) return *(const u32x4*)(lds_x + xb[j][kh >> 1] + (kh * 9 + (kw & 1 ? 5 : kw >> 1)) * 64);
        else return *(const u32x4*)(lds_x + xb[j][0] + (kh * G::LW + kw) * G::kPos);
    };

    f32x4 acc[TM][TN];
    // (no clearing of the accumulators: the centre step comes first in a stage, and the first stage's
    // writes a * b instead of adding to it)
    auto issue_copies = [&](int stage, char* buf, bool with_weights) {
        if (with_weights) issue_weight_copies(stage, buf);
#pragma unroll
        for (int k = 0; k < X_PER_WAVE; ++k) {
            const char* src = x_ptr[k] + stage * 64;
            if (RAG && stage == stages - 1 && !(tail_ok >> k & 1u)) src = zeros;
            copy16_to_lds(src, buf + A_BYTES + (PATCH ? wave * X_PER_WAVE + k : k * 4 + wave) * 1024);
        }
    };
    if constexpr (DB) issue_copies(0, smem, false);
    auto run_stage = [&](auto first_tag, int stage) {
        constexpr bool FIRST = decltype(first_tag)::value;
        if constexpr (DB) {
            __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this wave's copies of this stage have landed in LDS
            if constexpr (FIRST) scale_bias.store(lds_ep, ep, tid);
            __syncthreads();                     // ... and everybody's; and every wave is done reading the other buffer
            const int par = stage & 1;
            if (stage + 1 < stages) issue_copies(stage + 1, smem + (par ^ 1) * BUF, true);
            lds_a = smem + par * BUF;
            lds_x = lds_a + A_BYTES;
        } else {
            __syncthreads();  // every wave is done reading the previous stage
            issue_copies(stage, smem, !FIRST);  // (stage 0's weight fragments are already under way)
            __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this wave's copies have landed in LDS
            if constexpr (FIRST) scale_bias.store(lds_ep, ep, tid);
            __syncthreads();                     // ... and everybody's
        }

        // AHEAD: operand reads run ahead of the matrix instructions that use them: the centre step's and
        // the corner group's are issued together, the edge group's behind the centre step.  (The matrix
        // instructions are asm statements that loads are not moved across: source order is issue order.)
        // This hides the LDS latency inside a workgroup; shallow layers over large images, which live on
        // hiding HBM latency across workgroups, do better without it and with the registers it costs.
        u32x4 bc[TN], ac[TM];
        u32x4 rr[NG][TN][4], as[NG][TM][2];
        int iw2[NG][TM];
        auto load_group_x = [&](int group) {
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int f = 0; f < 4; ++f) {
                    const int t = LY.tap[group][f];
                    rr[group][j][f] = read_tap(j, t);
                }
        };
        auto load_group_a = [&](int group, int m) {
            const char* at = lds_a + m * TILE;
            iw2[group][m] = *(const int*)(at + FR * kFragBytes + (group * 64 + lane) * 4);
            as[group][m][0] = *(const u32x4*)(at + (group * 2 + 0) * kFragBytes + lane * 16);
            as[group][m][1] = *(const u32x4*)(at + (group * 2 + 1) * kFragBytes + lane * 16);
        };
        auto load_group = [&](int group) {
            load_group_x(group);
#pragma unroll
            for (int m = 0; m < TM; ++m) load_group_a(group, m);
        };
        u32x8 bf[2][TN];  // B operands of both sparse steps of a tap group
        auto permute_group = [&](int group) {
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int half = 0; half < 2; ++half) bf[half][j] = sparse_operand(rr[group][j], half);
        };
        auto multiply_group = [&](int group, int m) {
#pragma unroll
            for (int j = 0; j < TN; ++j) MatV<T>::template sparse<0>(as[group][m][0], bf[0][j], acc[m][j], iw2[group][m]);
#pragma unroll
            for (int j = 0; j < TN; ++j) MatV<T>::template sparse<1>(as[group][m][1], bf[1][j], acc[m][j], iw2[group][m]);
        };
        auto run_group = [&](int group) {
            permute_group(group);
#pragma unroll
            for (int m = 0; m < TM; ++m) multiply_group(group, m);
        };
        auto load_centre = [&]() {
#pragma unroll
            for (int j = 0; j < TN; ++j) bc[j] = read_tap(j, 4);
#pragma unroll
            for (int m = 0; m < TM; ++m) ac[m] = *(const u32x4*)(lds_a + m * TILE + 2 * NG * kFragBytes + lane * 16);
        };
        auto run_centre = [&]() {  // centre tap: dense step over the 32 channels of the stage
#pragma unroll
            for (int m = 0; m < TM; ++m)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    if constexpr (FIRST) MatV<T>::dense_first(ac[m], bc[j], acc[m][j]);
                    else MatV<T>::dense(ac[m], bc[j], acc[m][j]);
                }
        };
        if constexpr (AHEAD && LAY == 0) {
            load_centre();
            load_group(0);
            run_centre();
            load_group(1);
            run_group(0);
            run_group(1);
        } else {  // few operands live at a time: fewer registers, one more workgroup per compute unit
            if constexpr (LY.centre) {
                load_centre();
                run_centre();
            } else if constexpr (FIRST) {  // (no dense step that could write the first product: clear)
#pragma unroll
                for (int m = 0; m < TM; ++m)
#pragma unroll
                    for (int j = 0; j < TN; ++j) acc[m][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int group = 0; group < NG; ++group) {
                load_group_x(group);
                permute_group(group);
#pragma unroll
                for (int m = 0; m < TM; ++m) {
                    load_group_a(group, m);
                    multiply_group(group, m);
                }
            }
        }
    };
    run_stage(std::true_type{}, 0);
    for (int stage = 1; stage < stages; ++stage) run_stage(std::false_type{}, stage);

    // the last matrix instructions must have written their accumulators before anything reads them
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    // ---- epilogue: a D lane holds column nn (position) and rows 4*qq .. 4*qq+3 of every channel tile,
    // which tile_row_channel makes 16 consecutive output channels per group of 4 tiles ----
    static_assert(TM % 4 == 0, "whole groups of 4 channel tiles");
    auto finish = [&](auto shortcut_tag, auto form) {
        constexpr bool SHORTCUT = decltype(shortcut_tag)::value;
        EpiResidual<TO, 16> shortcut[TN][TM / 4];
        if constexpr (SHORTCUT) {  // its loads go out together, before any of them is needed
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int oh = oh_of[j] + pr, ow = ow_of[j] + pc;
#pragma unroll
                for (int mg = 0; mg < TM; mg += 4) {
                    const int co = 16 * mt0 + tile_quarter_offset(mg, qq);
                    if (live[j] && oh < Ho && ow < Wo && co < Co) shortcut[j][mg / 4].load(ep, ((int64_t)n_of[j] * Ho + oh) * Wo + ow, co);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            if (!live[j]) continue;  // uniform
            const int oh = oh_of[j] + pr, ow = ow_of[j] + pc;
            const bool row_inside = oh < Ho, inside = row_inside && ow < Wo;
            const int64_t pos = ((int64_t)n_of[j] * Ho + oh) * Wo + ow;
            TO* yp = y + pos * ep.ldy;
#pragma unroll
            for (int mg = 0; mg < TM; mg += 4) {
                const int co = 16 * mt0 + tile_quarter_offset(mg, qq);
                const bool mine = inside && co < Co;  // (not RAG: Co is a multiple of 16, a run of 16 channels is all in or all out)
                float vv[16];
#pragma unroll
                for (int m = 0; m < 4; ++m)
#pragma unroll
                    for (int e = 0; e < 4; ++e) vv[4 * m + e] = acc[mg + m][j][e];
                if constexpr (RAG) {
                    if (!mine) continue;
                    epi_ragged<TO, 16>(vv, ep, pos, co, Co);
                    store_ragged<TO, 16>(yp, vv, co, Co, ep.ldy);
                    continue;
                }
                epi_scale_bias_act_of<decltype(form)::value, 16>(vv, ep, lds_ep + co - 16 * mt0, lds_ep + 16 * TM + co - 16 * mt0);
                if constexpr (SHORTCUT) shortcut[j][mg / 4].add(vv);
                if constexpr (sizeof(TO) == 4) {
                    if (!mine) continue;
#pragma unroll
                    for (int g = 0; g < 4; ++g) *(f32x4*)(yp + co + 4 * g) = f32x4{vv[4 * g], vv[4 * g + 1], vv[4 * g + 2], vv[4 * g + 3]};
                } else {
                    u32x4 o[2] = {pack8_from_f32<TO>(vv), pack8_from_f32<TO>(vv + 8)};
                    if constexpr (!PATCH) {
                        if (!mine) continue;
#pragma unroll
                        for (int g = 0; g < 2; ++g) *(u32x4*)(yp + co + 8 * g) = o[g];
                        continue;
                    }
                    // stride 2: rows of 128 bytes past the L2's write-back (us before, with, 16 images with SiLU, tensors in caches, then in
                    // none: 128 -> 256 @ 80 24.7 23.2, 31.7 31.4, 256 -> 512 @ 40 19.6 19.0, 25.8 26.0; not at stride 1: 32 -> 32 @ 160 in a
                    // 57-layer forward 25.5 26.4)
                    const int odd = lane & 1;  // (the column's parity too)
                    pair_pieces(o[0], o[1], odd);
                    const bool row = row_inside && co < Co;
                    TO* yc = yp - odd * (int64_t)ep.ldy + co + 8 * odd;
                    if (row && ow - odd < Wo) store16_through(yc, o[0]);
                    if (row && ow - odd + 1 < Wo) store16_through(yc + ep.ldy, o[1]);
                }
            }
        }
    };
    if constexpr (RAG) finish(std::false_type{}, std::integral_constant<int, kEpiAny>{});
    else if (ep.residual) epi_by_form(ep, [&](auto form) { finish(std::true_type{}, form); });
    else epi_by_form(ep, [&](auto form) { finish(std::false_type{}, form); });
}

// Stride 2, layers of one or two stages of input channels in large launches: half of what the kernel above copies for 64
// positions is weights, and its workgroups are chains of copy, products and stores.  Here a workgroup keeps the weights of its 64
// channels, and its waves go over blocks of 4x4 positions by themselves, without a barrier: while a wave multiplies a stage's
// 9x9 patch, the next one is on its way into a buffer of its own.  With SiLU, tensors in no cache: 32 -> 64 on 16x320x320 42.9 ->
// 34.7 us (4.5 TB/s, the rate of a copy), 64 -> 128 on 16x160x160 34.0 -> 27.7: bound by the instructions around the products there
// (block numbers by division instead of addition 4 % more, three buffers a wave 7 %).
template <int STAGES> struct Resident {
    static constexpr int WAVES = 8, BUFS = 2;
    static constexpr int A_BYTES = 4 * layout_tile_bytes(kLayouts[0]);
    static constexpr int COPIES = patch_copies(1);
    static constexpr int LDS = STAGES * A_BYTES + WAVES * BUFS * kPatch + EpiScaleBias<64>::kBytes;
    static_assert(LDS <= 160 * 1024 && A_BYTES % 1024 == 0, "a compute unit's LDS");
};

template <typename T, int STAGES>
__global__ __launch_bounds__(64 * Resident<STAGES>::WAVES) __attribute__((amdgpu_waves_per_eu(2, 2)))
void conv3x3_resident_kernel(const T* __restrict__ x, T* __restrict__ y, const char* __restrict__ wfrag, const char* __restrict__ zeros, int H, int W,
                             int Co, int Ho, int Wo, int m_tiles_total, int blocks_c, int blocks_per_image, int co_blocks, int blocks,
                             int blocks_per_xcd, Epilogue ep)
{
    using R = Resident<STAGES>;
    constexpr TapLayout LY = kLayouts[0];
    constexpr int TILE = layout_tile_bytes(LY), FR = layout_fragments(LY), NG = LY.groups, CHUNKS = 4 * STAGES;  // 16-byte chunks of a position
    extern __shared__ __attribute__((aligned(16))) char smem[];  // [weights of all stages][each wave's buffers][scale, bias]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Workgroups are dealt to the 8 XCDs in turn; each XCD takes a contiguous range of blocks, the channel blocks next to each other.
    const int xcd = blockIdx.x % 8, slot = blockIdx.x / 8, cb = slot % co_blocks;
    const int step = (gridDim.x / 8 / co_blocks) * R::WAVES, end = min(blocks, (xcd + 1) * blocks_per_xcd);
    int blk = xcd * blocks_per_xcd + slot / co_blocks * R::WAVES + wave;

    float* lds_ep = (float*)(smem + STAGES * R::A_BYTES + R::WAVES * R::BUFS * kPatch);
    EpiScaleBias<64> scale_bias;
    scale_bias.load(ep, 64 * cb, Co, tid);
    for (int k = wave; k < STAGES * (R::A_BYTES / 1024); k += R::WAVES) {
        const int stage = k / (R::A_BYTES / 1024), part = k % (R::A_BYTES / 1024);
        copy16_to_lds(wfrag + ((int64_t)stage * m_tiles_total + 4 * cb) * TILE + part * 1024 + lane * 16, smem + k * 1024);
    }
    // ---- a lane's sources relative to a block's first input position (the layout in LDS: conv3x3_sparse_sb_kernel) ----
    char* const mine = smem + STAGES * R::A_BYTES + wave * (R::BUFS * kPatch);
    int rel[R::COPIES], row_of[R::COPIES], col_of[R::COPIES];
#pragma unroll
    for (int k = 0; k < R::COPIES; ++k) {
        const int c = k * 64 + lane, pos = c / 4 % 81, r = pos / 9, i = pos % 9;  // (past the patch: any of its positions)
        row_of[k] = r - 1;
        col_of[k] = (i < 5 ? 2 * i : 2 * i - 9) - 1;
        rel[k] = (row_of[k] * W + col_of[k]) * CHUNKS + ((c & 3) ^ (r & 2 ? 3 : 0));
    }
    // this wave's block: image, row and column of blocks (advanced by additions: a division is some forty scalar instructions)
    struct Block { int n, r, c; };
    const auto block_at = [&](int b) { return Block{b / blocks_per_image, b % blocks_per_image / blocks_c, b % blocks_per_image % blocks_c}; };
    const int blocks_r = blocks_per_image / blocks_c;
    Block here = block_at(blk);
    const Block by = block_at(step);
    auto next = [&](Block b) {
        b.c += by.c;
        b.r += by.r;
        b.n += by.n;
        if (b.c >= blocks_c) b.c -= blocks_c, ++b.r;
        if (b.r >= blocks_r) b.r -= blocks_r, ++b.n;
        return b;
    };
    auto issue_copies = [&](Block b, int stage, char* buf) {  // uniform
        const int ih = 8 * b.r, iw = 8 * b.c;
        const int first = ((b.n * H + ih) * W + iw) * CHUNKS + 4 * stage;  // (31 bits: checked by the launcher)
        const bool border = ih == 0 || iw == 0 || ih + 8 > H || iw + 8 > W;
#pragma unroll
        for (int k = 0; k < R::COPIES; ++k) {
            const char* src = (const char*)x + (int64_t)(first + rel[k]) * 16;
            if (border && !((unsigned)(ih + row_of[k]) < (unsigned)H && (unsigned)(iw + col_of[k]) < (unsigned)W)) src = zeros;
            if ((k + 1) * 1024 <= kPatch || k * 1024 + lane * 16 < kPatch) copy16_to_lds(src, buf + k * 1024);
        }
    };
    if (blk < end) issue_copies(here, 0, mine);
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
    scale_bias.store(lds_ep, ep, tid);
    __syncthreads();

    const int nn = lane & 15, qq = lane >> 4, pr = nn >> 2, pc = nn & 3, odd = lane & 1;
    const int xb0 = (2 * pr * 9 + pc) * 64 + (pr & 1 ? 3 - qq : qq) * 16, xb1 = (2 * pr * 9 + pc) * 64 + (pr & 1 ? qq : 3 - qq) * 16;
    epi_by_form(ep, [&](auto form) {
        int buf = 0;
        for (; blk < end; blk += step) {
            f32x4 acc[4];
            static_for<STAGES>([&](auto stage_tag) {
                constexpr int stage = decltype(stage_tag)::value;
                __builtin_amdgcn_sched_barrier(0);
                // this stage's copies have landed; behind them are at most the two stores of the block before
                if constexpr (stage == 0) asm volatile("s_waitcnt vmcnt(2)" ::: "memory");
                else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
                const char* at = mine + buf * kPatch;
                buf ^= 1;
                if constexpr (stage + 1 < STAGES) issue_copies(here, stage + 1, mine + buf * kPatch);
                else if (blk + step < end) issue_copies(next(here), 0, mine + buf * kPatch);
                __builtin_amdgcn_sched_barrier(0);
                const char* A = smem + stage * R::A_BYTES;
                auto read_tap = [&](int t) {
                    const int kh = t / 3, kw = t % 3;
                    return *(const u32x4*)(at + (kh < 2 ? xb0 : xb1) + (kh * 9 + (kw & 1 ? 5 : kw >> 1)) * 64);
                };
                // (the centre's and the first group's operands are asked for together, the second group's in front of their products: with
                // copies into LDS under way a wave waits for all of its reads, and left alone the compiler puts that wait behind every pair)
                u32x4 xs[NG][4], as[NG][4][2], ac[4];
                int idx[NG][4];
                auto fetch = [&](int g) {
#pragma unroll
                    for (int f = 0; f < 4; ++f) xs[g][f] = read_tap(LY.tap[g][f]);
#pragma unroll
                    for (int m = 0; m < 4; ++m) {
                        const char* frag = A + m * TILE;
                        idx[g][m] = *(const int*)(frag + FR * kFragBytes + (g * 64 + lane) * 4);
                        as[g][m][0] = *(const u32x4*)(frag + 2 * g * kFragBytes + lane * 16);
                        as[g][m][1] = *(const u32x4*)(frag + (2 * g + 1) * kFragBytes + lane * 16);
                    }
                };
                const u32x4 centre = read_tap(4);
#pragma unroll
                for (int m = 0; m < 4; ++m) ac[m] = *(const u32x4*)(A + m * TILE + 2 * NG * kFragBytes + lane * 16);
                fetch(0);
                __builtin_amdgcn_sched_barrier(0);
                __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
                fetch(1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int m = 0; m < 4; ++m) acc[m] = Dense16<T>::mma(ac[m], centre, stage == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[m]);
#pragma unroll
                for (int g = 0; g < NG; ++g) {
                    const u32x8 b[2] = {sparse_operand(xs[g], 0), sparse_operand(xs[g], 1)};
#pragma unroll
                    for (int m = 0; m < 4; ++m) acc[m] = Sparse64<T>::template mma<0>(as[g][m][0], b[0], acc[m], idx[g][m]);
#pragma unroll
                    for (int m = 0; m < 4; ++m) acc[m] = Sparse64<T>::template mma<1>(as[g][m][1], b[1], acc[m], idx[g][m]);
                }
            });
            // ---- 16 consecutive channels of one position a lane; rows of 128 bytes past the L2's write-back ----
            const int oh0 = 4 * here.r, ow0 = 4 * here.c;
            const int64_t pos0 = ((int64_t)here.n * Ho + oh0) * Wo + ow0;
            here = next(here);
            const bool row_inside = oh0 + pr < Ho && 64 * cb + 16 * qq < Co;  // (Co is a multiple of 16)
            float v[16];
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int e = 0; e < 4; ++e) v[4 * m + e] = acc[m][e];
            epi_scale_bias_act_of<decltype(form)::value, 16>(v, ep, lds_ep + 16 * qq, lds_ep + 64 + 16 * qq);
            if (row_inside && ow0 + pc < Wo) epi_residual<T, 16>(v, ep, pos0 + pr * Wo + pc, 64 * cb + 16 * qq);
            u32x4 o[2] = {pack8_from_f32<T>(v), pack8_from_f32<T>(v + 8)};
            pair_pieces(o[0], o[1], odd);
            const auto base = store_base(y + pos0 * ep.ldy + 64 * cb);
            const uint32_t to = (uint32_t)((pr * Wo + pc - odd) * ep.ldy + 16 * qq + 8 * odd) * 2;  // (within 32 bits: resident_ok)
            uint32_t to0 = row_inside && ow0 + pc - odd < Wo ? to : kNoStore, to1 = row_inside && ow0 + pc - odd + 1 < Wo ? to + 2 * ep.ldy : kNoStore;
            asm("" : "+v"(to0), "+v"(to1));  // (always two stores, for the count above: not a branch around each)
            __builtin_amdgcn_sched_barrier(0);
            store16_through(base, to0, o[0]);
            store16_through(base, to1, o[1]);
            __builtin_amdgcn_sched_barrier(0);
        }
    });
}

template <typename T, int STAGES>
rtoss_status launch_resident(const rtoss_wdesc& d, const ConvParams& c, const char* wfrag, const void* x, void* y, hipStream_t s)
{
    using R = Resident<STAGES>;
    const int Ho = (c.H - 1) / 2 + 1, Wo = (c.W - 1) / 2 + 1, blocks_c = (Wo + 3) / 4, blocks_per_image = (Ho + 3) / 4 * blocks_c;
    const int co_blocks = (d.Co + 63) / 64, blocks = blocks_per_image * c.N;
    auto kern = conv3x3_resident_kernel<T, STAGES>;
    static LaunchOnce lds_once;  // per instantiation
    if (rtoss_status st = ensure_dynamic_lds((const void*)kern, R::LDS, lds_once, c.dev.device, "conv3x3 shared memory attribute")) return st;
    const int slots = std::max(1, c.dev.cus / 8 / co_blocks) * co_blocks;  // workgroups of an XCD: one per compute unit
    kern<<<dim3(8 * slots), dim3(64 * R::WAVES), R::LDS, s>>>((const T*)x, (T*)y, wfrag, wfrag + fragment_bytes(d, 0), c.H, c.W, d.Co, Ho, Wo,
                                                                   padded_m_tiles(d.Co), blocks_c, blocks_per_image, co_blocks, blocks,
                                                                   (blocks + 7) / 8, c.ep);
    return check_hip(hipGetLastError(), "conv3x3 resident launch");
}

template <typename T, typename TO, int S, int TM, int TN, int RT, int CT, bool AHEAD = true, int LAY = 0, bool DB = false, bool RAG = false>
rtoss_status launch_variant_sb(const rtoss_wdesc& d, const ConvParams& c, const char* wfrag, const void* x, void* y,
                            hipStream_t s)
{
    using G = Geom<S, RT, CT>;
    const int Ho = (c.H + 2 - 3) / S + 1, Wo = (c.W + 2 - 3) / S + 1;
    constexpr int th = S == 2 ? 4 : G::TH, tw = S == 2 ? 4 : G::TW;  // (stride 2: blocks)
    const int tiles_r = (Ho + th - 1) / th, tiles_c = (Wo + tw - 1) / tw;
    const int64_t blocks = (int64_t)tiles_r * tiles_c * c.N;
    const int m_tiles_total = padded_m_tiles(d.Co);  // pitch of the packed section
    const int co_blocks = ((d.Co + 15) / 16 + TM - 1) / TM;
    constexpr size_t x_area = S == 2 ? patch_copies(TN) * 4096 : ((G::x_bytes / 16 + 63) / 64 + 3) / 4 * 4096;
    const size_t smem = (DB ? 2 : 1) * ((size_t)TM * layout_tile_bytes(kLayouts[LAY]) + x_area) + EpiScaleBias<16 * TM>::kBytes;
    auto kern = conv3x3_sparse_sb_kernel<T, TO, S, TM, TN, RT, CT, AHEAD, LAY, DB, RAG>;
    static LaunchOnce lds_once;  // per instantiation
    if (rtoss_status st = ensure_dynamic_lds((const void*)kern, smem, lds_once, c.dev.device, "conv3x3 shared memory attribute")) return st;
    const int64_t total = (S == 2 ? (blocks + 4 * TN - 1) / (4 * TN) : blocks) * co_blocks;
    if (total > 0x3fffffff || blocks > 0x7fffff00) return fail(RTOSS_ESHAPE, "conv: too many tiles");
    if ((int64_t)c.N * c.H * c.W * d.Ci / 8 > 0x7fffffff) return fail(RTOSS_ESHAPE, "conv: input too large for 32-bit chunk offsets");
    const WorkOrder order(total, co_blocks, tiles_r * tiles_c, tiles_c);
    dim3 grid(order.grid()), block(256);
    kern<<<grid, block, smem, s>>>((const T*)x, (TO*)y, wfrag, wfrag + fragment_bytes(d, LAY), c.H, c.W, d.Ci, d.Co, Ho, Wo,
                                   m_tiles_total, order, (int)blocks, c.ep);
    return check_hip(hipGetLastError(), "conv3x3 sparse launch");
}

inline bool ragged(const rtoss_wdesc& d) { return d.Ci % 32 != 0 || d.Co % 16 != 0; }

// Ragged channel counts: one variant per stride and layout, small tiles and few registers (such layers are narrow).
template <typename T, typename TO, int LAY>
rtoss_status launch_typed_ragged(const rtoss_wdesc& d, const ConvParams& c, const char* wfrag, const void* x, void* y, hipStream_t s)
{
    if (c.stride == 1) return launch_variant_sb<T, TO, 1, 4, 2, 2, 4, false, LAY, false, true>(d, c, wfrag, x, y, s);
    return launch_variant_sb<T, TO, 2, 4, 1, 1, 4, false, LAY, false, true>(d, c, wfrag, x, y, s);
}

// Large stride-1 layers (more than 64 channels in and out, enough 16x16 x 128-channel tiles to give most
// compute units one) take the pipelined kernel of conv3x3_rows.hip, whatever the layout.  (us, the kernels for smaller launches and the
// pipelined one, bf16, 3 entries / 4: 2x128@100x168, 154 tiles 10.3 12.1 / 11.8 13.9, 1x256@100x168, 154 tiles 15.4 18.8 / 18.2 21.3, 4x256@80x80,
// 200 tiles 22.3 19.5 / 27.0 23.2, 2x256@100x168, 308 tiles 38.1 24.1 / 32.6 28.5.)
// What the strips with helper waves hold in one round is theirs, whatever its tiles (conv3x3_ring.hip; us, pipelined and there: 16x512@20x20 33.6
// 25.8 / 39.9 31.9, 25x256@20x20 18.3 14.2 / 20.9 16.9, 64x128@20x32 12.7 10.4 / 15.4 12.1, with half a block of 128 channels empty
// 4x192@80x80 15.6 13.0 / 17.2 14.4, 25x256->320@20x20 21.0 14.4 / 24.2 17.0): it spreads over the units in strips of 64 channels.
inline bool takes_pipelined_kernel(const rtoss_wdesc& d, const ConvParams& c)
{
    if (c.stride != 1 || d.Co <= 64 || d.Ci <= 64 || ragged(d)) return false;
    if (!rows3x3_needs_fused_stage(c) && c.out_dt != RTOSS_F32 && !stores_in_reach(c)) return false;
    const int64_t tiles8 = (int64_t)((c.H + 15) / 16) * ((c.W + 15) / 16) * c.N * (((d.Co + 15) / 16 + 7) / 8);
    return tiles8 >= 200;
}

// Layout 1: where the strips without helpers would not be faster, because they waste less of small or oddly sized images and of half-empty
// channel blocks.  us: 0.6 and 0.54 a unit of the pipelined kernel's busiest workgroup; 3 and, per stage and round of two workgroups a
// unit, 1.75, 2.3, 2.75 and 3.85 of strips of 8, 12, 16 and 20 rows (1.0 where eight rows fit once).  Measured, strips and pipelined, 4 entries:
//     200x96->112@5x3 8.2 12.0   200x128@8x16 9.9 14.0   40x96->256@24x17 18.6 21.2   4x160->144@112x162 36.3 43.1   2x128->256@33x330 13.8 15.0
//     100x256@13x13 25.0 21.6    100x128@17x17 17.9 15.9   4x96@100x168 16.1 14.6    2x256@100x168 33.8 28.2       3x320@80x80 31.7 28.3
// (Tensors in caches.  In none, with half sectors a position and three or four stages, the pipelined kernel's rows past the write-back cost up to 5 %
// more than the strips: 96->240@1x200x168 19.2 20.2, in caches 17.3 15.3; 128->176@4x100x168 32.2 33.3, 30.4 29.6.)
inline double strips_us(const rtoss_wdesc& d, const ConvParams& c, int plan)
{
    const int rows = strip3x3_rows(plan);
    const int64_t groups = (int64_t)((c.W + 15) / 16) * ((c.H + rows - 1) / rows) * ((d.Co + 63) / 64) * c.N, cus = c.dev.cus;
    const double stage = rows == 8 ? (groups <= cus ? 1.0 : 1.75) : rows == 12 ? 2.3 : rows == 16 ? 2.75 : 3.85;
    return 3 + d.Ci / 32 * stage * (double)((groups + 2 * cus - 1) / (2 * cus));
}
inline double pipelined_us(const RowsLaunch& rows) { return 0.6 + 0.54 * rows.cost; }

// Stride 2, one or two blocks per wave: three workgroups per compute unit with one, two with two, whose rounds take about 4/3 as
// long (two halve the weights a block reads from LDS).  Two where that is the smaller sum; not for one or two stages, which
// the memory bounds (us, one and two, plain, in a loop over the same tensors; layout 0 / 1, batch x channels in -> out @ image):
//     16x256->256@40  12.7 16.4 / 15.4 19.2  one    16x256->512@40 25.6 20.8 / 31.3 24.5  two     4x64->128@112x140  6.1 8.0 / 6.8 8.6  one
//     4x128->256@56x70 7.2  9.7 /  8.5 11.0  one    4x128->256@112x140 15.4 13.1 / 17.6 14.4  two  16x64->128@160   25.9 28.5 / 29.7 31.3  one
inline bool two_blocks_per_wave(const rtoss_wdesc& d, const ConvParams& c)
{
    const int64_t blocks = (int64_t)(((c.H - 1) / 2 + 4) / 4) * (((c.W - 1) / 2 + 4) / 4) * c.N, co_blocks = (d.Co + 63) / 64, cus = c.dev.cus;
    const int64_t one = ((blocks + 3) / 4 * co_blocks + 3 * cus - 1) / (3 * cus), two = ((blocks + 7) / 8 * co_blocks + 2 * cus - 1) / (2 * cus);
    return d.Ci > 64 && 4 * two <= 3 * one;
}

// Stride 2, one or two stages: resident weights from one and a half blocks a wave on (us with SiLU, the single-buffered kernel and the
// resident one, tensors in caches, then in none; blocks of 64 channels x 16 positions a wave in brackets; batch x channels in -> out @ image):
//     16x32->64@320 (12.5)    35.9 27.1  42.9 34.7    16x64->128@160 (6.3)   28.3 22.0  34.0 27.7    16x64->256@80 (3.1)     16.1 13.2  19.1 16.8
//     16x32->32@160 (3.1)     10.8  9.4  13.6 11.8    4x64->448@90 (2.0)     10.8 10.9  13.1 12.7    4x32->64@240x250 (1.8)   7.9  6.2  10.5  8.9
//     2x64->256@160 (1.6)     10.3  8.1  12.1 10.0    4x64->128@160 (1.6)    10.4  8.1  12.8 10.6
//     2x32->128@203x211 (1.4)  6.0  6.1   7.3  7.2    3x64->128@160 (1.2)     8.2  8.0  10.1 10.3    4x64->128@112x140 (1.0)  6.2  6.1   8.7  7.6
// (the last line stays: plain layers of its first two lose 8 % in no cache.  Offsets of a block's stores within 32 bits.)
inline bool resident_ok(const rtoss_wdesc& d, const ConvParams& c)
{
    const int64_t Ho = (c.H - 1) / 2 + 1, Wo = (c.W - 1) / 2 + 1, blocks = (Ho + 3) / 4 * ((Wo + 3) / 4) * c.N, co_blocks = (d.Co + 63) / 64;
    if (d.Ci > 64 || co_blocks > 8 || 2 * (3 * Wo + 4) * c.ep.ldy >= kNoStore || blocks > 0x3fffffff || (int64_t)c.N * c.H * c.W * d.Ci / 8 > 0x7fffffff) return false;
    return blocks * co_blocks >= 12 * c.dev.cus;
}

// Layout 1 (three tap groups): the single-buffered kernel for every shape.
template <typename T, typename TO>
rtoss_status launch_typed_layout1(const rtoss_wdesc& d, const ConvParams& c, const char* wfrag, const void* x, void* y,
                                  hipStream_t s)
{
    if (ragged(d)) return launch_typed_ragged<T, TO, 1>(d, c, wfrag, x, y, s);
    if (c.stride == 1) return launch_variant_sb<T, TO, 1, 4, 2, 2, 4, false, 1>(d, c, wfrag, x, y, s);
    if (two_blocks_per_wave(d, c)) return launch_variant_sb<T, TO, 2, 4, 2, 2, 4, false, 1>(d, c, wfrag, x, y, s);
    return launch_variant_sb<T, TO, 2, 4, 1, 1, 4, false, 1>(d, c, wfrag, x, y, s);
}

template <typename T, typename TO>
rtoss_status launch_typed(const rtoss_wdesc& d, const ConvParams& c, const char* wfrag, const void* x, void* y,
                          hipStream_t s)
{
    if (ragged(d)) return launch_typed_ragged<T, TO, 0>(d, c, wfrag, x, y, s);
    // The fragment section is padded to a multiple of 8 channel tiles, so any TM <= 8 may over-read rows
    // that hold zeros; outputs beyond Co are never stored.
    // Layers with at most 64 output channels, or too few stages to amortise the pipelined kernel's
    // prologue, come here: 64 channels per workgroup.
    if (c.stride == 1) {
        // 8x16-position tiles for these: 38 KB of LDS per buffer.  (Measured: several resident workgroups beat one
        // workgroup per compute unit with larger buffers, and beat 16x16 tiles, on every such layer.)
        // (up to 64 input channels are one or two stages: nothing to gain inside a workgroup, see AHEAD; one buffer,
        // four workgroups per compute unit)
        if (d.Ci <= 64) return launch_variant_sb<T, TO, 1, 4, 2, 2, 4, false>(d, c, wfrag, x, y, s);
        // deeper layers of up to 64 output channels, in launches of several rounds (smaller ones: conv3x3_ksplit.hip,
        // conv3x3_strip.hip): two buffers per workgroup, still two workgroups per compute unit
        return launch_variant_sb<T, TO, 1, 4, 2, 2, 4, true, 0, true>(d, c, wfrag, x, y, s);
    }
    if constexpr (sizeof(TO) == 2)
        if (resident_ok(d, c)) return d.Ci == 32 ? launch_resident<T, 1>(d, c, wfrag, x, y, s) : launch_resident<T, 2>(d, c, wfrag, x, y, s);
    if (two_blocks_per_wave(d, c)) return launch_variant_sb<T, TO, 2, 4, 2, 2, 4>(d, c, wfrag, x, y, s);
    return launch_variant_sb<T, TO, 2, 4, 1, 1, 4>(d, c, wfrag, x, y, s);
}

}  // namespace

// ---- host-visible entry points of this file ----

// Dictionaries that need the repeated taps of layout 1 (5 entries): whole stages and channel tiles, at least 64 channels in and out and more in one
// of them.  Below, and for ragged counts, the dense mode's shorter chain is as fast or faster at every size (us, dense mode and 2-of-4,
// bf16: 1x32@28x36 3.1 3.6, 4x32@20x30 3.2 4.0, 1x24->80@50 3.6 5.9, 2x40->36@60 4.2 7.9, 4x64@20x30 3.8 4.0, 16x64@80 10.1 10.2), and
// only its section is packed; from there on it depends on the launch (sparse3x3_is_faster).
bool sparse3x3_shape_ok(const rtoss_wdesc& d, const Dict& dict)
{
    // (rows of 16-byte multiples: the activation copies move 8 channels per lane)
    if (d.ksize != 3 || (d.dt != RTOSS_F16 && d.dt != RTOSS_BF16) || d.Ci % 8 || dict.layout < 0) return false;
    return !dict.repeats || (!ragged(d) && d.Ci >= 64 && d.Co >= 64 && d.Ci + (int64_t)d.Co > 128);
}

constexpr int kDenseTaps = 2;  // the dense mode, as a layout of the other files' plans

// Of a dictionary that needs the repeated taps both sections are packed, for at odd sizes the dense mode has the better tiles: smaller ones in
// small launches, strips of fewer rows on low images.  Which, by the plans of both (1480 launches of 64 to 512 channels on 4 to 220 rows and
// columns, bf16 and fp16: the slower one by more than 3 % in 60 of them; always the 2-of-4 steps, up to 1.78 times as long; always dense mode, 21 %
// on average).  Packing both takes four layers 256 -> 256 6.7 -> 7.2 us, two of 512 8.0 -> 10.1.  us, dense mode and 2-of-4:
//     Channels split over the waves: 32 channels a workgroup against 16 of the dense mode's split (256@1x20x46 4.86 5.11), or against its small
//     tiles while two of them a unit hold the launch, where the split's four waves are unevenly deep (96@2x30x35 3.92 4.41, 64->80@1x56x56 3.65
//     4.32, 160@2x24x28 4.85 5.20; 160@2x30x37, 576 tiles 6.24 5.41; four stages 128@1x40x53 4.59 4.62; seven 224@1x22x49 5.92 5.62).
//     Stride 2: the small tiles while two a unit hold the launch (64->256@2x11x149 4.79 5.10, 192->384@2x32x61 7.87 9.91, 320->128@5x13x104
//     10.6 14.5; 576 tiles 128->256@2x47x65 8.5 7.6, 192->384@3x28x34 11.3 9.8).
//     Strips, eight rows once over the chip: the small tiles while three a unit hold the launch (128@3x32x48 5.53 6.47, 160@2x31x53 6.75 7.25;
//     128@1x65x96, 816 tiles 7.56 6.58), from nine stages on not.
//     Strips of more rows: the dense mode's, of 8, 12, 16 or 20 rows (weights past LDS), take 3.4 us and 0.07 a row, and per round of one a
//     unit 0.02 a row and, a stage, 0.28 and 0.064 a row; the others strips_us or 0.84 of pipelined_us, which fills its tiles better than
//     those are cut (192->160@200x7x6 16.5 29.4, 256->96@49x5x118 27.4 44.9, 96->256@40x24x17 15.9 18.4; 256@2x100x168 33.5 28.4).
// By the shape alone: results of either type, with an output stage or into a slice, add in one order.
bool sparse3x3_is_faster(const rtoss_wdesc& d, const Dict& dict, const ConvParams& call)
{
    if (!sparse3x3_launch_ok(d, dict, call)) return false;
    ConvParams c = call;
    c.out_dt = d.dt;
    c.ep = Epilogue{nullptr, nullptr, nullptr, 0, d.Co, d.Co};
    const int64_t cus = c.dev.cus;
    const int stages = d.Ci / 32, Ho = (c.H - 1) / c.stride + 1, Wo = (c.W - 1) / c.stride + 1;
    const auto groups = [&](int rows, int cols, int channels) {
        return (int64_t)((Ho + rows - 1) / rows) * ((Wo + cols - 1) / cols) * ((d.Co + channels - 1) / channels) * c.N;
    };
    const int64_t small = 4 * groups(4, 16, 64);   // the dense mode's small tiles, of 16 channels in blocks of 64, ...
    const bool tall = groups(16, 16, 64) >= 256;   // ... which larger launches do not take (conv3x3_dense.hip)
    const int split = ksplit3x3_plan(d, c, 1), dense_split = ksplit3x3_plan(d, c, kDenseTaps);
    if (c.stride == 2) return split || dense_split || tall || small > 2 * cus;
    if (split) return groups(4, 8, 16) <= cus || !(dense_split || (stages <= 5 && stages != 4 && small <= 2 * cus));
    const int dense = strip3x3_plan(d, c, kDenseTaps), plan = strip3x3_plan(d, c, 1);
    if (!dense) return tall || stages > 8 || small > 3 * cus;
    if (stages == 2 || !plan || ring3x3_plan(d, c, 1)) return true;
    const int rows = strip3x3_rows(dense);
    const double rounds = (double)((groups(rows, 16, 64) + cus - 1) / cus);
    const double dense_us = 3.4 + 0.07 * rows + rounds * ((0.28 + 0.064 * rows) * stages + 0.02 * rows);
    double us = strips_us(d, c, plan);
    if (takes_pipelined_kernel(d, c)) us = std::min(us, 0.84 * pipelined_us(plan_rows_for_device(c.N, c.H, c.W, d.Co, stages, c.dev.cus)));
    return us <= dense_us;
}

bool sparse3x3_launch_ok(const rtoss_wdesc& d, const Dict& dict, const ConvParams& c)
{
    if (!ragged(d) && !dict.repeats) return true;
    // the smallest tiles (launch_typed_ragged's; stride 2: four blocks, at least as many positions as a tile of 4x16)
    const int Ho = (c.H - 1) / c.stride + 1, Wo = (c.W - 1) / c.stride + 1, rows = c.stride == 1 ? 8 : 4;
    return (int64_t)c.N * c.H * c.W * d.Ci / 8 <= kMaxChunks &&
           (int64_t)((Ho + rows - 1) / rows) * ((Wo + 15) / 16) * ((d.Co + 63) / 64) * c.N <= kMaxGridGroups;
}

size_t sparse3x3_section_bytes(const rtoss_wdesc& d, int layout)
{
    return fragment_bytes(d, layout) + zero_block_bytes(d);
}

rtoss_status launch_conv3x3_sparse(const rtoss_wdesc& d, const ConvParams& c, int layout, const void* section, const void* x,
                                   void* y, hipStream_t s)
{
    const char* wf = (const char*)section;
    const bool f32out = c.out_dt == RTOSS_F32;
    if (const int plan = ksplit3x3_plan(d, c, layout))
        return launch_conv3x3_ksplit(d, c, layout, plan, section, wf + fragment_bytes(d, layout), x, y, s);
    if (const int plan = ring3x3_plan(d, c, layout))
        return launch_conv3x3_ring(d, c, layout, plan, section, wf + fragment_bytes(d, layout), x, y, s);
    bool pipelined = takes_pipelined_kernel(d, c);
    RowsLaunch rows;
    const RowsLaunch* planned = nullptr;
    if (!pipelined || layout == 1) {
        const int plan = strip3x3_plan(d, c, layout);
        if (pipelined && plan) {  // (a launch within the limits of strips)
            rows = plan_rows_for_device(c.N, c.H, c.W, d.Co, d.Ci / 32, c.dev.cus);
            planned = &rows;
            pipelined = strips_us(d, c, plan) >= pipelined_us(rows);
        }
        if (plan && !pipelined) return launch_conv3x3_strip(d, c, layout, plan, section, wf + fragment_bytes(d, layout), x, y, s);
    }
    if (layout != 0 && layout != 1) return fail(RTOSS_EINVAL, "conv: unknown tap layout %d", layout);
    if (pipelined) return launch_conv3x3_rows(d, c, layout, planned, section, x, y, s);
    if (layout == 1) {
        if (d.dt == RTOSS_F16)
            return f32out ? launch_typed_layout1<f16_t, float>(d, c, wf, x, y, s) : launch_typed_layout1<f16_t, f16_t>(d, c, wf, x, y, s);
        return f32out ? launch_typed_layout1<bf16_t, float>(d, c, wf, x, y, s) : launch_typed_layout1<bf16_t, bf16_t>(d, c, wf, x, y, s);
    }
    if (d.dt == RTOSS_F16)
        return f32out ? launch_typed<f16_t, float>(d, c, wf, x, y, s) : launch_typed<f16_t, f16_t>(d, c, wf, x, y, s);
    return f32out ? launch_typed<bf16_t, float>(d, c, wf, x, y, s) : launch_typed<bf16_t, bf16_t>(d, c, wf, x, y, s);
}

}  // namespace rtoss
