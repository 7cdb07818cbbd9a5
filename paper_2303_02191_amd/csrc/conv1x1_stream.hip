// 1x1 pattern-pruned convolution as a streaming kernel with register-resident weights
// (fp16 / bf16 / fp32, fp32 accumulate).
//
// Section IV.D prunes a 1x1 layer by cutting the flattened [Co][Ci] weight matrix into groups
// of 9 and keeping k weights per group; the pruned layer is the GEMM
//     Y[p][co] = sum_ci W'[co][ci] * X[p][ci]          (p runs over all N*H*W positions).
// The k-of-9 sparsity has no shape a matrix instruction could skip, and the layer moves every
// activation byte once for at most Ci*k/9 multiply-adds per output: it is bound by HBM, not by
// arithmetic.  So the weights are expanded to zero-filled dense fragments and the kernel is
// organised around the activation stream:
//   * Workgroups are persistent.  Each owns one block of output channels and a share of the buffers
//     of positions (share.h), and every wave loads its share of the weight fragments into registers once
//     (at most 32 fragments = 128 registers), so the K loop reads weights from nowhere.
//   * Activations arrive through a ring of 3 LDS buffers filled by global -> LDS copies.  A
//     buffer holds PB positions (16 per wave along positions) x all Ci channels, laid out
//     [32-channel stage][position][64 bytes] with the four 16-byte chunks of a position
//     XOR-swizzled by (position / 2) % 4: conflict-free 16-byte operand reads without padding.
//   * One or two helper waves move everything: they issue the copies (but for the first two buffers of a
//     workgroup, which the consumers fetch while they would otherwise idle) and store the outputs.  Both are
//     counted by the same counter in the order they were issued, and a turn issues a fixed number of each (lanes
//     with nothing to store write past the end of a bounded buffer), so "buffer b has landed" is an exact counted wait.
//     One barrier per buffer hands a filled buffer to the consumers, a drained one back, and an output tile over.
//   * The packer assigns output channels to matrix rows so that a lane's 4*MT accumulator values are
//     consecutive channels: row 4q+i of the wave's m-th fragment is channel 4*MT*q + 4*m + i of the wave's slice.  The
//     consumers put them into a tile in LDS, from which the helpers store whole rows, past the L2's
//     write-back: outputs of a few MB fit the L2s, and a launch that leaves them there ends with writing all of
//     them back (copies of 13 MB: 6.1 us, past it 5.4).  In pieces of 16 bytes that would cost more than it saves.
//     us with stores from the accumulators / with tiles / with tiles past the write-back: 64 -> 64 channels on 102 400
//     positions with SiLU 8.0  8.2  6.6, 128 -> 128 on 102 400 12.3  12.6  11.1, 256 -> 256 on 25 600 11.0  11.0  9.6.
//     Outputs of up to 2 MB, which are written back in no time, stay with the first way (direct_outputs).
//   * 512 channels: two or three buffers a workgroup and a wave to a SIMD, so that a turn is the sum of its parts.  The consumers
//     put the output stage of a buffer between the matrix instructions of the next one instead, and store from there (16-bit results
//     in rows of 64 bytes; a tile would be a turn more): 512 -> 256 on 6400 positions with SiLU 7.0 -> 6.2 us, 512 -> 512 9.4 -> 7.9.
//
// fp32 tensors of 32 to 256 channels have a kernel of their own, on the bf16 matrix instruction (the second one here).  Those of
// 16 and of 512 channels run through the first: a stage is then 16 channels (the same 64 bytes per position) and a fragment
// step is four v_mfma_f32_16x16x4_f32, instruction s on element s of every lane's 16 bytes.  (16 channels would fill half a
// step of the other instruction: 12 800 positions 3.0 us here, 3.3 there.  512 channels in three parts are more registers
// than a wave has room for beside what it prefetches: 512 -> 256 on 6400 positions 19.9 us here, 21.7 there.)
//
// Operand layout of v_mfma_f32_16x16x32 (wave64; r = lane % 16, q = lane / 16): A lane holds
// row r, K = 8q..8q+7; B lane holds column r, K = 8q..8q+7; D lane holds column r, rows 4q..4q+3.
#include <algorithm>

#include "common.h"
#include "dtypes.h"
#include "epilogue.h"
#include "fp32_split.h"
#include "mma.h"
#include "work_order.h"
#include "pack_plan.h"
#include "share.h"

namespace rtoss {

namespace {

constexpr int kFrag = 1024;  // one A fragment: 64 lanes x 16 bytes = 16 output channels x 32 input channels
constexpr int kHeadBuffers = 2;  // buffers of a workgroup's range that the consumer waves copy themselves

// Copies and stores cost a wave about 70 cycles each, a turn of the consumers 1000 to 2000: two helpers where one would be the slower side
// (1024 -> 512 on 6400 positions 18.2 and 14.3 us, 256 -> 256 on 51 200 11.4 and 10.8), and at 16 copies a turn, whose
// addresses would cost a workgroup per compute unit (128 -> 64 on 102 400: 9.0 and 8.5).
constexpr int helper_waves(int KS, int WM) { return KS >= 8 || 4 / WM * KS >= 16 ? 2 : 1; }

// Shape plan, a function of KS = Ci / 32 (fp32: Ci / 16; 1, 2, 4 ... 32) and of WM, the number of waves a
// workgroup spreads over output channels (the other 4 / WM spread over positions).
template <int KS, int WM> struct Plan {
    static constexpr int MT = stream_mt_of(KS);  // fragments per wave along output channels
    static constexpr int WN = 4 / WM;
    // 16-position blocks per wave and buffer: one.  (Buffers of up to four blocks per wave, 16 KB for most shapes,
    // measured slower on a 57-layer model, 0.906 against 0.892-0.895 ms: small buffers mean small workgroups in LDS,
    // more of them per compute unit and more independent streams in flight.)
    static constexpr int NB = 1;
    static constexpr int PB = 16 * NB * WN;                        // positions per buffer
    static constexpr int BUF = PB * KS * 64;                       // bytes per buffer
    static constexpr int COPIES = PB * KS / 16;                    // copy instructions (64 lanes x 16 B) per buffer
    static constexpr int SPAN = 16 * MT * WM;                      // output channels per workgroup
    // Ring depth: three buffers (one being multiplied, one landing, one being refilled).  The 6-bit counter of
    // outstanding copies would allow up to six for most shapes; measured on a 57-layer model, the shallow ring is
    // faster (0.900 vs 0.907 ms with four and 0.915 ms with up to six buffers): its 48 KB let three workgroups share a
    // compute unit, and their helpers together keep more copies in flight than one deep ring can count.
    static constexpr int RING = 3;
    static constexpr bool INTERLEAVED = KS == 16;                  // a buffer's output stage between the products of the next
    static constexpr int HELPERS = helper_waves(KS, WM);
    static constexpr int LANES = 64 * (4 + HELPERS);
    static_assert(COPIES >= 1 && COPIES * 16 == PB * KS, "a buffer is a whole number of copy instructions");
    static_assert(RING == 3, "the waits below count two turns");
};

// s_waitcnt immediate that waits for the vector-memory counter only (6 bits, split 4 + 2)
__device__ __host__ constexpr int vmcnt_imm(int n) { return 0x0f70 | (n & 15) | ((n >> 4) << 14); }

inline size_t frag_bytes(const rtoss_wdesc& d)
{
    const int KS = stage_count(d);
    return (size_t)stream_co_blocks_of(KS, d.Co) * stream_wm_of(KS, d.Co) * stream_mt_of(KS) * KS * kFrag;
}

// TILE: outputs through LDS tiles and the helpers; else straight from the accumulators, as they are.
template <typename T, typename TO, int KS, int WM, bool TILE>
__device__ __forceinline__ void stream_outputs(const T* __restrict__ x, TO* __restrict__ y, const char* __restrict__ wfrag, const char* __restrict__ zeros,
                                               int64_t P, int Co, Divisor co_blocks, const Share& share, int total_wgs, int work_per_xcd, const Epilogue& ep)
{
    using PL = Plan<KS, WM>;
    constexpr int MT = PL::MT, NB = PL::NB, PB = PL::PB, BUF = PL::BUF, COPIES = PL::COPIES, RING = PL::RING;
    constexpr int ROW = 64 * KS;  // bytes of one position
    extern __shared__ __attribute__((aligned(16))) char smem[];  // RING buffers, scale and bias of SPAN channels, two output tiles

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // XCD-contiguous order: the channel blocks of one share's positions meet in an L2
    const int work = (blockIdx.x % 8) * work_per_xcd + blockIdx.x / 8;
    if (work >= total_wgs) return;
    const int part = co_blocks.quotient(work), cb = co_blocks.remainder(work, part);
    const Buffers buffers = share.of(part);
    const int64_t count = buffers.count;  // (64 bits: 32 measured 1 to 2 % slower in small launches)

    constexpr int EB = (int)sizeof(TO), SPAN = PL::SPAN;
    constexpr int CPR = SPAN * EB / 16;                        // 16-byte chunks of a row of the output tile
    constexpr int OUT = PB * SPAN * EB, STORES = OUT / 1024;   // bytes and store instructions of a tile
    char* out = smem + RING * BUF + EpiScaleBias<SPAN>::kBytes;  // two output tiles
    // (chunks permuted by row, for writes and reads without bank conflicts)
    const auto chunk_at = [](int row, int c) { return row * CPR + (CPR >= 16 ? c ^ (row & 15) : c ^ ((row >> 1) & 7)); };
    static_assert(CPR >= 8 && STORES >= 1 && STORES * 1024 == OUT, "whole store instructions");
    // stores the tile of buffer b, one in `step` of its store instructions
    auto flush = [&](int64_t b, int first, auto step) {
        const char* tile = out + (b & 1) * OUT;
        const int64_t p0 = buffers.at(b) * PB;
        const auto base = store_base(y + p0 * ep.ldy + cb * SPAN);
        const int rows = (int)std::min<int64_t>(P - p0, PB), cols = Co - cb * SPAN;
        constexpr int STEP = decltype(step)::value, N = (STORES + STEP - 1) / STEP, AT_ONCE = N < 4 ? N : 4;
#pragma unroll
        for (int i0 = 0; i0 < N; i0 += AT_ONCE) {
            u32x4 v[AT_ONCE];
            uint32_t at[AT_ONCE];
#pragma unroll
            for (int i = 0; i < AT_ONCE; ++i) {
                const int store = first + (i0 + i) * STEP, k = store * 64 + lane, r = k / CPR, c = k % CPR;
                const bool whole = STORES % STEP == 0 || store < STORES;
                v[i] = *(const u32x4*)(tile + (whole ? chunk_at(r, c) * 16 : 0));
                at[i] = whole && r < rows && c * (16 / EB) < cols ? (uint32_t)r * ep.ldy * EB + c * 16 : kNoStore;
            }
#pragma unroll
            for (int i = 0; i < AT_ONCE; ++i) store16_through(base, at[i], v[i]);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    if (wave >= 4) {
        constexpr int H = PL::HELPERS, MINE = COPIES / H, FLUSH = STORES / H;
        static_assert(COPIES % H == 0 && STORES % H == 0, "helpers share the work");
        const int helper = wave - 4;
        // ---- helper waves: every H-th copy and store of the workgroup ----
        int src_off[MINE];  // byte offset from the buffer's first position of the chunk this lane fills
#pragma unroll
        for (int k = 0; k < MINE; ++k) {
            const int c = (k * H + helper) * 64 + lane;
            const int s = c / (PB * 4), rem = c % (PB * 4);
            const int pos = rem >> 2, q = (rem & 3) ^ ((pos >> 1) & 3);
            src_off[k] = pos * ROW + s * 64 + q * 16;
        }
        auto issue_buffer = [&](int64_t b, int slot) {  // (b: of this workgroup's)
            const int64_t p0 = buffers.at(b) * PB;
            const char* base = (const char*)x + p0 * ROW;
            char* dst = smem + slot * BUF + helper * 1024;
            if (p0 + PB <= P) {
#pragma unroll
                for (int k = 0; k < MINE; ++k) copy16_to_lds(base + src_off[k], dst + k * H * 1024);
            } else {  // ragged last buffer: positions past the end read the packer's block of zeros
                const int left = (int)(P - p0) * ROW;
#pragma unroll
                for (int k = 0; k < MINE; ++k) copy16_to_lds(src_off[k] < left ? base + src_off[k] : zeros, dst + k * H * 1024);
            }
        };
        // (the first kHeadBuffers buffers are copied by the consumer waves, see below)
        static_assert(kHeadBuffers == RING - 1, "the helpers' first copies are of the first turn");
        int slot = 0;
        for (int64_t b = 0; b < count; ++b) {
            asm volatile("" ::: "memory");
            if (!TILE && b >= kHeadBuffers) {
                if (b + 1 < count) __builtin_amdgcn_s_waitcnt(vmcnt_imm(MINE));
                else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
            } else if (b >= kHeadBuffers) {
                // buffer b has landed once no more is outstanding than was issued after its copies, two turns ago: the stores of
                // two turns (the first turn has none) and the copies of one (none at last)
                const bool first = b < 3, last = b + 1 == count;
                if (!first && !last) __builtin_amdgcn_s_waitcnt(vmcnt_imm(std::min(63, 2 * FLUSH + MINE)));
                else if (!first) __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * FLUSH));
                else if (!last) __builtin_amdgcn_s_waitcnt(vmcnt_imm(std::min(63, FLUSH + MINE)));
                else __builtin_amdgcn_s_waitcnt(vmcnt_imm(FLUSH));
            }
            __builtin_amdgcn_s_barrier();  // consumers may read buffer b; they are done with the slot refilled next
            asm volatile("" ::: "memory");
            if (b + RING - 1 < count) issue_buffer(b + RING - 1, (slot + RING - 1) % RING);
            if (TILE && b) flush(b - 1, helper, std::integral_constant<int, H>{});
            slot = slot + 1 == RING ? 0 : slot + 1;
        }
        if constexpr (TILE) {
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();  // the last output tile is complete (the consumers store it)
        }
        return;
    }

    // ---- consumer waves ----
    const int wm = wave % WM, wn = wave / WM;
    float* lds_ep = (float*)(smem + RING * BUF);
    EpiScaleBias<PL::SPAN> scale_bias;
    scale_bias.load(ep, cb * PL::SPAN, Co, tid);
    // this wave's weight fragments, resident for the whole kernel
    u32x4 a[MT][KS];
    {
        const char* af = wfrag + ((int64_t)(cb * WM + wm) * MT * KS) * kFrag + lane * 16;
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int s = 0; s < KS; ++s) a[m][s] = *(const u32x4*)(af + (m * KS + s) * kFrag);
    }
    // Start-up: one wave needs about 70 cycles per copy instruction, so helpers that fill the ring alone
    // deliver the first buffer late.  The four consumer waves, idle until then, issue the copies of the
    // first kHeadBuffers buffers (every fourth copy instruction each), and wait for them together with
    // their weight fragments before the first barrier.
    for (int i = 0; i < kHeadBuffers; ++i) {
        const int64_t b = i;
        if (b >= count) break;
        const int64_t p0 = buffers.at(b) * PB;
        const char* base = (const char*)x + p0 * ROW;
        char* dst = smem + i * BUF;
#pragma unroll
        for (int t = 0; t < (COPIES + 3) / 4; ++t) {
            const int k = wave + 4 * t;  // wave-uniform
            if (k >= COPIES) break;
            const int c = k * 64 + lane;
            const int st = c / (PB * 4), rem = c % (PB * 4);
            const int pos = rem >> 2, q = (rem & 3) ^ ((pos >> 1) & 3);
            copy16_to_lds(p0 + pos < P ? base + pos * ROW + st * 64 + q * 16 : zeros, dst + k * 1024);
        }
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    asm volatile("" ::: "memory");
    scale_bias.store(lds_ep, ep, tid);

    const int nn = lane & 15, qq = lane >> 4;
    // operand read offset within a buffer for stage 0, block 0 (the swizzle depends on nn only)
    const int x_lane = (wn * 16 + nn) * 64 + ((qq ^ ((nn >> 1) & 3)) * 16);
    const int co_lane = cb * PL::SPAN + wm * (16 * MT) + 4 * MT * qq;  // first of this lane's 4*MT channels
    const int co_local = wm * (16 * MT) + 4 * MT * qq;

    if constexpr (PL::INTERLEAVED) {
        // ---- each buffer's output stage between the matrix instructions of the next ----
        constexpr int RUN = 4 * MT;
        const int row = 16 * wn + nn;
        int slot = 0;
        auto next_buffer = [&] {
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): this wave's reads of the previous buffer are complete
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        };
        auto multiply = [&](f32x4 (&acc)[MT]) {
            const char* X = smem + slot * BUF + x_lane;
#pragma unroll
            for (int m = 0; m < MT; ++m) acc[m] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const u32x4 bv = *(const u32x4*)(X + s * PB * 64);
#pragma unroll
                for (int m = 0; m < MT; ++m) acc[m] = Dense16<T>::mma(a[m][s], bv, acc[m]);
            }
            slot = slot + 1 == RING ? 0 : slot + 1;
        };
        auto values = [&](float (&u)[RUN], const f32x4 (&acc)[MT]) {
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int e = 0; e < 4; ++e) u[4 * m + e] = acc[m][e];
        };
        auto finish = [&](float (&v)[RUN], int64_t b) {
            const int64_t p = buffers.at(b) * PB + row;
            const bool live = p < P && co_lane < Co;  // Co is a multiple of 16 and the run is 16-aligned: all in or all out
            if (ep.residual && live) epi_residual<TO, RUN>(v, ep, p, co_lane);
            if constexpr (EB == 4) {
                // (fp32 results: an instruction writes 16 bytes of every 32, half sectors.  Past the write-back on tensors in no cache
                // 512 -> 512 on 6400 positions 13.3 us, now 9.9; 512 -> 272 on 25 600 25.6, 17.7)
                TO* const yp = y + p * ep.ldy + co_lane;
#pragma unroll
                for (int g = 0; g < RUN / 4; ++g)
                    if (live) *(f32x4*)(yp + 4 * g) = f32x4{v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
                return;
            } else {
                const auto base = store_base(y + buffers.at(b) * PB * ep.ldy);
                const uint32_t at = live ? ((uint32_t)row * ep.ldy + co_lane) * EB : kNoStore;
#pragma unroll
                for (int g = 0; g < RUN / 8; ++g) {
                    store16_through(base, at + 16 * g, pack8_from_f32<TO>(v + 8 * g));
                }
            }
        };
        epi_by_form(ep, [&](auto form) {
            constexpr int FORM = decltype(form)::value;
            f32x4 held[MT];
            next_buffer();
            multiply(held);
            for (int64_t b = 1; b < count; ++b) {
                next_buffer();
                float v[RUN];
                f32x4 acc[MT];
                if constexpr (FORM == kEpiSilu) {
                    const char* X = smem + slot * BUF + x_lane;
                    u32x4 bv[KS];
#pragma unroll
                    for (int s = 0; s < KS; ++s) bv[s] = *(const u32x4*)(X + s * PB * 64);
                    float u[RUN], e[RUN], top = 0.f;
                    values(u, held);
                    epi_scale_bias_of<FORM, RUN>(u, ep, lds_ep + co_local, lds_ep + SPAN + co_local);
                    __builtin_amdgcn_sched_barrier(0);
                    static_for<MT * KS>([&](auto step) {
                        constexpr int i = decltype(step)::value, SLOTS = RUN + 2;
                        constexpr int s = i / MT, m = i % MT;
                        acc[m] = Dense16<T>::mma(a[m][s], bv[s], s == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[m]);
                        static_for<(i + 1) * SLOTS / (MT * KS) - i * SLOTS / (MT * KS)>([&](auto part) {
                            epi_silu_part<i * SLOTS / (MT * KS) + decltype(part)::value, RUN>(u, v, e, top);
                        });
                        __builtin_amdgcn_sched_barrier(0);
                    });
                    slot = slot + 1 == RING ? 0 : slot + 1;
                    epi_silu_end<RUN>(u, v, top);
                } else {
                    values(v, held);
                    epi_scale_bias_of<FORM, RUN>(v, ep, lds_ep + co_local, lds_ep + SPAN + co_local);
                    multiply(acc);
                    if constexpr (FORM == kEpiAny) epi_act<RUN>(v, ep.act);
                }
                finish(v, b - 1);
#pragma unroll
                for (int m = 0; m < MT; ++m) held[m] = acc[m];
            }
            float v[RUN];
            values(v, held);
            epi_scale_bias_act_of<FORM, RUN>(v, ep, lds_ep + co_local, lds_ep + SPAN + co_local);
            finish(v, count - 1);
        });
        return;
    }
    static_assert(NB == 1, "one block per wave and buffer");
    epi_by_form(ep, [&](auto form) {
        int slot = 0;
        for (int64_t b = 0; b < count; ++b) {
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): this wave's reads of the previous buffer are complete
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");

            const char* X = smem + slot * BUF + x_lane;
            f32x4 acc[MT][NB];
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int j = 0; j < NB; ++j) acc[m][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            // (deep layers: eight reads in flight, where the scheduler would have two.  1024 -> 512 on 6400 positions 14.4 -> 11.9 us;
            // shallower ones have other workgroups to fill in)
            constexpr int AHEAD = KS < 8 ? KS : 8;
#pragma unroll
            for (int s0 = 0; s0 < KS; s0 += AHEAD) {
                u32x4 bv[AHEAD];
#pragma unroll
                for (int s = 0; s < AHEAD; ++s) bv[s] = *(const u32x4*)(X + (s0 + s) * PB * 64);
                if constexpr (KS >= 8) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int s = 0; s < AHEAD; ++s)
#pragma unroll
                    for (int m = 0; m < MT; ++m) acc[m][0] = Dense16<T>::mma(a[m][s0 + s], bv[s], acc[m][0]);
            }

            float v[4 * MT];
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int e = 0; e < 4; ++e) v[4 * m + e] = acc[m][0][e];
            epi_scale_bias_act_of<decltype(form)::value, 4 * MT>(v, ep, lds_ep + co_local, lds_ep + SPAN + co_local);
            const int row = 16 * wn + nn;
            const int64_t p = buffers.at(b) * PB + row;
            const auto live = [&] { return p < P && co_lane < Co; };  // Co is a multiple of 16 and the run is 16-aligned: all in or all out
            if (ep.residual)
                if (live()) epi_residual<TO, 4 * MT>(v, ep, p, co_lane);
            if (!TILE && !live()) {
                slot = slot + 1 == RING ? 0 : slot + 1;
                continue;
            }
            // this lane's run: into its row of the tile, or of the output
            char* const tile = out + (b & 1) * OUT;
            TO* const yp = y + p * ep.ldy + co_lane;
            auto piece = [&](int g) { return TILE ? tile + chunk_at(row, co_local * EB / 16 + g) * 16 : (char*)yp + 16 * g; };
            if constexpr (EB == 4) {
#pragma unroll
                for (int g = 0; g < MT; ++g) *(f32x4*)piece(g) = f32x4{v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
            } else if constexpr (MT == 1) {
                uint2 o;
                o.x = pack2_from_f32<TO>(v[0], v[1]);
                o.y = pack2_from_f32<TO>(v[2], v[3]);
                *(uint2*)(piece(0) + (TILE ? (co_local & 4) * 2 : 0)) = o;
            } else {
#pragma unroll
                for (int g = 0; g < MT / 2; ++g) {
                    *(u32x4*)piece(g) = pack8_from_f32<TO>(v + 8 * g);
                }
            }
            slot = slot + 1 == RING ? 0 : slot + 1;
        }
    });
    if constexpr (TILE) {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xc07f);
        __builtin_amdgcn_s_barrier();  // the last output tile is complete
        asm volatile("" ::: "memory");
        flush(count - 1, wave, std::integral_constant<int, 4>{});
    }
}

template <typename T, typename TO, int KS, int WM>
__global__ __launch_bounds__(64 * (4 + helper_waves(KS, WM)))
void conv1x1_stream_kernel(const T* __restrict__ x, TO* __restrict__ y, const char* __restrict__ wfrag, const char* __restrict__ zeros, int64_t P,
                           int Co, Divisor co_blocks, Share share, int total_wgs, int work_per_xcd, Epilogue ep)
{
    stream_outputs<T, TO, KS, WM, !Plan<KS, WM>::INTERLEAVED>(x, y, wfrag, zeros, P, Co, co_blocks, share, total_wgs, work_per_xcd, ep);
}
template <typename T, typename TO, int KS, int WM, bool TILE>
__global__ __launch_bounds__(64 * (4 + helper_waves(KS, WM)))
void conv1x1_stream_kernel(const T* __restrict__ x, TO* __restrict__ y, const char* __restrict__ wfrag, const char* __restrict__ zeros, int64_t P,
                           int Co, Divisor co_blocks, Share share, int total_wgs, int work_per_xcd, Epilogue ep)
{
    stream_outputs<T, TO, KS, WM, TILE>(x, y, wfrag, zeros, P, Co, co_blocks, share, total_wgs, work_per_xcd, ep);
}

// fp32, 32 to 256 channels: products on the bf16 matrix instruction, every value split into three parts (fp32_split.h).
//
// A workgroup owns 64 output channels and its share (share.h) of the buffers of 32 or 64 positions; each wave holds 16 channels' weights,
// split once, in registers.  Per buffer all four waves split its activations into LDS (the next buffer's are on their way
// meanwhile), each multiplies all positions, and the outputs go through LDS, so that they leave in rows of 256 bytes with
// scale, bias and shortcut read the same way.  Chunks of 16 bytes in LDS are permuted by position, for reads without bank
// conflicts.
// What bounds it: large launches of few channels the memory (64 -> 128 on 102 400 positions 18.3 us for 79 MB, 4.3 TB/s;
// 29 on the fp32 instruction), deeper ones the matrix and the splitting instructions together, which the waves of a compute unit,
// started at once, do at the same time rather than in turn (128 -> 128 on 25 600 positions: 28 % of the cycles matrix, 55 %
// vector): 9.6 us, on the fp32 instruction 14.5; 256 -> 256 on 25 600: 23.8 us, 33 there.  Buffers of 64 positions, which halve the
// splitting of weights, leave two workgroups on a compute unit instead of four: no faster at 128 channels, slower at 64.
constexpr int f32_positions(int KS) { return KS == 2 ? 64 : 32; }

template <typename T, typename TO, int KS>
__global__ __launch_bounds__(256, KS <= 8 ? 4 : 2) void conv1x1_stream_kernel(const float* __restrict__ x, float* __restrict__ y,
                                                             const char* __restrict__ wfrag, int64_t P, int Co, Divisor co_blocks,
                                                             Share share, int total_wgs, int work_per_xcd, Epilogue ep)
{
    constexpr int KK = KS / 2, PB = f32_positions(KS), TN = PB / 16;  // steps of 32 channels; blocks of 16 positions
    constexpr int ROW = 64 * KS, PLANE = KK * PB * 64;  // bytes of a position; of one bf16 part of a buffer
    constexpr int U = PB * KK / 64;                     // pieces of 2 x 4 channels a lane splits per buffer
    constexpr int STEPS = KS == 2 ? kSplitAll : kSplitSix;  // (few_live_products; 64 channels with k = 1 take the K split)
    static_assert(U * 64 == PB * KK, "whole rounds of pieces");
    __shared__ __attribute__((aligned(16))) char X[3 * PLANE];
    __shared__ __attribute__((aligned(16))) char out[PB * 256];  // 64 channels of a position, its 16-byte chunks permuted by position % 16

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // XCD-contiguous order: the channel blocks of one share's positions meet in an L2
    const int work = (blockIdx.x % 8) * work_per_xcd + blockIdx.x / 8;
    if (work >= total_wgs) return;
    const int part = co_blocks.quotient(work), cb = co_blocks.remainder(work, part);
    const Buffers buffers = share.of(part);

    u32x4 raw[U][2];
    auto load_activations = [&](int b) {
        const char* base = (const char*)x + (int64_t)b * (PB * ROW);
        const int last = (int)std::min<int64_t>(P - 1 - (int64_t)b * PB, PB - 1);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = u * 256 + tid, q = c & 3, pos = (c >> 2) % PB, kk = (c >> 2) / PB;
            const char* at = base + (min(pos, last) * ROW + kk * 128 + q * 16);  // (past the end: any, it is not stored)
            raw[u][0] = *(const u32x4*)at;
            raw[u][1] = *(const u32x4*)(at + 64);
        }
    };
    load_activations((int)buffers.at(0));
    // this wave's 16 channels, resident for the whole kernel
    Split8 a[KK];
    {
        const char* af = wfrag + (int64_t)(4 * cb + wave) * KS * kFrag + lane * 16;
        u32x4 r[KK][2];
#pragma unroll
        for (int s = 0; s < KS; ++s) r[s / 2][s % 2] = *(const u32x4*)(af + s * kFrag);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) a[kk] = split8(r[kk][0], r[kk][1]);
    }
    // ... and the 4 channels it stores
    const int co = 64 * cb + 4 * (tid & 15);
    f32x4 scale, bias;
    if (co < Co) {
        if (ep.scale) scale = *(const f32x4*)(ep.scale + co);
        if (ep.bias) bias = *(const f32x4*)(ep.bias + co);
    }

    const int nn = lane & 15, qq = lane >> 4;
    constexpr int MT = stream_mt_of(KS);
    const char* x_lane = X + nn * 64 + ((qq ^ ((nn >> 1) & 3)) * 16);
    // matrix rows 4 qq .. 4 qq + 3 of this wave's tile are these channels of the block (pack_plan.h)
    char* o_lane = out + nn * 256 + ((((wave / MT) * (4 * MT) + MT * qq + wave % MT) ^ nn) * 16);

    for (int i = 0; i < buffers.count; ++i) {
        const int b = (int)buffers.at(i);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = u * 256 + tid, q = c & 3, row = c >> 2;  // (step, position)
            const Split8 s = split8(raw[u][0], raw[u][1]);
            char* at = X + row * 64 + ((q ^ ((row >> 1) & 3)) * 16);
            *(u32x4*)at = s.h;
            *(u32x4*)(at + PLANE) = s.m;
            *(u32x4*)(at + 2 * PLANE) = s.l;
        }
        if (i + 1 < buffers.count) load_activations(b + buffers.step);
        const int64_t p0 = (int64_t)b * PB;
        EpiResidual<float, 4> shortcut[TN];
        if (ep.residual && co < Co)
#pragma unroll
            for (int i = 0; i < TN; ++i) {
                const int64_t p = p0 + 16 * i + (tid >> 4);
                if (p < P) shortcut[i].load(ep, p, co);
            }
        __syncthreads();
        f32x4 main[TN], small[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) main[j] = small[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < KK * TN / 2; ++i) {  // two blocks of positions at a time: the operands of four do not fit beside the rest
            const int kk = i % KK, j0 = i / KK * 2;
            Split8 v[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const char* at = x_lane + (kk * PB + 16 * (j0 + j)) * 64;
                v[j] = Split8{*(const u32x4*)at, *(const u32x4*)(at + PLANE), *(const u32x4*)(at + 2 * PLANE)};
            }
            split_steps<STEPS>([&](auto step) {
#pragma unroll
                for (int j = 0; j < 2; ++j) split_step<decltype(step)::value>(a[kk], v[j], main[j0 + j], small[j0 + j]);
            });
            if constexpr (KS == 2) __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) *(f32x4*)(o_lane + 16 * j * 256) = split_sum(main[j], small[j]);
        __syncthreads();
        if (co >= Co) continue;
        const auto base = store_base(y + p0 * ep.ldy);
        float v[4 * TN];
#pragma unroll
        for (int i = 0; i < TN; ++i) {
            f32x4 t = *(const f32x4*)(out + (16 * i + (tid >> 4)) * 256 + (((tid & 15) ^ (tid >> 4)) * 16));
            if (ep.scale) t *= scale;
            if (ep.bias) t += bias;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[4 * i + e] = t[e];
        }
        epi_act<4 * TN>(v, ep.act);
#pragma unroll
        for (int i = 0; i < TN; ++i) {
            const int64_t p = p0 + 16 * i + (tid >> 4);
            if (p >= P) break;
            float o[4] = {v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]};
            if (ep.residual) shortcut[i].add(o);
            store16_through(base, ((uint32_t)(16 * i + (tid >> 4)) * ep.ldy + co) * 4, __builtin_bit_cast(u32x4, f32x4{o[0], o[1], o[2], o[3]}));
        }
    }
}

template <int KS>
rtoss_status launch_f32(const rtoss_wdesc& d, const ConvParams& c, const char* wfrag, const void* x, void* y, hipStream_t s)
{
    const int64_t P = (int64_t)c.N * c.H * c.W;
    constexpr int PB = f32_positions(KS);
    const int64_t nbuf = (P + PB - 1) / PB;
    const int co_blocks = (d.Co + 63) / 64;
    auto kern = conv1x1_stream_kernel<float, float, KS>;
    static std::atomic<int> per_cu_cached{0};  // per instantiation
    int per_cu = per_cu_cached.load(std::memory_order_relaxed);
    if (per_cu == 0) {
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)kern, 256, 0) != hipSuccess || per_cu < 1) per_cu = 1;
        per_cu_cached.store(per_cu, std::memory_order_relaxed);
    }
    const int resident = std::max(8, c.dev.cus) * per_cu;
    const int wgs_per_cb = (int)std::max<int64_t>(1, std::min<int64_t>(nbuf, resident / co_blocks));
    const int total = wgs_per_cb * co_blocks;
    const int work_per_xcd = (total + 7) / 8;
    if (P * d.Ci * 4 / PB > 0x7fffffffffffll || nbuf > 0x7fffffff) return fail(RTOSS_ESHAPE, "conv1x1: too many positions");
    dim3 grid((unsigned)(work_per_xcd * 8)), block(256);
    kern<<<grid, block, 0, s>>>((const float*)x, (float*)y, wfrag, P, d.Co, Divisor(co_blocks), Share(nbuf, wgs_per_cb), total, work_per_xcd,
                             c.ep);
    return check_hip(hipGetLastError(), "conv1x1 stream launch");
}

// Launches whose outputs go straight from the accumulators, as they are: those of so few bytes that writing them back when the launch
// ends costs less than the way through the tile (about 0.2 us, 1 MB).  Layers of 32 and 64 16-bit channels (deeper ones of that size
// take the channel split) and of 16 fp32 channels.  us, from the accumulators / tile (MB of output in brackets):
//     32 ->  64 (0.01) 2.34 2.57     64 ->  64, fp32 results (0.4) 3.12 3.40     64 -> 512 (1.6)               2.90 2.99
//     32 -> 512 (1.6)  2.76 2.86     32 ->  64, fp32 results (1.6) 3.28 3.27     32 -> 512, fp32 results (3.3) 3.79 3.32
// Where blocks of channels are full, the stores through the tile run beside SiLU (but for a 16-bit shortcut's loads) and beside the fp32
// products:
//     64 ->  64, SiLU (0.2)  3.50 3.54     64 -> 256, SiLU and shortcut (0.8)               3.99 4.26     fp32 16 -> 64 (1.6) 3.09 2.79
//     32 -> 512, SiLU (1.6)  3.54 3.41     32 -> 256, SiLU and shortcut, fp32 results (1.6) 4.70 4.50     fp32 16 -> 16 (1.6) 3.16 3.61
//     32 -> 144, SiLU, fp32 results (0.9) 3.42 3.73
inline bool direct_outputs(const rtoss_wdesc& d, const ConvParams& c)
{
    const int KS = stage_count(d), span = 16 * stream_mt_of(KS) * stream_wm_of(KS, d.Co);
    const bool full = d.Co % span == 0, covered = full && c.ep.act == 2 && (!c.ep.residual || c.out_dt == RTOSS_F32);
    if (!stores_in_reach(c)) return true;
    if (full && d.dt == RTOSS_F32) return false;
    return (int64_t)c.N * c.H * c.W * d.Co * (int)elem_bytes(c.out_dt) <= (covered ? 1 << 19 : 2 << 20);
}

template <typename T, typename TO, int KS, int WM, bool... TILE>
rtoss_status launch_plan(const rtoss_wdesc& d, const ConvParams& c, const char* wfrag, const void* x, void* y, hipStream_t s)
{
    using PL = Plan<KS, WM>;
    const int64_t P = (int64_t)c.N * c.H * c.W;
    const int64_t nbuf = (P + PL::PB - 1) / PL::PB;
    const int co_blocks = stream_co_blocks_of(KS, d.Co);
    constexpr bool tiles = !PL::INTERLEAVED && sizeof...(TILE) == 0;
    const size_t smem = (size_t)PL::RING * PL::BUF + EpiScaleBias<PL::SPAN>::kBytes + (tiles ? 2 * PL::PB * PL::SPAN * sizeof(TO) : 0);
    auto kern = conv1x1_stream_kernel<T, TO, KS, WM, TILE...>;
    static LaunchOnce lds_once;  // per instantiation
    if (rtoss_status st = ensure_dynamic_lds((const void*)kern, smem, lds_once, c.dev.device, "conv1x1 shared memory attribute")) return st;
    // Persistent workgroups: as many as are resident at once, but no fewer than 2 buffers each: every
    // workgroup loads its weight fragments once, which for deep layers is more bytes than a buffer.
    // fp32 steps take 16 times as long: there a launch that gives most compute units one workgroup or none is spread over
    // all of them, one buffer each (16 -> 16 channels on 12 800 positions: 2.8 us with one buffer, 3.2 with two).
    // (workgroups per compute unit depend on the instantiation's registers and LDS only: asked once; the
    // number of compute units is the current device's)
    static std::atomic<int> per_cu_cached{0};  // per instantiation
    int per_cu = per_cu_cached.load(std::memory_order_relaxed);
    if (per_cu == 0) {
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)kern, PL::LANES, smem) != hipSuccess || per_cu < 1) per_cu = 1;
        // The dispatcher spreads a workgroup's waves over the four SIMDs but does not fill every hole: of `waves` that fit a SIMD,
        // workgroups of five were resident at two per compute unit for four, three for five and four for six, one less
        // than the query says.  Workgroups beyond that are a second round of a launch planned for one
        // (128 -> 128 on 102 400 positions: 13.5 us with 768 of which 512 fit, 12.3 with 512; 280 shapes 0.96 of the time with the
        // query's number.  Workgroups of six come out at the query's number or within 2 % of its time).
        int waves = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&waves, (const void*)kern, 256, 0) == hipSuccess)
            per_cu = std::max(1, std::min(per_cu, (4 * waves - 4 + PL::HELPERS) / (4 + PL::HELPERS)));
        per_cu_cached.store(per_cu, std::memory_order_relaxed);
    }
    const DeviceInfo& dev = c.dev;
    const int resident = std::max(8, dev.cus) * per_cu;
    const bool spread = sizeof(T) == 4 && 2 * nbuf * co_blocks <= 3 * dev.cus;
    const int64_t by_work = spread ? nbuf : std::max<int64_t>(1, (nbuf + 1) / 2);
    const int wgs_per_cb = (int)std::max<int64_t>(1, std::min<int64_t>(by_work, resident / co_blocks));
    const int total = wgs_per_cb * co_blocks;
    const int work_per_xcd = (total + 7) / 8;
    if (P * d.Ci * (int)sizeof(T) / PL::PB > 0x7fffffffffffll || nbuf > 0x7fffffff) return fail(RTOSS_ESHAPE, "conv1x1: too many positions");
    dim3 grid((unsigned)(work_per_xcd * 8)), block(PL::LANES);
    kern<<<grid, block, smem, s>>>((const T*)x, (TO*)y, wfrag, wfrag + frag_bytes(d), P, d.Co, Divisor(co_blocks),
                                   Share(nbuf, wgs_per_cb), total, work_per_xcd, c.ep);
    return check_hip(hipGetLastError(), "conv1x1 stream launch");
}

constexpr bool has_direct_outputs(int KS, bool f32) { return KS <= (f32 ? 1 : 2); }
template <typename T, typename TO, int KS, int WM>
rtoss_status launch_wm(const rtoss_wdesc& d, const ConvParams& c, const char* wfrag, const void* x, void* y, hipStream_t s)
{
    if constexpr (has_direct_outputs(KS, sizeof(T) == 4))
        if (direct_outputs(d, c)) return launch_plan<T, TO, KS, WM, false>(d, c, wfrag, x, y, s);
    return launch_plan<T, TO, KS, WM>(d, c, wfrag, x, y, s);
}

template <typename T, typename TO, int KS>
rtoss_status launch_ks(const rtoss_wdesc& d, const ConvParams& c, const char* wfrag, const void* x, void* y, hipStream_t s)
{
    const int wm = stream_wm_of(KS, d.Co);
    if constexpr (KS <= 8)
        if (wm == 1) return launch_wm<T, TO, KS, 1>(d, c, wfrag, x, y, s);
    if constexpr (KS <= 16)
        if (wm == 2) return launch_wm<T, TO, KS, 2>(d, c, wfrag, x, y, s);
    return launch_wm<T, TO, KS, 4>(d, c, wfrag, x, y, s);
}

template <typename T, typename TO>
rtoss_status launch_typed(const rtoss_wdesc& d, const ConvParams& c, const char* wfrag, const void* x, void* y, hipStream_t s)
{
    const int KS = stage_count(d);
    if (KS == 1) return launch_ks<T, TO, 1>(d, c, wfrag, x, y, s);
    if (KS == 32) return launch_ks<T, TO, 32>(d, c, wfrag, x, y, s);
    if constexpr (sizeof(T) == 4) {
        if (KS == 2) return launch_f32<2>(d, c, wfrag, x, y, s);
        if (KS == 4) return launch_f32<4>(d, c, wfrag, x, y, s);
        if (KS == 8) return launch_f32<8>(d, c, wfrag, x, y, s);
        if (KS == 16) return launch_f32<16>(d, c, wfrag, x, y, s);
    } else {
        if (KS == 2) return launch_ks<T, TO, 2>(d, c, wfrag, x, y, s);
        if (KS == 4) return launch_ks<T, TO, 4>(d, c, wfrag, x, y, s);
        if (KS == 8) return launch_ks<T, TO, 8>(d, c, wfrag, x, y, s);
        if (KS == 16) return launch_ks<T, TO, 16>(d, c, wfrag, x, y, s);
    }
    return fail(RTOSS_ESHAPE, "conv1x1 stream: unsupported input channel count %d", d.Ci);
}

}  // namespace

// ---- host-visible entry points of this file ----

bool stream1x1_shape_ok(const rtoss_wdesc& d)
{
    const int KS = stage_count(d);
    return d.ksize == 1 && d.Ci * elem_bytes(d.dt) % 64 == 0 && d.Co % 16 == 0 && KS >= 1 && KS <= 32 && (KS & (KS - 1)) == 0;
}

// (fp32 results of 512 channels are stored at 64-bit addresses)
bool stream1x1_launch_ok(const rtoss_wdesc& d, const ConvParams& c)
{
    const int KS = stage_count(d);
    return stores_in_reach(c) || ksplit1x1_plan(d, c) || has_direct_outputs(KS, d.dt == RTOSS_F32) ||
           (KS == 16 && d.dt != RTOSS_F32 && c.out_dt == RTOSS_F32);
}

size_t stream1x1_section_bytes(const rtoss_wdesc& d) { return frag_bytes(d) + zero_section_bytes(stage_count(d)); }

rtoss_status launch_conv1x1_stream(const rtoss_wdesc& d, const ConvParams& c, const void* section, const void* x, void* y,
                                   hipStream_t s)
{
    const char* wf = (const char*)section;
    const bool f32out = c.out_dt == RTOSS_F32;
    if (const int plan = ksplit1x1_plan(d, c)) return launch_conv1x1_ksplit(d, c, plan, section, x, y, s);
    if (d.dt == RTOSS_F32) return launch_typed<float, float>(d, c, wf, x, y, s);
    if (d.dt == RTOSS_F16)
        return f32out ? launch_typed<f16_t, float>(d, c, wf, x, y, s) : launch_typed<f16_t, f16_t>(d, c, wf, x, y, s);
    return f32out ? launch_typed<bf16_t, float>(d, c, wf, x, y, s) : launch_typed<bf16_t, bf16_t>(d, c, wf, x, y, s);
}

}  // namespace rtoss
