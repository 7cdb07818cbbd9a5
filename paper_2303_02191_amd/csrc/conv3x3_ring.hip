// 3x3 pattern-pruned convolution, stride 1, over strips of output rows, with helper waves: launches of one round of workgroups that are too
// large for conv3x3_ksplit.hip and too small for the persistent pipeline (conv3x3_rows.hip).  Reads the packed sections of sparse_frag.h; operands
// as in conv3x3_strip.hip: a wave owns TN rows of 16 columns and the 64 channels of its workgroup.
//
// In the strips without helpers a stage of such a launch is a chain: the four waves issue its 34 to 50 copies (about 70 cycles each), wait
// for the stage before, meet and multiply, and one or two workgroups per compute unit cover little of each other.  Here four helper waves, one
// beside each of the four that multiply, keep a ring of three or four stages filled, and a wave that multiplies does nothing else: it crosses
// one barrier a stage, asks for the next stage's first operands behind it and permutes each row's operand behind the matrix instructions
// of the row in front (RingSchedule).  256 -> 256 channels, us: 1x50x84 9.8 -> 8.5, 1x100x168 17.5 -> 15.7 (0.39 and 0.42 of the matrix rate
// while the stages run).
// What bounds it: a stage takes 0.16 us and 0.21 us more per row, i.e. 20 matrix instructions of 16 cycles in 23 to 25 each, about four instructions
// around each of them in the one wave of a SIMD; with TN = 2 LDS, whose 1390 cycles a stage (fragments read by all four waves, windows, copies)
// are the whole 0.58 us.  Left to the compiler's own order the stages took 0.03 to 0.12 us more.
#include <type_traits>

#include "common.h"
#include "dtypes.h"
#include "epilogue.h"
#include "mma.h"
#include "sparse_frag.h"
#include "work_order.h"
#include "strip_output.h"

namespace rtoss {

namespace {

constexpr int kTM = kStripTM, kCols = kStripCols, kLW = kStripLW;

template <int TN, int LAY> struct Ring {
    static constexpr int ROWS = 4 * TN;  // output rows of a workgroup
    static constexpr int TILE = layout_tile_bytes(kLayouts[LAY]);
    static constexpr int A_BYTES = kTM * TILE;
    static constexpr int A_COPIES = A_BYTES / 1024;  // 64 lanes x 16 bytes each
    static constexpr int X_COPIES = ((ROWS + 2) * kLW * 4 + 63) / 64;
    static constexpr int COPIES = A_COPIES + X_COPIES;
    static constexpr int PER_WAVE = (COPIES + 3) / 4;  // of a helper
    static constexpr int BUF = COPIES * 1024;          // one stage: [weights][activations]
    static constexpr int EP_BYTES = EpiScaleBias<16 * kTM>::kBytes;
    static constexpr int BUFFERS = 4 * BUF + EP_BYTES <= 160 * 1024 ? 4 : 3;
    static constexpr int LDS = BUFFERS * BUF + EP_BYTES;
    static_assert(A_BYTES % 1024 == 0, "weight fragments are whole copy instructions");
    static_assert(LDS <= 160 * 1024, "a compute unit's LDS");
    static_assert((BUFFERS - 1) * PER_WAVE < 64, "copies under way within the counter's range");
    static_assert(4 * TN * 2048 <= BUF, "the output tiles of all waves fit a buffer");
};

// Waits until at most `left` of the copies that this wave has under way (whole stages of N each) have not landed.
template <int N> __device__ __forceinline__ void wait_stages(int left)
{
    constexpr auto vm = [](int n) { return 0x0f70 | (n & 15) | (n >> 4) << 14; };  // vmcnt(n) alone
    if (left >= 2) __builtin_amdgcn_s_waitcnt(vm(2 * N));
    else if (left == 1) __builtin_amdgcn_s_waitcnt(vm(N));
    else __builtin_amdgcn_s_waitcnt(vm(0));
}

__device__ __forceinline__ void bare_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// When a stage asks for what.  A stage is PHASES x TN rows x 4 matrix instructions (the centre's, then two halves of each group of four taps;
// the four channel tiles of a row of outputs), one slot each.  The operand of a row is permuted behind the four instructions of the row in front
// of it; reads go out kLead slots ahead of that.  Slots from SLOTS on are the last ones of the stage before, behind the barrier.
template <int TN, int LAY> struct RingSchedule {
    static constexpr TapLayout LY = kLayouts[LAY];
    static constexpr int PHASES = LY.centre + 2 * LY.groups;
    static constexpr int SLOTS = PHASES * TN * 4;
    static constexpr int kLead = 12;
    static constexpr int BARRIER = SLOTS - kLead - 6;
    static constexpr int group(int p) { return p < LY.centre ? -1 : (p - LY.centre) / 2; }
    static constexpr int half(int p) { return (p - LY.centre) % 2; }
    static constexpr int fragment(int p) { return p < LY.centre ? 2 * LY.groups : p - LY.centre; }
    static constexpr int tap(int g, int f) { return LY.tap[g][f]; }
    // a slot of the stage, or of the one before where that is too early
    static constexpr int place(int slot) { return slot >= 0 ? slot : slot + SLOTS > BARRIER ? slot + 2 * SLOTS : BARRIER + 1 + SLOTS; }
    // 16-byte reads of input row i at column shift kw
    static constexpr int window_slot(int i, int kw)
    {
        for (int row = 0; row < PHASES * TN; ++row) {
            const int p = row / TN, j = row % TN;
            if (group(p) < 0) {
                if (i == j + 1 && kw == 1) return place(4 * row - kLead);
                continue;
            }
            for (int f = 0; f < 4; ++f)
                if (i == j + tap(group(p), f) / 3 && kw == tap(group(p), f) % 3) return place(4 * (row - 1) - kLead);
        }
        return -1;
    }
    static constexpr int weight_slot(int p, int m) { return place(p > 0 && 4 * p * TN < kLead + 4 ? m : 4 * p * TN - kLead - 4 + m); }

    // The same as lists: what slot s reads, entries first[s] .. first[s + 1] - 1 (windows 3 * i + kw, then fragments 4 * p + m from kWindows on).
    static constexpr int kWindows = 3 * (TN + 2), kReads = kWindows + PHASES * kTM;
    struct Lists {
        int first[2 * SLOTS + 1] = {}, what[kReads] = {};
    };
    static constexpr Lists make()
    {
        Lists l;
        int slot[kReads] = {}, n = 0;
        for (int w = 0; w < kWindows; ++w) slot[w] = window_slot(w / 3, w % 3);
        for (int w = 0; w < PHASES * kTM; ++w) slot[kWindows + w] = weight_slot(w / kTM, w % kTM);
        for (int s = 0; s < 2 * SLOTS; ++s) {
            l.first[s] = n;
            for (int w = 0; w < kReads; ++w)
                if (slot[w] == s) l.what[n++] = w;
        }
        l.first[2 * SLOTS] = n;
        return l;
    }
    static constexpr Lists lists = make();
    static_assert(lists.first[2 * SLOTS] == kReads, "everything is read once");
};

template <int TN, int LAY, typename T, typename TO>
__global__ __launch_bounds__(512, 2) void conv3x3_ring_kernel(const T* __restrict__ x, TO* __restrict__ y, const char* __restrict__ wfrag,
                                                               const char* __restrict__ zeros, int H, int W, int Ci, int Co, int m_tiles_total,
                                                               WorkOrder order, Epilogue ep)
{
    using P = Ring<TN, LAY>;
    constexpr TapLayout LY = kLayouts[LAY];
    constexpr int FR = layout_fragments(LY), NB = P::BUFFERS;
    extern __shared__ __attribute__((aligned(16))) char smem[];  // [buffer]..., [scale, bias]
    float* const lds_ep = (float*)(smem + NB * P::BUF);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int work = order.item();
    if (work >= order.total) return;
    const int all_tile = order.co_blocks.quotient(work), cb = order.co_blocks.remainder(work, all_tile);
    const WorkOrder::Tile tile = order.tile(all_tile);
    const int n_img = tile.n_img, oh0 = tile.row * P::ROWS, ow0 = tile.col * kCols;
    const int stages = Ci / 32;

    // Barrier s, which every wave of the workgroup passes: stage s is in LDS, and nobody reads stage s - 1 any more.
    if (wave >= 4) {
        // ---- helpers: wave h issues copies h, h + 4, ... of a stage (weights, then activations; the last one again where there is none left) ----
        const int h = wave - 4;
        constexpr int A_ONLY = P::A_COPIES / 4, XN = P::PER_WAVE - A_ONLY;
        const char* a_src = wfrag + (int64_t)cb * P::A_BYTES + h * 1024 + lane * 16;
        const int64_t a_stage_stride = (int64_t)m_tiles_total * P::TILE;
        const char* src[XN];
        int64_t step[XN];
#pragma unroll
        for (int k = 0; k < XN; ++k) {
            const int c = min((A_ONLY + k) * 4 + h, P::COPIES - 1);
            const int pos = (c - P::A_COPIES) * 16 + (lane >> 2);
            const int xr = pos / kLW, xc = pos % kLW;
            const int ih = oh0 - 1 + xr, iw = ow0 - 1 + xc;
            const bool inside = xr < P::ROWS + 2 && (unsigned)ih < (unsigned)H && (unsigned)iw < (unsigned)W;
            const int off = ((n_img * H + ih) * W + iw) * (Ci / 8) + (lane & 3);  // in 16-byte chunks (31 bits: checked by the launcher)
            src[k] = inside ? (const char*)x + (int64_t)off * 16 : zeros;
            step[k] = 64;
            if (A_ONLY * 4 != P::A_COPIES && k == 0 && c < P::A_COPIES) src[k] = a_src + A_ONLY * 4096, step[k] = a_stage_stride;
        }
        auto issue = [&](int stage) {
            char* const buf = smem + stage % NB * P::BUF;
#pragma unroll
            for (int k = 0; k < A_ONLY; ++k) copy16_to_lds(a_src + stage * a_stage_stride + k * 4096, buf + (4 * k + h) * 1024);
#pragma unroll
            for (int k = 0; k < XN; ++k) copy16_to_lds(src[k] + stage * step[k], buf + min((A_ONLY + k) * 4 + h, P::COPIES - 1) * 1024);
        };
        // (the copies of two stages in front of the first barrier, the others behind it)
        int issued = 0;
        for (; issued < min(2, stages); ++issued) issue(issued);
        for (int s = 0; s < stages; ++s) {
            wait_stages<P::PER_WAVE>(issued - 1 - s);
            bare_barrier();
            for (; issued < min(s + NB, stages); ++issued) issue(issued);
        }
        return;
    }

    EpiScaleBias<16 * kTM> scale_bias;
    scale_bias.load(ep, 64 * cb, Co, tid);
    scale_bias.store(lds_ep, ep, tid);

    const int xoff = P::A_BYTES + (wave * TN * kLW + (lane & 15)) * 64 + (lane >> 4) * 16;
    using Q = RingSchedule<TN, LAY>;
    constexpr int S = Q::SLOTS;
    // What a stage asks for on behalf of the next: windows, the first phase's weights and, without a centre, its first operand.
    f32x4 acc[kTM][TN];
    u32x4 R_next[TN + 2][3], a_next[kTM];
    u32x8 b_next;
    int i_next[kTM];
#pragma unroll
    for (int m = 0; m < kTM; ++m)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[m][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto read_window = [&](const char* buf, int i, int kw) { return *(const u32x4*)(buf + xoff + (i * kLW + kw) * 64); };
    auto read_weights = [&](const char* buf, int p, int m) { return *(const u32x4*)(buf + m * P::TILE + Q::fragment(p) * kFragBytes + lane * 16); };
    auto read_index = [&](const char* buf, int p, int m) { return *(const int*)(buf + m * P::TILE + FR * kFragBytes + (Q::group(p) * 64 + lane) * 4); };
    // reads of slot s (a stage's own), or of slot s on behalf of the next stage (from SLOTS on)
    auto read_slot = [&](auto slot_tag, const char* buf, u32x4 (&r)[TN + 2][3], auto&& weights) {
        constexpr int s = decltype(slot_tag)::value, first = Q::lists.first[s];
        static_for<Q::lists.first[s + 1] - first>([&](auto n_tag) {
            constexpr int w = Q::lists.what[first + decltype(n_tag)::value], q = w - Q::kWindows;
            if constexpr (q < 0) r[w / 3][w % 3] = read_window(buf, w / 3, w % 3);
            else weights(std::integral_constant<int, q>{});
        });
    };
    auto read_next = [&](auto slot_tag, const char* buf) {
        read_slot(slot_tag, buf, R_next, [&](auto q_tag) {
            constexpr int m = decltype(q_tag)::value;
            static_assert(m < kTM, "the first phase's");
            a_next[m] = read_weights(buf, 0, m);
            if constexpr (Q::group(0) >= 0) i_next[m] = read_index(buf, 0, m);
        });
    };
    // two of the eight byte permutations of operand (p, row j): sparse_operand in four parts
    auto permute = [&](int part, int p, int j, const u32x4 (&r)[TN + 2][3], u32x8& b) __attribute__((always_inline)) {
        const int g = Q::group(p), d = 2 * Q::half(p) + part / 2;
        const uint32_t sel = part & 1 ? 0x07060302u : 0x05040100u;
        const int t0 = Q::tap(g, 0), t1 = Q::tap(g, 1), t2 = Q::tap(g, 2), t3 = Q::tap(g, 3);
        b[2 * part] = __builtin_amdgcn_perm(r[j + t1 / 3][t1 % 3][d], r[j + t0 / 3][t0 % 3][d], sel);
        b[2 * part + 1] = __builtin_amdgcn_perm(r[j + t3 / 3][t3 % 3][d], r[j + t2 / 3][t2 % 3][d], sel);
    };
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // (scale and bias)
    bare_barrier();
    static_for<S>([&](auto slot_tag) { read_next(std::integral_constant<int, S + decltype(slot_tag)::value>{}, smem); });
    if constexpr (Q::group(0) >= 0) {
#pragma unroll
        for (int part = 0; part < 4; ++part) permute(part, 0, 0, R_next, b_next);
    }

    auto run_stage = [&](auto last_tag, int stage) {
        constexpr bool LAST = decltype(last_tag)::value;
        const char* const buf = smem + stage % NB * P::BUF;
        const char* const next_buf = smem + (stage + 1) % NB * P::BUF;
        u32x4 R[TN + 2][3], a[Q::PHASES][kTM];
        u32x8 b[2];
        int idx[LY.groups][kTM];
#pragma unroll
        for (int w = 0; w < Q::kWindows; ++w) R[w / 3][w % 3] = R_next[w / 3][w % 3];
#pragma unroll
        for (int m = 0; m < kTM; ++m) {
            a[0][m] = a_next[m];
            if constexpr (Q::group(0) >= 0) idx[0][m] = i_next[m];
        }
        if constexpr (Q::group(0) >= 0) b[0] = b_next;
        static_for<S>([&](auto slot_tag) {
            constexpr int s = decltype(slot_tag)::value, p = s / (4 * TN), j = s / 4 % TN, m = s % 4, g = Q::group(p), row = s / 4;
            if constexpr (g < 0) acc[m][j] = Dense16<T>::mma(a[p][m], R[j + 1][1], acc[m][j]);
            else acc[m][j] = Sparse64<T>::template mma<Q::half(p)>(a[p][m], b[row % 2], acc[m][j], idx[g][m]);
            if constexpr (s == Q::BARRIER && !LAST) {
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // this wave's reads of the stage
                bare_barrier();
            }
            read_slot(slot_tag, buf, R, [&](auto q_tag) {
                constexpr int q = decltype(q_tag)::value, ph = q / kTM, n = q % kTM;
                a[ph][n] = read_weights(buf, ph, n);
                if constexpr (Q::group(ph) >= 0 && Q::half(ph) == 0) idx[Q::group(ph)][n] = read_index(buf, ph, n);
            });
            if constexpr (!LAST) read_next(std::integral_constant<int, s + S>{}, next_buf);
            // the next row's operand
            if constexpr (row + 1 < Q::PHASES * TN) {
                if constexpr (Q::group((row + 1) / TN) >= 0) permute(m, (row + 1) / TN, (row + 1) % TN, R, b[(row + 1) % 2]);
            } else if constexpr (Q::group(0) >= 0 && !LAST) {
                permute(m, 0, 0, R_next, b_next);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    for (int stage = 0; stage + 1 < stages; ++stage) run_stage(std::false_type{}, stage);
    run_stage(std::true_type{}, stages - 1);

    // (past the L2's write-back whatever the channels: half sectors cost the stores more on tensors in no cache, and the launch is still faster than
    // one that leaves them to the L2; us, strips with stores from the registers and here, tensors in caches, then in none, 4 entries: 256 -> 208
    // on 1x100x168 21.3 17.7, 23.7 20.1; 256 -> 80 on 1x200x168 21.7 19.0, 24.5 19.9; 128 -> 208 on 1x100x168 14.2 12.0, 15.2 13.8)
    constexpr bool ROWS_OUT = sizeof(TO) == 2;
    char* const area = smem + stages % NB * P::BUF + wave * (TN * RowTile<TO>::kBytes);  // (a buffer that the last stage does not read)
    strip_output<TO, TN, ROWS_OUT>(acc, area, lds_ep, y, H, W, Co, cb, n_img, oh0 + wave * TN, ow0, lane, ep);
}

template <int TN, int LAY, typename T, typename TO>
rtoss_status launch_ring(const rtoss_wdesc& d, const ConvParams& c, const char* wf, const char* zeros, const void* x, void* y, hipStream_t s)
{
    using P = Ring<TN, LAY>;
    const int strips = (c.W + kCols - 1) / kCols, rows = (c.H + P::ROWS - 1) / P::ROWS, co_blocks = (d.Co + 63) / 64;
    auto kern = conv3x3_ring_kernel<TN, LAY, T, TO>;
    static LaunchOnce lds_once;  // per instantiation
    if (rtoss_status st = ensure_dynamic_lds((const void*)kern, P::LDS, lds_once, c.dev.device, "conv3x3 shared memory attribute")) return st;
    const int64_t total = (int64_t)strips * rows * co_blocks * c.N;
    const WorkOrder order(total, co_blocks, strips * rows, strips);
    kern<<<dim3(order.grid()), dim3(512), P::LDS, s>>>((const T*)x, (TO*)y, wf, zeros, c.H, c.W, d.Ci, d.Co, padded_m_tiles(d.Co), order, c.ep);
    return check_hip(hipGetLastError(), "conv3x3 ring launch");
}

template <int TN, int LAY>
rtoss_status launch_typed(const rtoss_wdesc& d, const ConvParams& c, const char* wf, const char* zeros, const void* x, void* y, hipStream_t s)
{
    if (d.dt == RTOSS_F16) return launch_ring<TN, LAY, f16_t, f16_t>(d, c, wf, zeros, x, y, s);
    return launch_ring<TN, LAY, bf16_t, bf16_t>(d, c, wf, zeros, x, y, s);
}

template <int LAY>
rtoss_status launch_rows(const rtoss_wdesc& d, const ConvParams& c, int plan, const char* wf, const char* zeros, const void* x, void* y, hipStream_t s)
{
    switch (plan) {
    case 2: return launch_typed<2, LAY>(d, c, wf, zeros, x, y, s);
    case 3: return launch_typed<3, LAY>(d, c, wf, zeros, x, y, s);
    case 4: return launch_typed<4, LAY>(d, c, wf, zeros, x, y, s);
    case 5: return launch_typed<5, LAY>(d, c, wf, zeros, x, y, s);
    }
    return fail(RTOSS_EINVAL, "conv: unknown ring plan %d", plan);
}

}  // namespace

// The smallest TN whose workgroups the compute units hold at once, one each, where its stages are faster than those of the kernels without helpers by
// more than its longer start and end.  us a stage, layout 0 (layout 1: 1.2 times): here 0.58, 0.79, 1.0, 1.21 with TN = 2 .. 5; there 0.82 with
// eight rows once over the chip, 1.09 with twelve once, 1.29 and 1.87 twice, 3.1 in taller strips; the start costs 0.35 us more per TN here.
// (bf16, without helpers and with: 1x256@50x84 9.8 8.5, 16x256@20x20 11.9 10.6, 1x256@100x168 18.2 15.7, 1x512@50x84 20.6 18.3, 16x512@20x20
// 33.3 25.8, 1x128@100x168 7.8 7.4; layout 1: 11.5 9.8, 15.6 12.6, 21.4 18.5, 27.6 21.8, 39.1 31.5, 9.5 8.4.  Not 4x128@80x80, 8.6 8.7, nor
// 16x128@40x40, 8.8 9.9: eight rows twice over the chip.  Where eight rows go twice over the chip and 16 once, means of 22 to 30 launches of 64 to
// 384 output channels, on tensors in caches and in none: 3 stages 1.03 times as long with helpers (layout 1), 4 1.03 (layout 1: 1.01), 5 0.99 (0.98),
// 6 0.99 (0.97), 8 0.94 (0.93).)
// The pipelined kernel is not asked about: its least unit of work, a tile of 16 rows and 128 channels, takes 2.5 us a stage.
int ring3x3_plan(const rtoss_wdesc& d, const ConvParams& c, int layout)
{
    if (c.stride != 1 || d.Ci % 32 || d.Co % 16 || d.Ci < 64) return 0;
    if (c.out_dt == RTOSS_F32 || !stores_in_reach(c) || (int64_t)c.N * c.H * c.W * d.Ci / 8 > kMaxChunks) return 0;  // (16-bit results, in rows)
    const int64_t cus = c.dev.cus;
    const auto groups = [&](int tn) {
        return (int64_t)((c.W + kCols - 1) / kCols) * ((c.H + 4 * tn - 1) / (4 * tn)) * ((d.Co + 63) / 64) * c.N;
    };
    int tn = 2;
    while (tn <= 5 && groups(tn) > cus) ++tn;
    if (tn > 5) return 0;
    const double there = groups(2) <= cus                             ? 0.82
                         : layout == 0 && groups(3) <= cus            ? 1.09
                         : groups(2) <= 2 * cus                       ? 1.29
                         : groups(3) <= 2 * cus                       ? 1.87
                                                                      : 3.1;
    const double gain = there - (0.16 + 0.21 * tn);
    return d.Ci / 32 * (layout == 0 ? 1 : 1.2) * gain > 0.35 * tn ? tn : 0;
}

rtoss_status launch_conv3x3_ring(const rtoss_wdesc& d, const ConvParams& c, int layout, int plan, const void* section, const void* zeros,
                                 const void* x, void* y, hipStream_t s)
{
    const char *wf = (const char*)section, *z = (const char*)zeros;
    return layout == 1 ? launch_rows<1>(d, c, plan, wf, z, x, y, s) : launch_rows<0>(d, c, plan, wf, z, x, y, s);
}

}  // namespace rtoss
