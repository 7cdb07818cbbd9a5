// 3x3 stride-1 pattern-sparse convolution for large layers: the pipelined kernel on the sparse
// matrix instruction (operand layouts, fragment format and the corner / edge / centre split of the
// taps: see conv3x3_sparse.hip and sparse_frag.h).
//
// Shape of the work.  A workgroup (4 waves) owns 128 output channels x a strip of 16 output columns x
// 4*TN output rows; wave v owns the TN rows [v*TN, v*TN + TN) of the strip, all 128 channels.  The 16
// columns of a matrix instruction are 16 CONSECUTIVE positions of one output row.  That makes the B
// operands (activations) of the nine taps overlapping windows of the same LDS rows: with
//     R[i][kw] = the 16-byte read (8 channels) of input row i of the wave at column shift kw,
// output row j takes tap (kh, kw) from R[j + kh][kw].  A wave reads the 3 * (TN + 2) vectors R once per
// stage and every one serves up to three output rows and three taps, instead of nine reads per output
// row: the LDS read traffic of the activations drops by half (TN = 5: 21 reads instead of 45), and each
// read is 1024 contiguous bytes, free of bank conflicts at any row pitch.
//
// K runs over stages of 32 input channels, double-buffered in LDS: the stage's weight fragments (one
// contiguous chunk of the packed blob) and its activation tile with halo are copied global -> LDS
// without passing through registers while the previous stage is multiplied.  A stage is 5 phases
// (centre, corner step 0/1, edge step 0/1) x 4 pairs of channel tiles = 20 units of 2*TN matrix
// instructions.  The centre phase multiplies R[j+1][1] as it is; the sparse phases need, per lane,
// 4 channels x the 4 taps of a group, i.e. 4x4 (tap x channel) transposes of four R vectors, done with
// byte permutes behind the matrix instructions of earlier units.
//
// Workgroups are persistent, one per compute unit.  Rows of a strip are cut into tall tiles (TN = 5:
// 20 rows) and short ones (TN = 4: 16 rows); the host picks the cut per strip so that every workgroup's
// share of tiles takes about the same time (rows_cut.h): a workgroup runs its tall tiles, then
// its short ones.
#pragma once
#include <type_traits>

#include "common.h"
#include "dtypes.h"
#include "epilogue.h"
#include "mma.h"
#include "rows_plan.h"
#include "sparse_frag.h"

namespace rtoss {

namespace {

// Which unit of a stage reads and permutes what (TN = rows per wave).
//   prologue (issued inside the previous stage's last unit): R[1..TN][1], R[0..3][0], R[0..3][2]
//   unit u <= TN-3: R[u+4][0], R[u+4][2];   unit TN-2: R[0][1], R[TN+1][1]
//   corner job j (taps 0,2,6,8 of output row j: R[j][0], R[j][2], R[j+2][0], R[j+2][2]) is permuted in unit
//   max(0, j-1), the unit after its last read; edge job j (taps 1,3,5,7: R[j][1], R[j+1][0], R[j+1][2],
//   R[j+2][1]) in unit TN-1+j.  Corner operands are complete before unit 4, edge operands before unit 12.
template <int TN> struct RowSchedule {
    static_assert(TN >= 3 && TN <= 5, "corner jobs must be permuted within the centre phase");
    static constexpr int jobs = 2 * TN;  // job q < TN: corner taps of row q; job TN + j: edge taps of row j
    static constexpr int perm_unit(int q) { return q < TN ? (q < 2 ? 0 : q - 1) : TN - 1 + (q - TN); }
    static constexpr int perm_count(int u)
    {
        int n = 0;
        for (int q = 0; q < jobs; ++q) n += perm_unit(q) == u;
        return n;
    }
    static constexpr int perm_first(int u)
    {
        for (int q = 0; q < jobs; ++q)
            if (perm_unit(q) == u) return q;
        return 0;
    }
    // row whose shifted columns 0 and 2 are read in unit u (-1: none)
    static constexpr int side_row(int u) { return u <= TN - 3 ? u + 4 : -1; }
    static constexpr bool reads_outer_mid(int u) { return u == TN - 2; }
};

// (input row, column shift) of tap slot f of a job
template <int TN> struct JobTap {
    static constexpr int row(int q, int f)
    {
        return q < TN ? q + (f >> 1) * 2                               // corners: rows j, j, j+2, j+2
                      : (q - TN) + (f == 0 ? 0 : f == 3 ? 2 : 1);      // edges: rows j, j+1, j+1, j+2
    }
    static constexpr int shift(int q, int f)
    {
        return q < TN ? (f & 1) * 2                                    // corners: columns 0, 2, 0, 2
                      : (f == 1 ? 0 : f == 2 ? 2 : 1);                 // edges: columns 1, 0, 2, 1
    }
};

// The same for a layout of tap groups without a centre (layout 1).  A stage is 6 phases (two steps a group) x 4 pairs of channel tiles = 24
// units.  There is no centre phase under which the first operands could be permuted, so every phase permutes the next one's, one
// permute behind each matrix instruction, and the last phase those of the next stage: the stage is handed over at the start of that phase,
// when all of its activations have been read and permuted; only the fragments of the last units are read ahead for that.  (Hand-over before
// that phase would overwrite windows that are still to be permuted.)
// What bounds it: a stage of a tall tile is 240 matrix instructions of 18 cycles in 6.1 k cycles (layout 0: 200 in 4.8 k); LDS is busy for half of
// that.  us, bf16, 5 entries, before in dense mode / 4 entries, before in strips: 256 -> 256 on 2x100x168 33.5 28.4 / 33.8 28.2, on 4x100x168
// 64.2 52.2 / 64.4 52.0, 128 -> 128 on 4x100x168 19.8 17.4 / 19.2 17.3.  The next stage's reads over 20 slots instead of 25: 29.0 and 52.9.
template <int TN> struct GroupSchedule {
    static constexpr TapLayout LY = kLayouts[1];
    static constexpr int kUnits = 24, kHandOver = 20, UNIT = 2 * TN;
    static constexpr int kReadSlots = 2 * UNIT + UNIT / 2, kPermuteUnit = 22;  // from the hand-over on; first unit of the next stage's permutes
    static constexpr int kPermutes = 8 * TN;  // of a phase's operands
    static constexpr int row(int g, int f) { return LY.tap[g][f] / 3; }
    static constexpr int shift(int g, int f) { return LY.tap[g][f] % 3; }
    // unit behind whose first matrix instruction the fragments of unit v are read (before the hand-over, which frees the region)
    static constexpr int fragment_unit(int v) { return v <= kHandOver ? v - 1 : kHandOver - 1 - (v - kHandOver) / 2; }
    // Windows (3 * input row + column shift) in the order in which the rows of the first group need them; the others behind them.
    static constexpr int kWindows = 3 * (TN + 2);
    struct Order {
        int first = 0, what[kWindows] = {};  // first: how many the first group needs
    };
    static constexpr Order make()
    {
        Order o;
        bool seen[kWindows] = {};
        int n = 0;
        for (int j = 0; j < TN; ++j)
            for (int f = 0; f < 4; ++f) {
                const int w = 3 * (j + row(0, f)) + shift(0, f);
                if (!seen[w]) o.what[n++] = w, seen[w] = true;
            }
        o.first = n;
        for (int w = 0; w < kWindows; ++w)
            if (!seen[w]) o.what[n++] = w;
        return o;
    }
    static constexpr Order order = make();
    // The next stage's: reads (windows of the first group in the order above, then the fragments of unit 0) and permutes in front of slot s,
    // counted from the hand-over's instruction.
    static constexpr int kReads = order.first + 2, kNextSlots = (kUnits - kHandOver) * UNIT;
    static constexpr int reads_before(int s) { return s < kReadSlots ? s * kReads / kReadSlots : kReads; }
    static constexpr int kPermuteSlot = (kPermuteUnit - kHandOver) * UNIT;
    static constexpr int permutes_before(int s) { return s < kPermuteSlot ? 0 : (s - kPermuteSlot) * kPermutes / (kNextSlots - kPermuteSlot); }
    static constexpr bool permuted_behind_reads()
    {
        for (int s = 0; s < kNextSlots; ++s)
            for (int o = permutes_before(s); o < permutes_before(s + 1); ++o)
                for (int f = 0; f < 4; ++f)
                    for (int n = reads_before(s); n < order.first; ++n)
                        if (order.what[n] == 3 * (o / 8 + row(0, f)) + shift(0, f)) return false;
        return permutes_before(kNextSlots) == kPermutes && reads_before(kNextSlots) == kReads;
    }
    static_assert(permuted_behind_reads(), "read in an earlier slot");
};

// One pipeline buffer.  Copies past the last (a wave has as many as any other) repeat it.
template <int LAY> struct Region {
    static constexpr int TILE = layout_tile_bytes(kLayouts[LAY]);
    static constexpr int A_BYTES = kRowsTM * TILE;
    static constexpr int A_COPIES = A_BYTES / 1024;  // 64 lanes x 16 bytes each
    static constexpr int X_LEAST = ((4 * kTall + 2) * kLW * 4 + 63) / 64;  // the tall tile's activation tile
    static constexpr int A_PER_WAVE = (A_COPIES + 3) / 4, X_PER_WAVE = (X_LEAST + 3) / 4;
    static constexpr int X_COPIES = 2 * (A_BYTES + X_PER_WAVE * 4096) <= 160 * 1024 ? X_PER_WAVE * 4 : X_LEAST;
    // the copy of a wave's slot
    template <int COPIES> static __device__ __forceinline__ int copy_of(int slot, int wave)
    {
        return COPIES % 4 == 0 ? slot * 4 + wave : min(slot * 4 + wave, COPIES - 1);
    }
    static constexpr int REGION = A_BYTES + X_COPIES * 1024;
    static constexpr int LDS = 2 * REGION;
    static_assert(A_BYTES % 1024 == 0, "weight fragments are whole copy instructions");
    static_assert(LDS <= 160 * 1024, "a compute unit's LDS");
};

// FUSED: scale / bias / SiLU / residual in the epilogue.  The plain instantiation (ReLU or nothing) keeps
// its branch-free epilogue; the fused one pays for generality with a few uniform branches per tile.
// LAY: tap layout (sparse_frag.h)
template <typename T, typename TO, bool FUSED, int LAY>
__global__ __launch_bounds__(256, 1) void conv3x3_rows_kernel(const T* __restrict__ x, TO* __restrict__ y,
                                                              const char* __restrict__ wfrag,
                                                              const char* __restrict__ zeros, int H, int W, int Ci,
                                                              int Co, int m_tiles_total, RowPlan plan, Epilogue ep)
{
    constexpr int TM = kRowsTM;
    using G = Region<LAY>;
    constexpr int TILE = G::TILE, A_BYTES = G::A_BYTES, REGION = G::REGION;  // one pipeline buffer: [weights][activations]
    constexpr int A_PER_WAVE = G::A_PER_WAVE, X_PER_WAVE = G::X_PER_WAVE;
    constexpr int COPY_SLOTS = A_PER_WAVE + X_PER_WAVE;
    static_assert(COPY_SLOTS <= 22, "two copies per unit in the first eleven units of a stage");
    extern __shared__ __attribute__((aligned(16))) char smem[];  // two regions

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int stages = Ci / 32;
    const int Ho = H, Wo = W;  // stride 1, padding 1
    const int64_t a_stage_stride = (int64_t)m_tiles_total * TILE;

    // ---- this workgroup's entries: tall tiles first, then short ones.  Within an XCD the tall list is
    // dealt to the slots in ascending order and the short list in descending order, so that the slots
    // that get one tall tile fewer are the first to get a short one. ----
    const int xcd = blockIdx.x % 8, slot = blockIdx.x / 8, slots = gridDim.x / 8;
    const int tall_end = min((xcd + 1) * plan.tall_per_xcd, plan.tall_total);
    const int short_end = min((xcd + 1) * plan.short_per_xcd, plan.short_total);
    int tall_next = xcd * plan.tall_per_xcd + slot;
    int short_next = xcd * plan.short_per_xcd + (slots - 1 - slot);
    if (tall_next >= tall_end && short_next >= short_end) return;

    // ---- copy state: the tile whose stages are being fetched (runs ahead of the tile being multiplied
    // by one stage at tile boundaries).  Every lane copies 16 bytes in every copy instruction, so the copy
    // code has no branches: a lane whose LDS slot is zero padding of the tile reads from a block of zeros
    // that the packer appended to the weight fragments (2*Ci + 16 bytes, so that the per-stage advance of
    // 64 bytes stays inside it). ----
    int c_mt0 = 0;
    const char* x_ptr[X_PER_WAVE];  // per lane and copy slot: source address for stage 0
    // A lane's source of activation copy slot k for tile t, worked out in four parts (position in the tile;
    // image coordinates and chunk number; address; zero padding).  The first tile does them in one go; after
    // that the last stage of a tile spreads the parts of the next tile's sources over its matrix instructions
    // (as one block in front of a stage they cost ~1.3 k cycles with nothing to overlap them).  The empty asm
    // statements pin each part's results where it is written: they are ordered with the matrix instructions.
    int sp_a = 0, sp_b = 0, sp_off = 0;
    const char* sp_addr = nullptr;
    auto source_part = [&](auto K, auto P, const TileCoord& t, int in_rows) {
        constexpr int k = decltype(K)::value, part = decltype(P)::value;
        if constexpr (part == 0) {
            int l = lane;
            asm volatile("" : "+v"(l));  // recomputed here rather than kept in registers through the K loop
            const int pos = G::template copy_of<G::X_COPIES>(k, wave) * 16 + (l >> 2);
            sp_a = pos / kLW;
            sp_b = pos - sp_a * kLW;
            asm volatile("" : "+v"(sp_a), "+v"(sp_b));
        } else if constexpr (part == 1) {
            sp_a += t.oh0 - 1;  // input row and column
            sp_b += t.ow0 - 1;
            // offset in 16-byte chunks: fits 31 bits (checked by the launcher)
            sp_off = ((t.n_img * H + sp_a) * W + sp_b) * (Ci >> 3) + (lane & 3);
            asm volatile("" : "+v"(sp_a), "+v"(sp_b), "+v"(sp_off));
        } else if constexpr (part == 2) {
            sp_addr = (const char*)x + (int64_t)sp_off * 16;
            asm volatile("" : "+v"(sp_addr));
        } else {
            const int row_end = min(H, t.oh0 - 1 + in_rows);  // rows of the tile, and of the image
            const bool inside = (unsigned)sp_a < (unsigned)row_end && (unsigned)sp_b < (unsigned)W;
            x_ptr[k] = inside ? sp_addr : zeros;
            asm volatile("" : "+v"(x_ptr[k]));
        }
    };
    auto setup_tile_sources = [&](const TileCoord& t, int in_rows) {
        c_mt0 = t.mt0;
        static_for<X_PER_WAVE>([&](auto K) {
            static_for<4>([&](auto P) { source_part(K, P, t, in_rows); });
        });
    };
    // One copy instruction (64 lanes x 16 bytes) of stage `stage` of the copy state's tile into region
    // `par`: slots 0 .. A_PER_WAVE-1 move weight fragments, the rest move activations.
    auto issue_copy_slot = [&](int cslot, int stage, int par) {
        char* region = smem + par * REGION;
        if (cslot < A_PER_WAVE) {
            const int kk = G::template copy_of<G::A_COPIES>(cslot, wave);
            const char* asrc = wfrag + (int64_t)c_mt0 * TILE + lane * 16 + stage * a_stage_stride;
            copy16_to_lds(asrc + kk * 1024, region + kk * 1024);
        } else {
            const int k = cslot - A_PER_WAVE;
            const int kk = G::template copy_of<G::X_COPIES>(k, wave);
            copy16_to_lds(x_ptr[k] + stage * 64, region + A_BYTES + kk * 1024);
        }
    };

    const int nn = lane & 15, qq = lane >> 4;

    f32x4 acc[TM][kTall];
    // Operand registers that cross stage boundaries: what a stage needs before its first matrix
    // instruction is read from inside the previous stage's last unit.
    u32x4 R[kTall + 2][3];
    u32x4 a_nxt[2];
    int g_nxt[2];      // (layouts without a centre: index words of unit 0, and the operands of the first phase)
    u32x8 b_nxt[kTall];
    int gpar = 0;  // region that holds the stage about to be multiplied

    // byte offset in the activation tile of a lane's column (shift 0) of its wave's first input row, for a
    // tile of tn rows per wave
    auto lane_x_offset = [&](int tn) { return ((wave * tn) * kLW + nn) * kPosBytes + qq * 16; };
    // The reads a stage needs before its first matrix instruction: centre-tap operands of its rows, weight
    // fragments of unit 0, side columns of rows 0..3 (corner jobs 0 and 1).  xoff: lane_x_offset of the tile
    // the stage belongs to.  (Rows are read for a tall tile; a short tile has one fewer, and the extra row is
    // inside its activation tile too.)
    auto load_stage_prologue = [&](int par, int xoff) {
        const char* A = smem + par * REGION + lane * 16;
        const char* X = smem + par * REGION + A_BYTES + xoff;
#pragma unroll
        for (int j = 1; j <= kTall; ++j) R[j][1] = *(const u32x4*)(X + (j * kLW + 1) * kPosBytes);
        a_nxt[0] = *(const u32x4*)(A + 4 * kFragBytes);
        a_nxt[1] = *(const u32x4*)(A + TILE + 4 * kFragBytes);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            R[i][0] = *(const u32x4*)(X + (i * kLW + 0) * kPosBytes);
            R[i][2] = *(const u32x4*)(X + (i * kLW + 2) * kPosBytes);
        }
    };

    // ---- one tile of TN rows per wave ----
    auto run_tile = [&](auto tn_tag, const TileCoord& cur, bool has_next, const TileCoord& nxt, bool nxt_tall) {
        constexpr int TN = decltype(tn_tag)::value;
        using Sched = RowSchedule<TN>;
        using Tap = JobTap<TN>;
        constexpr int UNIT = 2 * TN;  // matrix instructions per unit
        const int xrd = lane_x_offset(TN);
        const int nxt_in_rows = nxt_tall ? 4 * kTall + 2 : 4 * kShort + 2;
        auto read_R = [&](const char* X, int i, int kw) {
            R[i][kw] = *(const u32x4*)(X + xrd + (i * kLW + kw) * kPosBytes);
        };

        // The first reads of the tile's first stage.  (Its data landed, and the workgroup met, inside the previous
        // tile's last stage.  That stage also issued reads for "its next stage", but nothing except the stage loop
        // may lie between such reads and their use: across the epilogue the register allocator would park the
        // values and bring them back right in front of the first matrix instructions -- too late for them, see
        // mma.h.  So a tile starts with reads of its own.)
        if constexpr (LAY == 0) load_stage_prologue(gpar, xrd);

        auto run_stage = [&](auto first_tag, auto last_tag, int stage) {
            constexpr bool FIRST = decltype(first_tag)::value, LAST = decltype(last_tag)::value;
            // the stage copied while this one is multiplied: the tile's next stage, or the next tile's first
            // (in the very last stage of the last tile there is nothing left to fetch; `nxt` is the same
            // tile then and its stage 0 is fetched again into the free region, which keeps this code free of
            // branches).  The last stage works out the next tile's activation sources as it goes: slot k in
            // unit k, before the unit (>= 5) that issues the slot's copy.
            const int copy_stage = LAST ? 0 : stage + 1;
            if constexpr (LAST) c_mt0 = nxt.mt0;
            const char* A = smem + gpar * REGION + lane * 16;
            const char* AI = smem + gpar * REGION + 5 * kFragBytes + lane * 4;
            const char* X = smem + gpar * REGION + A_BYTES;

            // output o (0..15) of a job: dword o%8 of step o/8; element 4*c + f of a step's B operand =
            // channel c (of this lane's 4 in that step), tap slot f
            auto transposed = [&](auto Q, int o) -> uint32_t {
                constexpr int q = decltype(Q)::value;
                const int d = o & 7, comp = (o >> 3) * 2 + (d >> 2);
                const uint32_t sel = (d & 2) ? 0x07060302u : 0x05040100u;
                return (d & 1) ? __builtin_amdgcn_perm(R[Tap::row(q, 3)][Tap::shift(q, 3)][comp],
                                                       R[Tap::row(q, 2)][Tap::shift(q, 2)][comp], sel)
                               : __builtin_amdgcn_perm(R[Tap::row(q, 1)][Tap::shift(q, 1)][comp],
                                                       R[Tap::row(q, 0)][Tap::shift(q, 0)][comp], sel);
            };
            u32x8 bfc[2][TN], bfe[2][TN];  // B operands of the sparse phases
            u32x4 a_cur[2] = {a_nxt[0], a_nxt[1]};
            int i_cur[2] = {0, 0}, i_nxt[2] = {0, 0};
            static_for<20>([&](auto U) {
                constexpr int u = decltype(U)::value;
                constexpr int phase = u / 4, m0 = (u % 4) * 2;
                constexpr int perm_first = Sched::perm_first(u), perm_count = Sched::perm_count(u);
                static_for<UNIT>([&](auto I) {
                    constexpr int i = decltype(I)::value;
                    constexpr int mi = i / TN, j = i % TN, m = m0 + mi;
                    if constexpr (phase == 0) {
                        if constexpr (FIRST) Mat<T>::dense_first(a_cur[mi], R[j + 1][1], acc[m][j]);
                        else Mat<T>::dense(a_cur[mi], R[j + 1][1], acc[m][j]);
                    }
                    if constexpr (phase == 1) Mat<T>::template sparse<0>(a_cur[mi], bfc[0][j], acc[m][j], i_cur[mi]);
                    if constexpr (phase == 2) Mat<T>::template sparse<1>(a_cur[mi], bfc[1][j], acc[m][j], i_cur[mi]);
                    if constexpr (phase == 3) Mat<T>::template sparse<0>(a_cur[mi], bfe[0][j], acc[m][j], i_cur[mi]);
                    if constexpr (phase == 4) Mat<T>::template sparse<1>(a_cur[mi], bfe[1][j], acc[m][j], i_cur[mi]);
                    if constexpr (LAST && u < X_PER_WAVE) {
                        constexpr int part = i == 1 ? 0 : i == 3 ? 1 : i == 4 ? 2 : i == 5 ? 3 : -1;
                        if constexpr (part >= 0)
                            source_part(std::integral_constant<int, u>{}, std::integral_constant<int, part>{}, nxt, nxt_in_rows);
                    }
                    if constexpr (i == 2 && 2 * u < COPY_SLOTS) issue_copy_slot(2 * u, copy_stage, gpar ^ 1);
                    if constexpr (i == 2 + TN && 2 * u + 1 < COPY_SLOTS) issue_copy_slot(2 * u + 1, copy_stage, gpar ^ 1);
                    if constexpr (i == 0) {  // issue the next unit's LDS reads behind the first matrix instruction
                        if constexpr (u + 1 < 20) {
                            constexpr int np = (u + 1) / 4, nm0 = ((u + 1) % 4) * 2;
                            constexpr int nstep = np == 0 ? 4 : np - 1;
#pragma unroll
                            for (int t = 0; t < 2; ++t) {
                                a_nxt[t] = *(const u32x4*)(A + (nm0 + t) * TILE + nstep * kFragBytes);
                                if constexpr (np > 0) i_nxt[t] = *(const int*)(AI + (nm0 + t) * TILE + ((np - 1) >> 1) * 256);
                            }
                        }
                        if constexpr (Sched::side_row(u) >= 0) {
                            read_R(X, Sched::side_row(u), 0);
                            read_R(X, Sched::side_row(u), 2);
                        }
                        if constexpr (Sched::reads_outer_mid(u)) {
                            read_R(X, 0, 1);
                            read_R(X, TN + 1, 1);
                        }
                        if constexpr (u == 19) {
                            // Stage hand-over without a bubble: all copies of the next stage were issued in
                            // this stage's first ten units and this unit's operands were read in unit 18; the
                            // wave waits for its copies and its reads, meets the others at a bare barrier (the
                            // next stage's data is now complete and nobody reads this stage's region any more)
                            // and issues the next stage's first reads (below), which complete under the rest of this unit.
                            asm volatile("" ::: "memory");
                            __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0): copies landed, reads of this region done
                            __builtin_amdgcn_s_barrier();
                            asm volatile("" ::: "memory");
                        }
                    }
                    if constexpr (u == 19) {
                        // The next stage's first reads (load_stage_prologue), one or two behind each instruction.  All behind the first they kept
                        // the matrix pipe waiting for their issue: 256 -> 256 on 4x100x168 42.5 us, now 41.6, on 2x100x168 22.5, 22.2.
                        constexpr int kReads = 2 + kTall + 8, first = i * kReads / UNIT;
                        const char* const nA = smem + (gpar ^ 1) * REGION + lane * 16;
                        const char* const nX = smem + (gpar ^ 1) * REGION + A_BYTES + xrd;
                        static_for<(i + 1) * kReads / UNIT - first>([&](auto k_tag) {
                            constexpr int n = first + decltype(k_tag)::value, centre = n - 1, side = n - 2 - kTall;
                            if constexpr (n < 2) a_nxt[n] = *(const u32x4*)(nA + n * TILE + 4 * kFragBytes);
                            else if constexpr (side < 0) R[centre][1] = *(const u32x4*)(nX + (centre * kLW + 1) * kPosBytes);
                            else R[side / 2][side % 2 * 2] = *(const u32x4*)(nX + (side / 2 * kLW + side % 2 * 2) * kPosBytes);
                        });
                    }
                    // this instruction's share of the unit's 16 * perm_count permutes
                    constexpr int o_begin = i * 16 * perm_count / UNIT, o_end = (i + 1) * 16 * perm_count / UNIT;
                    static_for<o_end - o_begin>([&](auto O) {
                        constexpr int o = o_begin + decltype(O)::value;
                        constexpr int q = perm_first + o / 16, oo = o % 16;
                        const uint32_t v = transposed(std::integral_constant<int, q>{}, oo);
                        if constexpr (q < TN) bfc[oo >> 3][q][oo & 7] = v;
                        else bfe[oo >> 3][q - TN][oo & 7] = v;
                    });
                    __builtin_amdgcn_sched_barrier(0);
                });
                if constexpr (u + 1 < 20) {
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        a_cur[t] = a_nxt[t];
                        i_cur[t] = i_nxt[t];
                    }
                }
            });
            gpar = __builtin_amdgcn_readfirstlane(gpar ^ 1);  // (kept scalar: it feeds the LDS address of every copy)
        };
        // ---- a stage of a layout of groups (GroupSchedule) ----
        using Q = GroupSchedule<TN>;
        // window w and permute o (0..8*TN-1) of half `half` of a group's operands: dword o%8 of row o/8's, as sparse_operand
        auto read_window = [&](const char* X, int w) { R[w / 3][w % 3] = *(const u32x4*)(X + xrd + (w / 3 * kLW + w % 3) * kPosBytes); };
        auto permuted = [&](auto g_tag, int half, int o) -> uint32_t {
            constexpr int g = decltype(g_tag)::value;
            const int j = o / 8, d = o % 8, comp = 2 * half + d / 4, f = d % 2 * 2;
            return __builtin_amdgcn_perm(R[j + Q::row(g, f + 1)][Q::shift(g, f + 1)][comp], R[j + Q::row(g, f)][Q::shift(g, f)][comp],
                                         d & 2 ? 0x07060302u : 0x05040100u);
        };
        auto read_first = [&](const char* region, auto n_tag) {  // what a stage needs at its start, in turn
            constexpr int n = decltype(n_tag)::value;
            if constexpr (n < Q::order.first) {
                read_window(region + A_BYTES, Q::order.what[n]);
            } else {
                constexpr int t = n - Q::order.first;
                a_nxt[t] = *(const u32x4*)(region + lane * 16 + t * TILE);
                g_nxt[t] = *(const int*)(region + lane * 4 + t * TILE + 6 * kFragBytes);
            }
        };
        auto run_group_stage = [&](auto last_tag, int stage) {
            constexpr bool LAST = decltype(last_tag)::value;
            const int copy_stage = LAST ? 0 : stage + 1;
            if constexpr (LAST) c_mt0 = nxt.mt0;
            const char* const region = smem + gpar * REGION;
            u32x4 a[Q::kUnits][2];
            int idx[3][TM];
            u32x8 b[6][TN];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                a[0][t] = a_nxt[t];
                idx[0][t] = g_nxt[t];
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) b[0][j] = b_nxt[j];
            static_for<Q::kUnits>([&](auto U) {
                constexpr int u = decltype(U)::value, p = u / 4, m0 = u % 4 * 2;
                static_for<UNIT>([&](auto I) {
                    constexpr int i = decltype(I)::value, mi = i / TN, j = i % TN;
                    Mat<T>::template sparse<p % 2>(a[u][mi], b[p][j], acc[m0 + mi][j], idx[p / 2][m0 + mi]);
                    if constexpr (LAST && u < X_PER_WAVE) {
                        constexpr int part = i == 1 ? 0 : i == 3 ? 1 : i == 4 ? 2 : i == 5 ? 3 : -1;
                        if constexpr (part >= 0)
                            source_part(std::integral_constant<int, u>{}, std::integral_constant<int, part>{}, nxt, nxt_in_rows);
                    }
                    if constexpr (i == 2 && 2 * u < COPY_SLOTS) issue_copy_slot(2 * u, copy_stage, gpar ^ 1);
                    if constexpr (i == 2 + TN && 2 * u + 1 < COPY_SLOTS) issue_copy_slot(2 * u + 1, copy_stage, gpar ^ 1);
                    if constexpr (i == 0) {
                        static_for<Q::kUnits>([&](auto V) {
                            constexpr int v = decltype(V)::value, vp = v / 4, vm = v % 4 * 2;
                            if constexpr (v > 0 && Q::fragment_unit(v) == u) {
#pragma unroll
                                for (int t = 0; t < 2; ++t) {
                                    a[v][t] = *(const u32x4*)(region + lane * 16 + (vm + t) * TILE + vp * kFragBytes);
                                    if constexpr (vp % 2 == 0)
                                        idx[vp / 2][vm + t] = *(const int*)(region + lane * 4 + (vm + t) * TILE + 6 * kFragBytes + vp / 2 * 256);
                                }
                            }
                        });
                        if constexpr (u == 0)
                            static_for<Q::kWindows - Q::order.first>([&](auto n) { read_window(region + A_BYTES, Q::order.what[Q::order.first + n]); });
                        if constexpr (u == Q::kHandOver) {
                            asm volatile("" ::: "memory");
                            __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0): copies landed, reads of this region done
                            __builtin_amdgcn_s_barrier();
                            asm volatile("" ::: "memory");
                        }
                    }
                    // (a tile starts with reads of its own: see above)
                    if constexpr (!LAST && u >= Q::kHandOver) {
                        constexpr int n = (u - Q::kHandOver) * UNIT + i, r = Q::reads_before(n), o = Q::permutes_before(n);
                        static_for<Q::reads_before(n + 1) - r>(
                            [&](auto k) { read_first(smem + (gpar ^ 1) * REGION, std::integral_constant<int, r + decltype(k)::value>{}); });
                        static_for<Q::permutes_before(n + 1) - o>([&](auto k) {
                            constexpr int e = o + decltype(k)::value;
                            b_nxt[e / 8][e % 8] = permuted(std::integral_constant<int, 0>{}, 0, e);
                        });
                    }
                    if constexpr (p < 5) {
                        constexpr int o = (u % 4) * UNIT + i;
                        b[p + 1][o / 8][o % 8] = permuted(std::integral_constant<int, (p + 1) / 2>{}, (p + 1) % 2, o);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
            });
            gpar = __builtin_amdgcn_readfirstlane(gpar ^ 1);
        };
        if constexpr (LAY == 0) {
            run_stage(std::true_type{}, std::false_type{}, 0);  // (the launcher admits Ci >= 96: three stages or more)
            for (int stage = 1; stage + 1 < stages; ++stage) run_stage(std::false_type{}, std::false_type{}, stage);
            run_stage(std::false_type{}, std::true_type{}, stages - 1);
        } else {
            // the accumulators are cleared by products of zeros (640 cycles; see mma.h) under the first reads
            static_for<Q::kReads>([&](auto n) { read_first(smem + gpar * REGION, n); });
            u32x4 nothing = {0, 0, 0, 0};
            asm volatile("" : "+v"(nothing));
            static_for<TM>([&](auto m) { static_for<TN>([&](auto j) { Mat<T>::dense_first(nothing, nothing, acc[m][j]); }); });
            static_for<Q::kPermutes>([&](auto o) { b_nxt[o / 8][o % 8] = permuted(std::integral_constant<int, 0>{}, 0, o); });
            for (int stage = 0; stage + 1 < stages; ++stage) run_group_stage(std::false_type{}, stage);
            run_group_stage(std::true_type{}, stages - 1);
        }

        // the last matrix instructions must have written their accumulators before anything reads them
        asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
        // ---- epilogue ----
        // Per lane and group of 4 channel tiles the accumulators hold 16 consecutive output channels of one
        // position (tile_row_channel): column nn of row j of the wave.  16-bit outputs without a fused output
        // stage leave in rows of 128 bytes past the L2's write-back (RowTile).  Otherwise each wave transposes its
        // 16*TN positions x 16*TM channels through its own slice of the region that was multiplied last
        // (free now; the other region is receiving the next tile's first stage) and writes whole
        // channel rows, 16 bytes per lane; fp32 output goes in two halves of the channel tiles.
        {
            constexpr int EB = (int)sizeof(TO);
            constexpr int HALVES = EB == 4 ? 2 : 1;
            constexpr int TMH = TM / HALVES;
            static_assert(TM % HALVES == 0 && TMH % 4 == 0, "each half is whole groups of 4 channel tiles (tile_row_channel)");
            constexpr int ROW = TMH * 16 * EB + (EB == 2 ? 8 : 16);  // padded row pitch: spreads the banks
            // output rows staged together: as many as fit when the four waves share one region
            constexpr int JG = (REGION / (4 * 16 * ROW)) < TN ? (REGION / (4 * 16 * ROW)) : TN;
            static_assert(JG >= 1, "epilogue staging must fit in one region");
            char* stage_out = smem + (gpar ^ 1) * REGION + wave * (16 * JG * ROW);
            // lane-derived addresses of the epilogue are recomputed per tile (opaque copy of the lane id)
            // instead of staying live in registers through the K loop
            int lane_e = lane;
            asm volatile("" : "+v"(lane_e));
            const int nn_e = lane_e & 15, qq_e = lane_e >> 4;
            const int row_first = cur.oh0 + wave * TN;  // first output row of the wave
            // (positions within a tile count in 32 bits, elements in 64: a channel slice's pitch may be millions)
            const int64_t pos_tile = ((int64_t)cur.n_img * Ho + cur.oh0) * Wo + cur.ow0;  // position number
            TO* const y_tile = y + pos_tile * ep.ldy;
            const float relu_floor = ep.act == 1 ? 0.f : -__builtin_inff();
            if constexpr (EB == 2 && !FUSED) {
                // (four tiles of a wave in turn, two on their way: 256 -> 256 on 4x100x168 45.5 -> 44.0 us, on 2x100x168 25.4 -> 23.6,
                // 192 -> 128 on 8x80x80 17.9 -> 16.7, against 32 bytes a lane from the accumulators, written back when the launch ends)
                char* const area = smem + (gpar ^ 1) * REGION + wave * (4 * RowTile<TO>::kBytes);
                auto flush = [&](auto t_tag) {
                    constexpr int t = decltype(t_tag)::value, j = t / (TM / 4), mg = t % (TM / 4) * 4;
                    if (row_first + j >= Ho) return;
                    const auto base = store_base(y_tile + (int64_t)((wave * TN + j) * Wo) * ep.ldy + 16 * (cur.mt0 + mg));
                    RowTile<TO>::store(area + t % 4 * RowTile<TO>::kBytes, lane_e, base, [&](int row, int c) {
                        return cur.ow0 + row < Wo && 16 * (cur.mt0 + mg) + 8 * c < Co ? (uint32_t)row * ep.ldy * 2 + c * 16 : kNoStore;
                    });
                };
                static_for<TN * (TM / 4)>([&](auto t_tag) {
                    constexpr int t = decltype(t_tag)::value, j = t / (TM / 4), mg = t % (TM / 4) * 4;
                    uint32_t o[8];
#pragma unroll
                    for (int m = 0; m < 4; ++m) {
                        float r[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) asm("v_max_f32 %0, %1, %2" : "=v"(r[e]) : "v"(acc[mg + m][j][e]), "v"(relu_floor));
                        o[2 * m] = pack2_from_f32<TO>(r[0], r[1]);
                        o[2 * m + 1] = pack2_from_f32<TO>(r[2], r[3]);
                    }
                    RowTile<TO>::put(area + t % 4 * RowTile<TO>::kBytes, lane_e, u32x4{o[0], o[1], o[2], o[3]}, u32x4{o[4], o[5], o[6], o[7]});
                    if constexpr (t >= 2) flush(std::integral_constant<int, t - 2>{});
                });
                flush(std::integral_constant<int, TN * (TM / 4) - 2>{});
                flush(std::integral_constant<int, TN * (TM / 4) - 1>{});
            } else {
                // (loops over types: a pragma gives up on bodies of this size, and the accumulators would go to memory)
                static_for<HALVES>([&](auto h_tag) {
                    constexpr int h = decltype(h_tag)::value;
                    static_for<(TN + JG - 1) / JG>([&](auto g_tag) {
                        constexpr int j0 = decltype(g_tag)::value * JG;
                        constexpr int jn = j0 + JG <= TN ? JG : TN - j0;  // rows in this group
                        static_for<jn>([&](auto jj_tag) {
                            constexpr int jj = decltype(jj_tag)::value, j = j0 + jj;
                            f32x4 vals[TMH];
#pragma unroll
                            for (int mm = 0; mm < TMH; ++mm) vals[mm] = acc[h * TMH + mm][j];
                            if constexpr (FUSED) {
                                // this lane's position in row j and its 4 consecutive channels of every channel tile
                                const int dr_f = wave * TN + j;
                                const bool inside_f = cur.oh0 + dr_f < Ho && cur.ow0 + nn_e < Wo;
                                const int64_t pos_f = pos_tile + dr_f * Wo + nn_e;
#pragma unroll
                                for (int mm = 0; mm < TMH; ++mm) {
                                    const int co4 = 16 * (cur.mt0 + h * TMH) + tile_quarter_offset(mm, qq_e);
                                    if (inside_f && co4 < Co) {
                                        float vv[4] = {vals[mm].x, vals[mm].y, vals[mm].z, vals[mm].w};
                                        epi_scale_bias_act<4>(vv, ep, co4);
                                        epi_residual<TO, 4>(vv, ep, pos_f, co4);
                                        vals[mm] = f32x4{vv[0], vv[1], vv[2], vv[3]};
                                    }
                                }
                            } else {
                                // fused ReLU without a branch: max with 0, or with -inf when ReLU is off (one v_max_f32
                                // per value, written as asm so that no NaN-quieting pass is put in front of it)
#pragma unroll
                                for (int mm = 0; mm < TMH; ++mm)
#pragma unroll
                                    for (int e = 0; e < 4; ++e) {
                                        float r;
                                        asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(vals[mm][e]), "v"(relu_floor));
                                        vals[mm][e] = r;
                                    }
                            }
#pragma unroll
                            for (int mm = 0; mm < TMH; ++mm) {
                                char* dst = stage_out + (jj * 16 + nn_e) * ROW + tile_quarter_offset(mm, qq_e) * EB;
                                if constexpr (EB == 4) {
                                    *(f32x4*)dst = vals[mm];
                                } else {
                                    uint2 o;
                                    o.x = pack2_from_f32<TO>(vals[mm].x, vals[mm].y);
                                    o.y = pack2_from_f32<TO>(vals[mm].z, vals[mm].w);
                                    *(uint2*)dst = o;
                                }
                            }
                        });
                        // read back: a row of 16*TMH channels is CH 16-byte chunks; 64 lanes cover 64/CH positions
                        // per pass.  (A wave's LDS accesses execute in order, so the next group's writes to this
                        // slice cannot pass these reads.)
                        constexpr int CH = TMH * 16 * EB / 16;
                        static_assert(64 % CH == 0, "row chunks must tile the wave");
                        constexpr int POS_PER_PASS = 64 / CH;
                        constexpr int passes = (16 * jn) / POS_PER_PASS;
                        const int co_first = 16 * (cur.mt0 + h * TMH);
                        const int sub = lane_e / CH, chunk = lane_e % CH;  // position within the pass, chunk within the row
                        const int co = co_first + chunk * (16 / EB);
#pragma unroll
                        for (int ps = 0; ps < passes; ++ps) {
                            const int p = ps * POS_PER_PASS + sub;
                            const int dr = wave * TN + j0 + (p >> 4), dc = p & 15;
                            const u32x4 v = *(const u32x4*)(stage_out + p * ROW + chunk * 16);
                            if (cur.oh0 + dr < Ho && cur.ow0 + dc < Wo && co < Co)  // Co is a multiple of 16: a chunk is all in or all out
                                *(u32x4*)(y_tile + (int64_t)(dr * Wo + dc) * ep.ldy + co) = v;
                        }
                    });
                });
            }
        }
        // staging slices are read (LDS only): the region may be overwritten by the next copies.  A bare
        // barrier, because __syncthreads() carries a fence that would wait here for this tile's output
        // stores to drain; they drain behind the next tile's first stage instead.
        {
            if (has_next) {
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0) only
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            }
        }
    };

    // ---- walk the entries ----
    bool cur_tall = tall_next < tall_end;
    TileCoord cur = decode_entry(plan, cur_tall, cur_tall ? tall_next : short_next);
    if (cur_tall) tall_next += slots;
    else short_next += slots;
    // (the weight copies need only the tile's channel block: they are under way while the lanes work out
    // their activation sources, ~3 k cycles of address arithmetic)
    c_mt0 = cur.mt0;
#pragma unroll
    for (int s = 0; s < A_PER_WAVE; ++s) issue_copy_slot(s, 0, 0);
    setup_tile_sources(cur, cur_tall ? 4 * kTall + 2 : 4 * kShort + 2);
#pragma unroll
    for (int s = A_PER_WAVE; s < COPY_SLOTS; ++s) issue_copy_slot(s, 0, 0);
    bool first_tile = true;
    for (;;) {
        const bool nxt_tall = tall_next < tall_end;
        const bool has_next = nxt_tall || short_next < short_end;
        TileCoord nxt = cur;
        if (has_next) {
            nxt = decode_entry(plan, nxt_tall, nxt_tall ? tall_next : short_next);
            if (nxt_tall) tall_next += slots;
            else short_next += slots;
        }
        if (first_tile) {
            __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this wave's copies have landed in LDS
            __syncthreads();                     // ... and everybody's
            first_tile = false;
        }
        if (cur_tall) run_tile(std::integral_constant<int, kTall>{}, cur, has_next, nxt, nxt_tall);
        else run_tile(std::integral_constant<int, kShort>{}, cur, has_next, nxt, nxt_tall);
        if (!has_next) break;
        cur = nxt;
        cur_tall = nxt_tall;
    }
}

template <typename T, typename TO, bool FUSED, int LAY>
rtoss_status launch_rows(const rtoss_wdesc& d, const ConvParams& c, const RowsLaunch* planned, const char* wfrag, const void* x, void* y, hipStream_t s)
{
    const size_t smem = Region<LAY>::LDS;
    auto kern = conv3x3_rows_kernel<T, TO, FUSED, LAY>;
    static LaunchOnce lds_once;  // per instantiation
    if (rtoss_status st = ensure_dynamic_lds((const void*)kern, smem, lds_once, c.dev.device, "conv3x3 shared memory attribute")) return st;
    const DeviceInfo& dev = c.dev;
    const int co_blocks = ((d.Co + 15) / 16 + kRowsTM - 1) / kRowsTM;
    if (c.stride != 1 || d.Ci % 32 || d.Ci < 96) return fail(RTOSS_ESHAPE, "conv: the pipelined kernel needs stride 1 and three or more stages of 32 input channels");
    if ((int64_t)c.N * c.H * c.W * d.Ci / 8 > 0x7fffffff) return fail(RTOSS_ESHAPE, "conv: input too large for 32-bit chunk offsets");
    if ((int64_t)c.N * ((c.W + 15) / 16) * ((c.H + 15) / 16 + 1) * co_blocks > 0x3fffffff) return fail(RTOSS_ESHAPE, "conv: too many tiles");
    const RowsLaunch launch = planned ? *planned : plan_rows_for_device(c.N, c.H, c.W, d.Co, d.Ci / 32, dev.cus);
    dim3 grid((unsigned)(launch.slots * 8)), block(256);
    kern<<<grid, block, smem, s>>>((const T*)x, (TO*)y, wfrag, wfrag + fragment_bytes(d, LAY), c.H, c.W, d.Ci, d.Co,
                                   padded_m_tiles(d.Co), launch.plan, c.ep);
    return check_hip(hipGetLastError(), "conv3x3 rows launch");
}

template <int LAY>
rtoss_status launch_rows_typed(const rtoss_wdesc& d, const ConvParams& c, const RowsLaunch* planned, const void* section, const void* x, void* y, hipStream_t s)
{
    const char* wf = (const char*)section;
    const bool f32out = c.out_dt == RTOSS_F32;
    const bool fused = rows3x3_needs_fused_stage(c);
#define RTOSS_ROWS(T, TO) (fused ? launch_rows<T, TO, true, LAY>(d, c, planned, wf, x, y, s) : launch_rows<T, TO, false, LAY>(d, c, planned, wf, x, y, s))
    if (d.dt == RTOSS_F16) return f32out ? RTOSS_ROWS(f16_t, float) : RTOSS_ROWS(f16_t, f16_t);
    return f32out ? RTOSS_ROWS(bf16_t, float) : RTOSS_ROWS(bf16_t, bf16_t);
#undef RTOSS_ROWS
}

}  // namespace

}  // namespace rtoss
