// Packing: prune (Section II.B mask semantics: survivors keep their value, the rest are dropped; Section IV.D: the tail
// of a flattened 1x1 tensor is dropped) and write the packed blobs of any number of layers in one launch.
//
// A blob is the public section (k survivors and the pattern index of every group) and a private one: weight fragments
// in the order one of the convolution kernels reads them (formats: pack_plan.h, sparse_frag.h).  All formats of one
// dtype share this kernel, so a model is packed by one launch: the layers are small (0.1-1 MB) and a launch per format,
// or per 24 layers, left the chip idle between them.
//
// What bounds it: latency (index -> mask -> weight are dependent loads), then HBM.  So nothing is gathered from memory:
//   * 3x3 fragments: a workgroup owns one (stage of input channels, tile of 16 output channels).  Its kernels are 16
//     rows of 576 contiguous bytes; they and their indices are staged in LDS with 16-byte loads, and both the public
//     section's part and the fragments are assembled from there.  Every weight is read once.
//   * 1x1 fragments: a lane's 16 bytes are consecutive elements of one row of [Co][Ci], which touch at most two groups:
//     one vector load and two index loads, all independent.
//   * public sections of 1x1 layers: runs of 256 groups through LDS (pack_live.h).
//   * workgroups of the 1x1 formats do several runs or pieces each, and the 3x3 tiles, which take longest, come first.
// Measured, 57 layers with 7.0 M fp16 weights, 2-entry patterns: 10.3 us in one launch (13.1 with a workgroup per run, in the order
// of the layers; 38 in four launches).  A workgroup of the 3x3 path takes 10 000 cycles, 2000 of them for the launch arguments, 2000
// for weights and indices, 1800 for its part of the public section and 3300 for the fragments.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "dtypes.h"
#include "mma.h"
#include "pack_live.h"
#include "pack_plan.h"
#include "sparse_frag.h"

namespace rtoss {

namespace {

// One layer of a launch.  Kept small: the table travels in the launch arguments (4 KB).
struct PackEntry {
    const void* w;
    const uint8_t* idx;
    char* blob;
    uint32_t idx_off, mat_off;  // sections of the blob, in units of 256 bytes
    int Co, Ci;
    uint32_t items;             // 3x3: (stage, channel tile) pairs; 1x1 and stem: 16-byte pieces of the fragments
    uint8_t format, a, b, c;    // MatrixFormat; 3x3: tap layout, fragments alone, repeated taps needed; streaming 1x1: log2 of KS, of MT; without fragments (c): weights per kernel
};
constexpr int kPackMax = 60, kPackFew = 8;
template <int N> struct PackTable {
    PackEntry e[N];
    int first_block[N];
};
static_assert(sizeof(PackTable<kPackMax>) + sizeof(Dict) <= 4096, "launch arguments");
constexpr int kOneWave = 64;  // patterns from which on the per-pattern tables take all waves of a workgroup
// The dictionary of a launch, by size.  (A launch with few layers and patterns writes 0.6 KB of arguments instead of 3.7, which takes
// the host 1.3 us less.)
struct SmallDict {
    uint16_t mask[kOneWave];  // (entries past the last pattern: 0)
    int k;
};

// Input channel (within a 32-channel stage) that pair g of lane-quarter q refers to in sparse step `half`.
__device__ __forceinline__ int stage_channel(int q, int g, int half)
{
    return 8 * (2 * (q & 1) + (g >> 1)) + 4 * half + 2 * (q >> 1) + (g & 1);
}

constexpr int kTapGroups = 3;  // at most (TapLayout::tap)

// 16-byte pieces of a 1x1 section that a lane writes, and runs of 256 groups of a public section that a workgroup does: what a
// workgroup spends to find its layer is as much as one of either.
constexpr int kPieces = 4, kLiveRuns = 2;

// Fragments and survivors are stored past the L2's write-back, which would otherwise end the launch (57 layers, selection included,
// replayed from a graph 19.6 -> 18.4 us; calls from the host, whose time they hide behind, 15.6 us either way).

// LDS of a workgroup
template <typename T> struct TileLds {
    static constexpr int SC = 64 / (int)sizeof(T);  // channels of a stage
    __attribute__((aligned(16))) T w[16][SC * 9];   // [row][channel][tap]
    uint8_t idx[16][SC];
    uint64_t taps[256];                             // 4 bits per live tap of a pattern, ascending; 15: none
    uint16_t slots[256 * kTapGroups];
};

// (stage, tile) of a 3x3 layer: public section and fragments
// (LAY: tap layout, or kDenseTaps; a template parameter so that the walks over a layout's taps are constants)
constexpr int kDenseTaps = kNumLayouts;
template <typename T, int LAY, bool SMALL>
__device__ __forceinline__ void pack_tile3x3(const PackEntry& en, int k, unsigned mask, const uint16_t* masks, int tile,
                                             int m_tiles, TileLds<T>& L)
{
    constexpr int SC = TileLds<T>::SC;
    const T* __restrict__ w = (const T*)en.w;
    const uint8_t* __restrict__ idx = en.idx;
    constexpr bool SPARSE = LAY != kDenseTaps;
    constexpr TapLayout lay = kLayouts[SPARSE ? LAY : 0];
    const int Co = en.Co, Ci = en.Ci, tid = threadIdx.x;
    const int mt = tile % m_tiles, stage = tile / m_tiles;
    const int channels = min(SC, Ci - SC * stage);
    // ---- stage weights and indices (rows past Co and channels past Ci: zeros), all of a lane's loads in flight ----
    constexpr int IDX_PER = 16 * SC / 256;
    uint8_t iv[IDX_PER];
#pragma unroll
    for (int i = 0; i < IDX_PER; ++i) {
        const int c = tid + 256 * i, r = c / SC, e = c % SC, co = tile_row_channel(mt, r);
        iv[i] = co < Co && e < channels ? idx[(int64_t)co * Ci + SC * stage + e] : (uint8_t)0;
    }
    if (Ci % SC == 0 && (reinterpret_cast<uintptr_t>(w) & 15) == 0) {
        u32x4 v[3];  // 16 rows x 36 vectors
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int c = tid + 256 * i, r = c / 36, q = c % 36, co = tile_row_channel(mt, r);
            v[i] = u32x4{0, 0, 0, 0};
            if (c < 16 * 36 && co < Co) v[i] = *(const u32x4*)((const char*)w + ((int64_t)co * Ci + SC * stage) * (9 * (int)sizeof(T)) + q * 16);
        }
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int c = tid + 256 * i, r = c / 36, q = c % 36;
            if (c < 16 * 36) *(u32x4*)((char*)&L.w[r][0] + q * 16) = v[i];
        }
    } else {  // (the interface asks for element alignment only)
#pragma unroll 6
        for (int c = tid; c < 16 * SC * 9; c += 256) {
            const int r = c / (SC * 9), e = c % (SC * 9), co = tile_row_channel(mt, r);
            T v;
            __builtin_memset(&v, 0, sizeof(T));
            if (co < Co && e < 9 * channels) v = w[((int64_t)co * Ci + SC * stage) * 9 + e];
            L.w[r][e] = v;
        }
    }
    uint8_t entry[IDX_PER];  // of the per-pattern tables: an index outside the dictionary finds an entry without taps
#pragma unroll
    for (int i = 0; i < IDX_PER; ++i) {
        entry[i] = SMALL ? (uint8_t)min((int)iv[i], kOneWave - 1) : iv[i];
        L.idx[(tid + 256 * i) / SC][(tid + 256 * i) % SC] = entry[i];
    }
    // ---- per-pattern tables (under the loads above); a small dictionary (one entry at least without a pattern): one wave, not the first, which has
    // a fragment more than the others ----
    const bool tables = !SMALL || tid >= 192;  // (uniform over a wave)
    const int pattern = SMALL ? tid & (kOneWave - 1) : tid;
    if (tables) {
        uint64_t t = ~(uint64_t)0;
        unsigned m = mask;
        for (int j = 0; m; ++j, m &= m - 1) t = (t & ~((uint64_t)15 << (4 * j))) | (uint64_t)__builtin_ctz(m) << (4 * j);
        L.taps[pattern] = t;
    }
    // slots[p][group]: taps of pattern p's first and second live tap in the group (bits 0-3, 4-7; 15: none) and the
    // slots they take (bits 8-9, 10-11; a missing second value points at the slot after the first, a group without
    // live taps at slots 0 and 1: padding values of 0 may point anywhere, as long as the two differ)
    constexpr unsigned kNoTaps = 15u | (15u << 4) | (0u << 8) | (1u << 10);
    if (SPARSE && tables) {
        unsigned taken[kTapGroups];  // taps of every group, by the pattern's choice (tap_choice)
        static_for<lay.groups>([&](auto g) { taken[g] = group_taps(lay, g, 0); });
        if (lay.repeats && en.c) {  // (a dictionary that does not need them skips the search: four layers 256 -> 256, 4 entries, 6.35 -> 6.0 us)
            static_for<kTapChoices>([&](auto n) {
                constexpr int c = kTapChoices - 1 - n;
                bool fits = true;
                static_for<lay.groups>([&](auto g) { fits = fits && __builtin_popcount(mask & group_taps(lay, g, c)) <= 2; });
                static_for<lay.groups>([&](auto g) { taken[g] = fits ? group_taps(lay, g, c) : taken[g]; });
            });
        }
        static_for<lay.groups>([&](auto g_tag) {
            constexpr int g = decltype(g_tag)::value;
            constexpr unsigned taps = (unsigned)lay.tap[g][0] | (unsigned)lay.tap[g][1] << 4 | (unsigned)lay.tap[g][2] << 8 | (unsigned)lay.tap[g][3] << 12;
            unsigned live = 0;  // slots
            static_for<4>([&](auto sl) { live |= ((mask & taken[g]) >> (unsigned)lay.tap[g][sl] & 1u) << sl; });
            const unsigned second = live & (live - 1);
            const unsigned f0 = live ? __builtin_ctz(live) : 0u, f1 = second ? __builtin_ctz(second) : (f0 + 1) & 3;
            const unsigned t0 = live ? taps >> (4 * f0) & 15u : 15u, t1 = second ? taps >> (4 * f1) & 15u : 15u;
            L.slots[pattern * kTapGroups + g] = (uint16_t)(t0 | (t1 << 4) | (f0 << 8) | (f1 << 10));
        });
    }
    __syncthreads();
    // ---- public section: rows of 32 (or 16) groups, k values and an index each ----
    T* live = (T*)en.blob;
    uint8_t* live_idx = (uint8_t*)en.blob + (size_t)en.idx_off * 256;
    // (a lane takes a group at a time and writes its k values; consecutive lanes, consecutive groups of a row)
#pragma unroll
    for (int i = 0; i < IDX_PER; ++i) {
        const int c = (tid + 256 * i) % SC, r = (tid + 256 * i) / SC, co = tile_row_channel(mt, r);
        if (co >= Co || c >= channels || en.b) continue;
        const int64_t g = (int64_t)co * Ci + SC * stage + c;
        live_idx[g] = iv[i];
        const uint64_t taps = L.taps[entry[i]];
        for (int j = 0; j < k; ++j) {
            const unsigned t = (unsigned)(taps >> (4 * j)) & 15u;
            T v = L.w[r][c * 9 + (t < 9 ? t : 0)];
            if (t >= 9) __builtin_memset(&v, 0, sizeof(T));  // an index outside the dictionary
            live[g * k + j] = v;
        }
    }
    // ---- fragments: item = (fragment, lane) ----
    char* out = en.blob + (size_t)en.mat_off * 256;
    if constexpr (SPARSE) {
        constexpr int frags = layout_fragments(lay);
        char* tile_out = out + (size_t)tile * layout_tile_bytes(lay);
        for (int item = tid; item < 64 * frags; item += 256) {
            const int lane = item % 64, step = item / 64;  // (step is uniform over a wave)
            const int r = lane % 16, q = lane / 16;
            const bool row_live = tile_row_channel(mt, r) < Co;
            uint16_t vals[8];
            if (step == 2 * lay.groups) {  // dense centre tap: K = 8q + j
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int c = 8 * q + j;
                    const uint16_t v = __builtin_bit_cast(uint16_t, L.w[r][c * 9 + 4]);
                    vals[j] = (row_live && ((masks[L.idx[r][c]] >> 4) & 1u)) ? v : (uint16_t)0;
                }
            } else {
                const int group = step >> 1, half = step & 1;
                unsigned fields = 0;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int c = stage_channel(q, g, half), p = L.idx[r][c];
                    const unsigned e = row_live ? L.slots[p * kTapGroups + group] : kNoTaps;
                    const unsigned t0 = e & 15u, t1 = (e >> 4) & 15u;  // taps of the two values (15: none)
                    const uint16_t v0 = __builtin_bit_cast(uint16_t, L.w[r][c * 9 + (t0 < 9 ? t0 : 0)]);
                    const uint16_t v1 = __builtin_bit_cast(uint16_t, L.w[r][c * 9 + (t1 < 9 ? t1 : 0)]);
                    vals[2 * g] = t0 < 9 ? v0 : (uint16_t)0;
                    vals[2 * g + 1] = t1 < 9 ? v1 : (uint16_t)0;
                    fields |= ((e >> 8) & 15u) << (4 * g);  // slot of the first value | slot of the second << 2
                }
                *(uint16_t*)(tile_out + frags * kFragBytes + (group * 64 + lane) * 4 + half * 2) = (uint16_t)fields;
            }
            u32x4 pk;
            __builtin_memcpy(&pk, vals, 16);
            store16_through(tile_out + step * kFragBytes + lane * 16, pk);
        }
    } else {
        constexpr int PER = 16 / (int)sizeof(T);
        char* tile_out = out + (size_t)tile * kDenseTileBytes;
        for (int item = tid; item < 64 * 9; item += 256) {
            const int lane = item % 64, t = item / 64;
            const int r = lane % 16, q = lane / 16;
            T v[PER];
#pragma unroll
            for (int j = 0; j < PER; ++j) {
                const int c = PER * q + j;
                v[j] = L.w[r][c * 9 + t];
                if (!((masks[L.idx[r][c]] >> t) & 1u)) __builtin_memset(&v[j], 0, sizeof(T));  // (rows past Co are zeros)
            }
            u32x4 pk;
            __builtin_memcpy(&pk, v, 16);
            store16_through(tile_out + item * 16, pk);
        }
    }
}

// A lane's 16 bytes of a 1x1 fragment: consecutive elements of row co starting at channel ci0, pruned.  In two steps, so that the
// loads of a lane's pieces are in flight together: what is loaded, and what becomes of it.
template <typename T> struct Piece1x1 {
    static constexpr int PER = 16 / (int)sizeof(T);
    u32x4 raw;
    uint8_t p0, p1;  // pattern indices of the two groups the piece touches (p1 past the last group: none)
    int t0;          // first element's tap in its group
    bool first, second;  // which of them exist
    __device__ __forceinline__ void load(const T* __restrict__ w, const uint8_t* __restrict__ idx, int Co, int Ci, int co, int ci0)
    {
        raw = u32x4{0, 0, 0, 0};
        p0 = p1 = 0;
        t0 = 0;
        first = second = false;
        if (co >= Co || ci0 >= Ci) return;
        // element f of the flattened matrix sits in group f/9 at tap f%9 (groups may straddle rows; the tail has no group)
        const int64_t f0 = (int64_t)co * Ci + ci0, G = (int64_t)Co * Ci / 9;
        const int64_t g0 = f0 < (int64_t)1 << 31 ? (int64_t)((uint32_t)f0 / 9u) : f0 / 9;
        t0 = (int)(f0 - 9 * g0);
        first = g0 < G;  // else all tail (a tensor of fewer than nine weights may come without pointers)
        if (!first) return;
        second = g0 + 1 < G;
        p0 = idx[g0];
        if (second) p1 = idx[g0 + 1];
        if (Ci % PER == 0 && (reinterpret_cast<uintptr_t>(w) & 15) == 0) {
            raw = *(const u32x4*)(w + f0);
        } else {
            T v[PER];
#pragma unroll
            for (int j = 0; j < PER; ++j) {
                __builtin_memset(&v[j], 0, sizeof(T));
                if (ci0 + j < Ci) v[j] = w[f0 + j];
            }
            __builtin_memcpy(&raw, v, 16);
        }
    }
    __device__ __forceinline__ u32x4 pruned(const uint16_t* masks) const
    {
        const unsigned m0 = first ? masks[p0] : 0u, m1 = second ? masks[p1] : 0u;
        const unsigned live = (m0 | m1 << 9) >> t0;  // bit j: the piece's element j survives
        u32x4 pk;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            if constexpr (sizeof(T) == 4) {
                pk[d] = (live >> d) & 1u ? raw[d] : 0u;
            } else {
                const unsigned pair = live >> (2 * d);
                pk[d] = raw[d] & (((pair & 1u) ? 0xffffu : 0u) | ((pair & 2u) ? 0xffff0000u : 0u));
            }
        }
        return pk;
    }
};

// A lane's 16 bytes of a stem fragment (Ci <= 3): K = kh*3*Ci + kw*Ci + ci.  Rows are dealt over each pair of channel
// tiles so that the 4 + 4 accumulator values a lane holds are the 8 consecutive channels 32*(mt/2) + 8q .. +7.
template <typename T>
__device__ __forceinline__ u32x4 pack_piece_stem(const T* __restrict__ w, const uint8_t* __restrict__ idx, const uint16_t* masks,
                                                 int Co, int Ci, int item)
{
    const int lane = item % 64, mt = item / 64, r = lane % 16, q = lane / 16;
    const int co = 32 * (mt >> 1) + 8 * (r >> 2) + 4 * (mt & 1) + (r & 3);
    uint16_t v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int k = 8 * q + j;
        v[j] = 0;
        if (co < Co && k < 9 * Ci) {
            const int t = k / Ci, ci = k - t * Ci;
            const int g9 = co * Ci + ci;
            if ((masks[idx[g9]] >> t) & 1u) v[j] = __builtin_bit_cast(uint16_t, w[g9 * 9 + t]);
        }
    }
    u32x4 pk;
    __builtin_memcpy(&pk, v, 16);
    return pk;
}

template <typename T, int N, typename D>
__global__ __launch_bounds__(256) void pack_kernel(PackTable<N> tab, D dict)
{
    constexpr bool SMALL = std::is_same_v<D, SmallDict>;
    __shared__ uint16_t masks[256];
    union Lds {
        TileLds<T> tile;
        __attribute__((aligned(16))) char live[live_block_lds_bytes<T>()];
    };
    __shared__ Lds lds;
    const int tid = threadIdx.x;
    // A block's layer is the last entry that starts at or before it.  Every lane loads one entry along with the table of
    // first blocks and its mask, and the layer's is broadcast from its lane: one round trip to the launch arguments,
    // which no cache holds yet, instead of two.
    const int lane0 = tid & 63;
    const int slot = lane0 < N ? lane0 : 0;
    const int my_first = lane0 < N ? tab.first_block[slot] : 0x7fffffff;  // (entries past the last layer: past every block)
    union {
        PackEntry e;
        uint32_t w[sizeof(PackEntry) / 4];
    } row, pick;
    row.e = tab.e[slot];
    const unsigned mask = dict.mask[SMALL ? tid & (kOneWave - 1) : tid];  // of the pattern whose table entries this lane makes
    masks[tid] = SMALL && tid >= kOneWave ? (uint16_t)0 : (uint16_t)mask;
    const int t = __builtin_popcountll(__ballot(my_first <= (int)blockIdx.x)) - 1;
#pragma unroll
    for (int i = 0; i < (int)(sizeof(PackEntry) / 4); ++i) pick.w[i] = (uint32_t)__builtin_amdgcn_readlane((int)row.w[i], t);
    const PackEntry en = pick.e;
    int block = (int)blockIdx.x - __builtin_amdgcn_readlane(my_first, t);
    const bool is3x3 = en.format == kFormatSparse24 || en.format == kFormatDense3x3;
    char* section = en.blob + (size_t)en.mat_off * 256;
    const int stages = (en.Ci + stage_channels(sizeof(T) == 4 ? RTOSS_F32 : RTOSS_F16) - 1) / (64 / (int)sizeof(T));
    if (is3x3) {
        const int m_tiles = (int)en.items / stages;
        if (block < (int)en.items) {
            if constexpr (sizeof(T) == 2)
                if (en.format == kFormatSparse24) {
                    if (en.a == 0) pack_tile3x3<T, 0, SMALL>(en, dict.k, mask, masks, block, m_tiles, lds.tile);
                    else pack_tile3x3<T, 1, SMALL>(en, dict.k, mask, masks, block, m_tiles, lds.tile);
                    return;
                }
            pack_tile3x3<T, kDenseTaps, SMALL>(en, dict.k, mask, masks, block, m_tiles, lds.tile);
            return;
        }
        // the block behind the tiles writes the block of zeros
        const size_t end = (size_t)en.items * (en.format == kFormatSparse24 ? layout_tile_bytes(kLayouts[en.a]) : kDenseTileBytes);
        for (int b = tid * 16; b < zero_section_bytes(stages); b += 4096) *(u32x4*)(section + end + b) = u32x4{0, 0, 0, 0};
        return;
    }
    __syncthreads();  // masks  (3x3 tiles have a barrier of their own in front of their first use)
    // other formats: first the public section
    const int ks2 = en.format == kFormatStem || en.c == 9 ? 9 : 1;
    LiveJob job;
    job.G = (int64_t)en.Co * en.Ci * ks2 / 9;
    job.blocks = (int)((job.G + 256 * kLiveRuns - 1) / (256 * kLiveRuns));
    if (block < job.blocks) {
        job.live = en.blob;
        job.live_idx = (uint8_t*)en.blob + (size_t)en.idx_off * 256;
        for (int i = 0; i < kLiveRuns && (int64_t)(block * kLiveRuns + i) * 256 < job.G; ++i)
            pack_live_block<T>((const T*)en.w, en.idx, masks, dict.k, job, block * kLiveRuns + i, lds.live);
        return;
    }
    const int base = (block - job.blocks) * 256 * kPieces + tid;
    const T* w = (const T*)en.w;
    constexpr int PER = 16 / (int)sizeof(T);
    const int zeros = en.format == kFormatStem ? 0 : zero_section_bytes(stages) / 16;
    if constexpr (sizeof(T) == 2)
        if (en.format == kFormatStem) {
            for (int i = 0; i < kPieces; ++i) {
                const int item = base + 256 * i;
                if (item < (int)en.items) *(u32x4*)(section + (size_t)item * 16) = pack_piece_stem<T>(w, en.idx, masks, en.Co, en.Ci, item);
            }
            return;
        }
    if (en.format != kFormatDenseStream && en.format != kFormatDense) return;
    Piece1x1<T> piece[kPieces];
#pragma unroll
    for (int i = 0; i < kPieces; ++i) {
        const int item = base + 256 * i, lane = item % 64, r = lane % 16, q = lane / 16;
        int co = en.Co, s = 0;  // (past the fragments: nothing)
        int f = item / 64;
        if (item < (int)en.items) {
            if (en.format == kFormatDenseStream) {
                // rows permuted so that a lane's 4*MT accumulator values are consecutive channels (KS and MT are powers of two)
                const int log_ks = en.a, log_mt = en.b;
                s = f & ((1 << log_ks) - 1);
                f >>= log_ks;
                const int m = f & ((1 << log_mt) - 1);
                f >>= log_mt;
                co = ((f * 16 + (r / 4) * 4) << log_mt) + 4 * m + (r % 4);  // (f: channel block and wave slice)
            } else {
                const int m_tiles = (int)en.items / (64 * stages);
                s = f / m_tiles;
                co = 16 * (f - s * m_tiles) + r;
            }
        }
        piece[i].load(w, en.idx, en.Co, en.Ci, co, 4 * PER * s + PER * q);
    }
#pragma unroll
    for (int i = 0; i < kPieces; ++i) {
        const int item = base + 256 * i;
        if (item < (int)en.items + zeros) store16_through(section + (size_t)item * 16, piece[i].pruned(masks));
    }
}

// Table entry of one layer and the number of blocks it takes.
rtoss_status make_entry(const PackItem& it, const BlobGeometry& g, int layout, PackEntry* en, int64_t* blocks)
{
    const rtoss_wdesc& d = it.d;
    en->w = it.w;
    en->idx = it.idx;
    en->blob = (char*)it.live;  // section 0 starts the blob
    if (g.total / 256 > 0xffffffffull) return fail(RTOSS_ESHAPE, "pack: blob too large");
    en->idx_off = (uint32_t)(g.idx_off / 256);
    en->mat_off = (uint32_t)(g.mat_off / 256);
    en->Co = d.Co;
    en->Ci = d.Ci;
    en->format = (uint8_t)g.format;
    en->a = en->b = en->c = 0;
    const int stages = stage_count(d);
    const int64_t live_blocks = (g.G + 256 * kLiveRuns - 1) / (256 * kLiveRuns);
    const auto piece_blocks = [](int64_t pieces) { return (pieces + 256 * kPieces - 1) / (256 * kPieces); };
    int64_t items = 0;
    switch (g.format) {
    case kFormatSparse24:
        en->a = (uint8_t)layout;
        en->c = g.dense_off != 0;
        items = (int64_t)stages * padded_m_tiles(d.Co);
        *blocks = items + 1;
        break;
    case kFormatDense3x3:
        en->b = g.dense_off != 0;
        items = (int64_t)stages * 4 * dense_channel_blocks(d.Co);
        *blocks = items + 1;
        break;
    case kFormatDenseStream: {
        const int KS = stages, MT = stream_mt_of(KS), WM = stream_wm_of(KS, d.Co);
        en->a = (uint8_t)__builtin_ctz(KS);
        en->b = (uint8_t)__builtin_ctz(MT);
        items = (int64_t)stream_co_blocks_of(KS, d.Co) * WM * MT * KS * 64;
        *blocks = live_blocks + piece_blocks(items + zero_section_bytes(stages) / 16);
        break;
    }
    case kFormatDense:
        items = (int64_t)stages * ring_padded_tiles(d.Co) * 64;
        *blocks = live_blocks + piece_blocks(items + zero_section_bytes(stages) / 16);
        break;
    case kFormatStem:
        items = 4 * 64;
        *blocks = live_blocks + 1;
        break;
    default:
        en->c = d.ksize == 3 ? 9 : 0;
        *blocks = live_blocks;
    }
    if (items > 0x7fffff00 || *blocks > kMaxGridGroups) return fail(RTOSS_ESHAPE, "pack: layer too large");
    en->items = (uint32_t)items;
    return RTOSS_OK;
}

}  // namespace

namespace {

template <typename T, int N, typename D> rtoss_status launch_table(const PackTable<N>& tab, const D& dict, int64_t blocks, hipStream_t s)
{
    pack_kernel<T, N, D><<<dim3((unsigned)blocks), dim3(256), 0, s>>>(tab, dict);
    return check_hip(hipGetLastError(), "pack launch");
}

template <typename T> rtoss_status launch_entries(const PackTable<kPackMax>& tab, int m, const Dict& dict, int64_t blocks, hipStream_t s)
{
    if (dict.P >= kOneWave) return launch_table<T>(tab, dict, blocks, s);
    SmallDict d{};
    std::copy(dict.mask, dict.mask + dict.P, d.mask);
    d.k = dict.k;
    if (m > kPackFew) return launch_table<T>(tab, d, blocks, s);
    PackTable<kPackFew> few;
    std::copy(tab.e, tab.e + kPackFew, few.e);
    std::copy(tab.first_block, tab.first_block + kPackFew, few.first_block);
    return launch_table<T>(few, d, blocks, s);
}

}  // namespace

rtoss_status launch_pack(const PackItem* items, const BlobGeometry* geo, int n, const Dict& dict, hipStream_t s)
{
    const int layout = std::max(0, dict.layout);
    // 3x3 layers first: their workgroups take longest.  (Two walks over the layers instead of a sorted list: nothing here allocates,
    // so that nothing can throw through the C interface.)
    for (int dt : {(int)RTOSS_F32, (int)RTOSS_F16, (int)RTOSS_BF16})
        for (int64_t i = 0; i < 2 * (int64_t)n;) {  // i runs on across launches
            PackTable<kPackMax> tab;
            int m = 0;
            int64_t total = 0;
            for (; i < 2 * (int64_t)n && m < kPackMax; ++i) {
                const int l = (int)(i < n ? i : i - n);
                const PackItem& it = items[l];
                if ((int)it.d.dt != dt || it.d.ksize != (i < n ? 3 : 1)) continue;
                int64_t blocks = 0;
                if (rtoss_status st = make_entry(it, geo[l], layout, &tab.e[m], &blocks)) return st;
                if (blocks == 0) continue;
                if (total + blocks > kMaxGridGroups) break;  // (one layer fits: make_entry)
                tab.first_block[m++] = (int)total;
                total += blocks;
            }
            if (m == 0) continue;
            for (int t = m; t < kPackMax; ++t) tab.first_block[t] = 0x7fffffff;
            const rtoss_status st = dt == RTOSS_F32   ? launch_entries<float>(tab, m, dict, total, s)
                                    : dt == RTOSS_F16 ? launch_entries<f16_t>(tab, m, dict, total, s)
                                                      : launch_entries<bf16_t>(tab, m, dict, total, s);
            if (st) return st;
        }
    return RTOSS_OK;
}

}  // namespace rtoss
