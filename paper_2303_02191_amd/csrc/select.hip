// Pattern selection (Section IV.C, Algorithm 2 scoring loop and best-fit choice, on the
// flat 9-element groups of Section IV.D, Algorithm 3).
//
// Mapping: a workgroup is one wave; it scores chunks of 256 groups, four consecutive ones per lane, against
// the whole dictionary.  The 9*256 weights of a chunk are one contiguous span, copied global -> LDS as whole
// 16-byte vectors; each lane takes its own 36 weights from there, squares them in fp64 and keeps the squares in
// registers, and the LDS is free for the wave's next chunk, which is copied while this one is scored.
// Sums run over the live taps in ascending tap order in fp64 and the patterns are scanned in ascending order with a
// strict comparison, which is the definition's serial scan: the result is bit-exact.
//
// What bounds it: instruction issue.  A dictionary in the launch arguments makes the walk over a pattern's taps scalar
// control flow, one uniform branch per tap position: 9 branches for 3 adds, and a wave alone on its SIMD needs 4 us for
// 22 patterns of which the vector unit works a quarter.  So the default rule's dictionaries of 2 to 5 entries
// (edge-connected patterns, the ones Table 3 compares) are compiled in: straight-line code, in which patterns that
// begin alike also share their partial sums (a dictionary in lexicographic order has runs of these; the order of the
// additions stays).  Any other dictionary takes the branching form.
// Measured: 2^20 fp32 groups, 22 patterns, 16.3 us with branches, 9.2 us without; 2^18 bf16 groups 8.0 and 3.0 us.
//
// All tensors of a call share a launch: the table of tensors travels in the launch arguments, every lane loads one
// entry of it, and a chunk's entry is broadcast from its lane.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "counts.h"
#include "dtypes.h"
#include "mma.h"

namespace rtoss {

constexpr int kSelBlock = 64;
constexpr int kSelPerLane = 4;
constexpr int kSelGroupsPerChunk = kSelBlock * kSelPerLane;  // 256

// Tensors of one launch (the selection of a 1x1 tensor is over its own flattening, Section IV.D, so tensors cannot
// simply be concatenated); chunks are numbered through the tensors in table order.
// (One tensor has a table of its own size: 1 KB of launch arguments takes the host 0.4 us to write.)
template <int N> struct SelectBatch {
    const void* w[N];
    uint8_t* idx[N];
    int64_t G[N];
    int first_chunk[N];  // entries past the last tensor hold the total
    int chunks;
};
static_assert(kSelectBatchMax == 64, "one entry per lane");
struct NoDict {};  // in the launch arguments of a compiled-in dictionary

template <typename T> constexpr int kSelSpan = kSelGroupsPerChunk * 9 * (int)sizeof(T);  // bytes of a chunk: 4608 or 9216

__device__ __forceinline__ uint64_t from_lane(uint64_t v, int lane)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane);
    return (uint64_t)hi << 32 | lo;
}

// The edge-connected dictionary of k-entry patterns, as rtoss_pattern_dict generates it: k-subsets of the taps in
// lexicographic order of their ascending tuples.
struct ConnectedDict {
    uint16_t mask[64] = {};
    int P = 0;
};
constexpr bool edge_connected(unsigned m)
{
    unsigned reach = m & (~m + 1u);
    for (;;) {
        unsigned grown = reach;
        for (int t = 0; t < 9; ++t)
            if (reach >> t & 1u) {
                if (t >= 3) grown |= 1u << (t - 3);
                if (t < 6) grown |= 1u << (t + 3);
                if (t % 3 > 0) grown |= 1u << (t - 1);
                if (t % 3 < 2) grown |= 1u << (t + 1);
            }
        grown &= m;
        if (grown == reach) return reach == m;
        reach = grown;
    }
}
constexpr ConnectedDict connected_dict(int k)
{
    ConnectedDict d;
    for (unsigned r = 511; r > 0; --r) {  // tap t as bit 8 - t: lexicographic order of tuples is descending order of r
        unsigned m = 0;
        int n = 0;
        for (int t = 0; t < 9; ++t)
            if (r >> (8 - t) & 1u) {
                m |= 1u << t;
                ++n;
            }
        if (n == k && edge_connected(m)) d.mask[d.P++] = (uint16_t)m;
    }
    return d;
}
template <int K> struct Connected {
    static constexpr ConnectedDict dict = connected_dict(K);
};

// Sum of the live taps of M below tap END, ascending.
template <unsigned M, int END> __device__ __forceinline__ double tap_sum(const double (&sq)[9])
{
    constexpr unsigned below = M & ((1u << END) - 1u);
    constexpr int top = 31 - __builtin_clz(below);  // the last tap to add
    if constexpr ((below & (below - 1)) == 0) return sq[top];
    else return tap_sum<M, top>(sq) + sq[top];
}

// K: the edge-connected dictionary of K-entry patterns; 0: the dictionary in the launch arguments.
template <typename T, int K, int N>
__global__ __launch_bounds__(kSelBlock) void select_kernel(SelectBatch<N> batch, std::conditional_t<(K > 0), NoDict, Dict> dict)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];  // one chunk
    constexpr int SPAN = kSelSpan<T>, COPIES = (SPAN + 1023) / 1024;
    const int lane = threadIdx.x;
    const int entry = N == 1 ? 0 : lane;
    const int my_first = batch.first_chunk[entry];
    const uint64_t my_w = (uint64_t)batch.w[entry], my_idx = (uint64_t)batch.idx[entry], my_G = (uint64_t)batch.G[entry];

    struct Chunk {
        const T* span;
        uint8_t* out;  // index of the chunk's first group
        int groups;
    };
    // finds a chunk and starts copying it; whole chunks on 16-byte boundaries go straight to LDS
    auto fetch = [&](int chunk, char* lds) -> Chunk {
        const int t = N == 1 ? 0 : __builtin_popcountll(__ballot(my_first <= chunk)) - 1;
        const int64_t g0 = (int64_t)(chunk - __builtin_amdgcn_readlane(my_first, t)) * kSelGroupsPerChunk;
        const int64_t remaining = (int64_t)from_lane(my_G, t) - g0;
        Chunk c;
        c.groups = remaining < kSelGroupsPerChunk ? (int)remaining : kSelGroupsPerChunk;
        c.span = (const T*)from_lane(my_w, t) + g0 * 9;
        c.out = (uint8_t*)from_lane(my_idx, t) + g0;
        // Whole vectors go straight to LDS; the few elements behind the last one, and spans that do not start on a 16-byte
        // boundary (the interface asks for element alignment only), one by one.
        const int bytes = c.groups * 9 * (int)sizeof(T);
        const bool vectors = (reinterpret_cast<uintptr_t>(c.span) & 15) == 0;
        const int whole = vectors ? bytes / 16 * 16 : 0;
#pragma unroll
        for (int k = 0; k < COPIES; ++k)
            if (k * 1024 + lane * 16 < whole) copy16_to_lds((const char*)c.span + k * 1024 + lane * 16, lds + k * 1024);
        T* at = (T*)lds;
#pragma unroll 4
        for (int e = whole / (int)sizeof(T) + lane; e < c.groups * 9; e += kSelBlock) at[e] = c.span[e];
        return c;
    };

    int chunk = blockIdx.x;  // (the grid has no more workgroups than chunks)
    Chunk here = fetch(chunk, smem);
    for (;;) {
        // (one wave: the waits order its own copies and LDS writes before the reads below)
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        // lane's groups 4*lane .. 4*lane+3: 36 consecutive elements.  Lanes past the end of the tensor read
        // whatever LDS holds and their results are dropped.
        double sq[kSelPerLane][9];
        {
            T mine[kSelPerLane * 9];
            constexpr int kBytes = kSelPerLane * 9 * (int)sizeof(T);  // 72 or 144: multiples of 8
            const char* src = smem + lane * kBytes;
#pragma unroll
            for (int i = 0; i < kBytes / 8; ++i)
                reinterpret_cast<uint64_t*>(mine)[i] = reinterpret_cast<const uint64_t*>(src)[i];
#pragma unroll
            for (int j = 0; j < kSelPerLane; ++j)
#pragma unroll
                for (int t = 0; t < 9; ++t) {
                    const double d = (double)to_f32(mine[j * 9 + t]);
                    sq[j][t] = d * d;
                }
        }
        const int next = chunk + (int)gridDim.x;
        Chunk coming = here;
        if (next < batch.chunks) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the weights are in registers: the chunk's LDS is free
            coming = fetch(next, smem);
        }

        double best_s[kSelPerLane];
        int best_p[kSelPerLane];
#pragma unroll
        for (int j = 0; j < kSelPerLane; ++j) { best_s[j] = -1.0; best_p[j] = 0; }  // below every real score
        const auto keep = [&](int j, double s, int p) {
            best_p[j] = s > best_s[j] ? p : best_p[j];  // strict: the first of equal scores stays
            best_s[j] = fmax(best_s[j], s);
        };
        if constexpr (K > 0) {
            static_for<Connected<K>::dict.P>([&](auto p_tag) {
                constexpr int p = decltype(p_tag)::value;
                constexpr unsigned m = Connected<K>::dict.mask[p];
#pragma unroll
                for (int j = 0; j < kSelPerLane; ++j) keep(j, tap_sum<m, 9>(sq[j]), p);
            });
        } else {
            for (int p2 = 0; 2 * p2 < dict.P; ++p2) {
                uint32_t pair;  // masks 2*p2 and 2*p2+1 in one 32-bit scalar load (there is no 16-bit one)
                __builtin_memcpy(&pair, &dict.mask[2 * p2], 4);
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int p = 2 * p2 + h;
                    if (p >= dict.P) break;
                    const unsigned m = (pair >> (16 * h)) & 0xffffu;
                    double s[kSelPerLane];
#pragma unroll
                    for (int j = 0; j < kSelPerLane; ++j) s[j] = 0.0;
#pragma unroll
                    for (int t = 0; t < 9; ++t)
                        if (m & (1u << t)) {  // wave-uniform
                            asm volatile("");  // keeps this a branch: as selects it would cost three times the adds
#pragma unroll
                            for (int j = 0; j < kSelPerLane; ++j) s[j] += sq[j][t];
                        }
#pragma unroll
                    for (int j = 0; j < kSelPerLane; ++j) keep(j, s[j], p);
                }
            }
        }

        const int first = kSelPerLane * lane;
        uint8_t* o = here.out + first;
        if (first + kSelPerLane <= here.groups && (reinterpret_cast<uintptr_t>(o) & 3) == 0) {
            *reinterpret_cast<uint32_t*>(o) =
                (uint32_t)best_p[0] | ((uint32_t)best_p[1] << 8) | ((uint32_t)best_p[2] << 16) | ((uint32_t)best_p[3] << 24);
        } else {
#pragma unroll
            for (int j = 0; j < kSelPerLane; ++j)
                if (first + j < here.groups) o[j] = (uint8_t)best_p[j];
        }
        if (next >= batch.chunks) break;
        here = coming;
        chunk = next;
    }
}

template <typename T, int K, int N> static rtoss_status launch_dict(const SelectBatch<N>& b, const Dict& dict, hipStream_t s)
{
    DeviceInfo dev;
    if (rtoss_status st = current_device(&dev)) return st;
    // as many waves as are resident at once (four per SIMD, by registers): fewer, each with several chunks, measured
    // slower (2^20 groups: 13.3 us with 16 waves per compute unit, 14.8 with 12, 17.4 with 8)
    constexpr int kPerCu = 16;
    dim3 grid((unsigned)std::min(b.chunks, dev.cus * kPerCu)), block(kSelBlock);
    if constexpr (K > 0) select_kernel<T, K, N><<<grid, block, kSelSpan<T>, s>>>(b, NoDict{});
    else select_kernel<T, K, N><<<grid, block, kSelSpan<T>, s>>>(b, dict);
    return check_hip(hipGetLastError(), "select launch");
}

template <int K> static bool is_connected(const Dict& dict)
{
    constexpr const ConnectedDict& c = Connected<K>::dict;
    return dict.P == c.P && std::equal(c.mask, c.mask + c.P, dict.mask);
}

template <typename T, int N> static rtoss_status launch_table(const SelectBatch<N>& b, const Dict& dict, hipStream_t s)
{
    if (is_connected<2>(dict)) return launch_dict<T, 2, N>(b, dict, s);
    if (is_connected<3>(dict)) return launch_dict<T, 3, N>(b, dict, s);
    if (is_connected<4>(dict)) return launch_dict<T, 4, N>(b, dict, s);
    if (is_connected<5>(dict)) return launch_dict<T, 5, N>(b, dict, s);
    return launch_dict<T, 0, N>(b, dict, s);
}

template <int N> static rtoss_status launch_dtype(const SelectBatch<N>& b, rtoss_dtype dt, const Dict& dict, hipStream_t s)
{
    return dt == RTOSS_F32 ? launch_table<float, N>(b, dict, s) : dt == RTOSS_F16 ? launch_table<f16_t, N>(b, dict, s) : launch_table<bf16_t, N>(b, dict, s);
}

rtoss_status launch_select_batch(const rtoss_select_item* items, int n, rtoss_dtype dt, const Dict& dict, hipStream_t s)
{
    for (int i = 0; i < n;) {  // i runs on across launches: tensors without a whole group take no table entry
        SelectBatch<kSelectBatchMax> b;
        int m = 0;
        int64_t chunks = 0;
        for (; i < n && m < kSelectBatchMax; ++i) {
            const int64_t G = items[i].n_elems / 9;
            if (G == 0) continue;
            b.w[m] = items[i].w_dev;
            b.idx[m] = items[i].idx_dev;
            b.G[m] = G;
            b.first_chunk[m] = (int)chunks;
            chunks += (G + kSelGroupsPerChunk - 1) / kSelGroupsPerChunk;
            if (chunks > 0x3fffffffLL) return fail(RTOSS_ESHAPE, "select: too many groups in one call");
            ++m;
        }
        if (m == 0) continue;
        for (int t = m; t < kSelectBatchMax; ++t) b.first_chunk[t] = (int)chunks;  // never at or before a chunk
        b.chunks = (int)chunks;
        rtoss_status st;
        if (m == 1) st = launch_dtype(SelectBatch<1>{{b.w[0]}, {b.idx[0]}, {b.G[0]}, {0}, b.chunks}, dt, dict, s);
        else st = launch_dtype(b, dt, dict, s);
        if (st) return st;
    }
    return RTOSS_OK;
}

rtoss_status launch_select(const void* w, rtoss_dtype dt, int64_t G, const Dict& dict, uint8_t* idx, hipStream_t s)
{
    const rtoss_select_item item{w, G * 9, idx};
    return launch_select_batch(&item, 1, dt, dict, s);
}

// Usage count of every pattern (Section IV.B, second narrowing criterion): one byte per group in,
// P counters out.  Each workgroup counts a slice in LDS (integer atomics; the result is independent
// of their order) and adds its non-zero bins to the global counters.
// Bound by latency: a lane takes 16 indices with one vector load, and every bin exists kHistCopies times, by lane, so
// that the lanes of a wave, whose indices come from a few dozen values, seldom meet at a counter.  2^20 indices:
// 6.0 us with byte loads and single bins, now 3.3 us.
constexpr int kHistBytesPerThread = 16;
constexpr int kHistCopies = 16;

template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void histogram_kernel(const uint8_t* __restrict__ idx, int64_t G, int P,
                                                               uint32_t* __restrict__ hist)
{
    constexpr int kChunk = BLOCK * kHistBytesPerThread;  // indices per workgroup and pass
    __shared__ uint32_t bins[256 * kHistCopies];
    const int tid = threadIdx.x, copy = tid % kHistCopies;
    const bool vectors = (reinterpret_cast<uintptr_t>(idx) & 15) == 0;  // (the index tensor may start anywhere)
    for (int b = tid; b < P * kHistCopies; b += BLOCK) bins[b] = 0;
    __syncthreads();
    for (int64_t base = (int64_t)blockIdx.x * kChunk; base < G; base += (int64_t)gridDim.x * kChunk) {
        const int64_t g0 = base + (int64_t)tid * kHistBytesPerThread;
        if (vectors && g0 + kHistBytesPerThread <= G) {
            const u32x4 v = *(const u32x4*)(idx + g0);
#pragma unroll
            for (int i = 0; i < kHistBytesPerThread; ++i) {
                const int p = (int)(v[i / 4] >> (8 * (i % 4))) & 0xff;
                if (p < P) atomicAdd(&bins[p * kHistCopies + copy], 1u);
            }
        } else {
            for (int i = 0; i < kHistBytesPerThread; ++i)
                if (g0 + i < G) {
                    const int p = idx[g0 + i];
                    if (p < P) atomicAdd(&bins[p * kHistCopies + copy], 1u);
                }
        }
    }
    __syncthreads();
    if (tid < P) {
        uint32_t c = 0;
#pragma unroll
        for (int i = 0; i < kHistCopies; ++i) c += bins[tid * kHistCopies + (i + tid) % kHistCopies];
        if (c != 0) atomicAdd(&hist[tid], c);
    }
}

__global__ __launch_bounds__(256) void clear_kernel(uint32_t* p, int n)
{
    if ((int)threadIdx.x < n) p[threadIdx.x] = 0;
}

rtoss_status clear_counts(uint32_t* hist, int P, hipStream_t s)
{
    clear_kernel<<<dim3(1), dim3(256), 0, s>>>(hist, P);
    return check_hip(hipGetLastError(), "histogram launch");
}

rtoss_status launch_histogram(const uint8_t* idx, int64_t G, int P, uint32_t* hist, hipStream_t s)
{
    if (G == 0) return RTOSS_OK;
    // Large workgroups from 2^18 indices on: every workgroup adds its bins to the same few counters, one after the other,
    // so fewer of them end sooner (2^20 indices: 3.3 us with 64 workgroups of 1024 lanes, 4.0-5.2 with 128-512 of 256).
    // Below that their start-up costs 0.3 us more than it saves.
    const auto blocks = [&](int lanes, int most) {
        return (unsigned)std::min<int64_t>((G + lanes * kHistBytesPerThread - 1) / (lanes * kHistBytesPerThread), most);
    };
    if (G >= (int64_t)1 << 18) histogram_kernel<1024><<<dim3(blocks(1024, 64)), dim3(1024), 0, s>>>(idx, G, P, hist);
    else histogram_kernel<256><<<dim3(blocks(256, 128)), dim3(256), 0, s>>>(idx, G, P, hist);
    return check_hip(hipGetLastError(), "histogram launch");
}

}  // namespace rtoss
