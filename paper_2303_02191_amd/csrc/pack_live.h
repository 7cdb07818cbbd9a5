// The blob's public section 0 (the k survivors of every group in ascending tap order, plus a copy
// of the group's pattern index): this is the mask step W' = W (.) M of Section II.B, and the
// zeroing of a flattened 1x1 tensor's tail (Section IV.D) in the sense that the tail belongs to
// no group.  Shared by the packers, which do this work in their first blocks so that a layer is
// packed by one launch.
#pragma once
#include "common.h"
#include "dtypes.h"
#include "mma.h"

namespace rtoss {

struct LiveJob {
    void* live;         // [G][k] values
    uint8_t* live_idx;  // [G]
    int64_t G;
    int blocks;         // workgroups: of 256 groups each, or of as many runs of 256 as the caller has them do
};

inline LiveJob make_live_job(void* live, uint8_t* live_idx, int64_t G)
{
    LiveJob j;
    j.live = live;
    j.live_idx = live_idx;
    j.G = G;
    j.blocks = (int)((G + 255) / 256);
    return j;
}

template <typename T> constexpr int live_block_lds_bytes() { return 2 * 256 * 9 * (int)sizeof(T); }

// One workgroup's 256 groups; `masks` is the dictionary in LDS (entries past P are 0), `lds` live_block_lds_bytes<T>()
// bytes, 16-byte aligned.  The 2304 weights come in and the 256*k survivors go out as whole 16-byte vectors, through
// LDS: a lane's own nine weights lie 18 (or 36) bytes from its neighbour's, so reading them from memory one tap at a
// time took nine loads over the same lines.
template <typename T>
__device__ __forceinline__ void pack_live_block(const T* __restrict__ w, const uint8_t* __restrict__ idx,
                                                const uint16_t* masks, int k, const LiveJob& job, int block, char* lds)
{
    constexpr int EPV = 16 / (int)sizeof(T);
    T* in = (T*)lds;
    T* out = in + 256 * 9;
    const int tid = threadIdx.x;
    const int64_t g0 = (int64_t)block * 256;
    const int n = job.G - g0 < 256 ? (int)(job.G - g0) : 256;
    const T* src = w + g0 * 9;
    const int n_in = n * 9;
    const bool mine = tid < n;
    const uint8_t p = mine ? idx[g0 + tid] : 0;
    if ((reinterpret_cast<uintptr_t>(src) & 15) == 0) {
        for (int e = tid * EPV; e + EPV <= n_in; e += 256 * EPV) *(u32x4*)(in + e) = *(const u32x4*)(src + e);
        for (int e = n_in / EPV * EPV + tid; e < n_in; e += 256) in[e] = src[e];
    } else {
        for (int e = tid; e < n_in; e += 256) in[e] = src[e];
    }
    __syncthreads();
    if (mine) {
        const unsigned m = masks[p];
        int j = 0;
#pragma unroll
        for (int t = 0; t < 9; ++t)
            if ((m >> t) & 1u) {
                if (j < k) out[tid * k + j] = in[tid * 9 + t];
                ++j;
            }
        T zero;
        __builtin_memset(&zero, 0, sizeof(T));
        for (; j < k; ++j) out[tid * k + j] = zero;  // only reached for an index outside the dictionary
        job.live_idx[g0 + tid] = p;
    }
    __syncthreads();
    T* dst = (T*)job.live + g0 * k;  // (a multiple of 16 bytes from the blob's start)
    const int n_out = n * k;
    for (int e = tid * EPV; e + EPV <= n_out; e += 256 * EPV) store16_through(dst + e, *(const u32x4*)(out + e));
    for (int e = n_out / EPV * EPV + tid; e < n_out; e += 256) dst[e] = out[e];
}

}  // namespace rtoss
