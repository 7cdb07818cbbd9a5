// How the streaming 1x1 kernels (conv1x1_stream.hip) deal the buffers of a launch out to workgroups: in turn, so that what all of them
// read and write at a time lies close together.
//
// The first turn goes through the XCDs (the workgroups of an XCD are an eighth of all in a row: work order of those kernels), so that
// those with a buffer more than the others are spread over the XCDs and the compute units of an XCD.  us with a range for every
// workgroup, the longer ones in front of all (one XCD's then) / with the longer ones spread like this / with buffers in turn (240 shapes:
// 1 / 0.98 / 0.97 of the time; in turn within an XCD's range 0.98):
//     16 bit  32 -> 256 (51 200 positions), fp32 results  22.4  19.3  19.3     64 -> 256 (51 200), SiLU  12.0  11.2  10.9
//     fp32   256 ->  64 (21 888)                          11.2   8.1   8.1     64 ->  64 (51 200)         8.2   6.8   6.9
//     16 bit  32 ->  64 (102 400)                          6.3   6.7   6.4    512 -> 512 (51 200), SiLU  42.0  43.4  41.0
// (worked out from the host's quotients: dividing in the kernel is some hundred scalar instructions before a workgroup's first load)
#pragma once
#include <cstdint>

namespace rtoss {

struct Buffers {  // first, first + step, ...
    int first, step, count;
    __host__ __device__ int64_t at(int64_t i) const { return first + i * step; }
};

struct Share {
    int each, longer, shares;  // buffers of a share; shares that have one more
    int eighth;                // shares of an XCD, or all where they do not divide
    uint32_t per_eighth;       // 2^32 / eighth, rounded up; 0 where they do not divide

    Share(int64_t buffers, int n)  // (n at most buffers)
    {
        const bool divides = n % 8 == 0 && n >= 16;
        shares = n;
        each = (int)(buffers / n);
        longer = (int)(buffers % n);
        eighth = divides ? n / 8 : n;
        per_eighth = divides ? (uint32_t)(((uint64_t)1 << 32) / eighth + 1) : 0;  // (exact quotients: n * eighth < 2^32)
    }
    __host__ __device__ Buffers of(int share) const
    {
        const int xcd = (int)((uint64_t)(uint32_t)share * per_eighth >> 32), at = share - xcd * eighth;
        const int turn = per_eighth ? at * 8 + xcd : share;
        return {turn, shares, each + (turn < longer ? 1 : 0)};
    }
};

}  // namespace rtoss
