// How the streaming 1x1 kernels (conv1x1_stream.hip) deal the buffers of a launch out to workgroups: contiguous ranges whose lengths differ
// by one at most.
//
// Which of them are longer: the ranges of an XCD are an eighth of all in a row (work order of those kernels), and each eighth has the
// same number of longer ones, at its front, so that the XCDs and the compute units of an XCD are loaded alike.  us with the
// longer ones in front of all (one XCD's then), spread evenly, and this way:
//     16 bit  32 -> 256 (51 200 positions), fp32 results  22.3  20.8  19.3     64 -> 256 (51 200), SiLU  12.1  12.3  11.2
//     fp32   256 ->  64 (21 888)                          11.2   9.8   8.1     64 ->  64 (51 200)         8.1   7.5   6.8
//     16 bit  32 ->  64 (102 400)                          6.3   6.3   6.7    512 -> 512 (51 200), SiLU  42.0  42.1  43.4  (the worst two of 240)
// (worked out from the host's quotients: dividing in the kernel is some hundred scalar instructions before a workgroup's first load)
#pragma once
#include <cstdint>

namespace rtoss {

struct Range { int first, end; };

struct Share {
    int each, part, more, rest;  // buffers of a range; ranges of a part; longer ranges of a part, parts that have one more of them
    uint32_t per_part;           // 2^32 / part, rounded up

    Share(int64_t buffers, int ranges)
    {
        const int parts = ranges % 8 == 0 && ranges >= 16 ? 8 : 1, longer = (int)(buffers % ranges);
        each = (int)(buffers / ranges);
        part = ranges / parts;
        more = longer / parts;
        rest = longer % parts;
        per_part = part > 1 ? (uint32_t)(((uint64_t)1 << 32) / part + 1) : 0;  // (exact quotients: ranges * part < 2^32)
    }
    __host__ __device__ Range of(int range) const
    {
        const int p = (int)((uint64_t)(uint32_t)range * per_part >> 32), at = range - p * part, longer = more + (p < rest ? 1 : 0);
        const int first = range * each + p * more + (p < rest ? p : rest) + (at < longer ? at : longer);
        return {first, first + each + (at < longer ? 1 : 0)};
    }
};

}  // namespace rtoss
