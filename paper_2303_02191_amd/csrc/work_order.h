// Which tile a workgroup has: numbers taken apart by multiplication.
//
// A division by a launch argument is about 30 dependent scalar instructions (a float reciprocal and its corrections), and a workgroup of
// the 3x3 kernels has three in front of its first copy, at the start of a chain of latencies that nothing covers.  The host
// knows the divisors.  (us, divided in the kernel and multiplied: fp32 64 -> 64 @ 56 5.67 5.53, 20 launches of a pyramid of 256 channels
// 152.5 149.4, 57 layers of a detector at batch 16 709.1 706.8.)
#pragma once
#include <cstdint>

namespace rtoss {

// n / by for 0 <= n < 2^31, by multiplication with 2^32 * 2^shift / by (Granlund and Montgomery, Division by Invariant Integers using
// Multiplication: the factor less 2^32, rounded up, whose high product with n is then added to n).
struct Divisor {
    int by, shift;
    uint32_t factor;

    explicit Divisor(int divisor)  // (at least 1)
    {
        by = divisor;
        shift = by > 1 ? 32 - __builtin_clz(by - 1) : 0;
        factor = (uint32_t)(((((uint64_t)1 << shift) - by) << 32) / by + 1);
    }
    __host__ __device__ int quotient(int n) const
    {
        const uint32_t u = (uint32_t)n;
        return (int)((uint32_t)((uint64_t)u * factor >> 32) + u >> shift);
    }
    __host__ __device__ int remainder(int n, int q) const { return n - q * by; }
};

// XCD-contiguous work order, channel block fastest: workgroups are dealt to the 8 XCDs in turn, and each XCD takes a contiguous range of
// the work items, so that those that read one activation tile run on one XCD at about the same time and share its L2.
struct WorkOrder {
    Divisor co_blocks, per_image, across;  // channel blocks; tiles (blocks) of an image, and of a row of the image
    int total, per_xcd;

    WorkOrder(int64_t items, int channel_blocks, int tiles_per_image, int tiles_across)  // (items below 2^30)
        : co_blocks(channel_blocks), per_image(tiles_per_image), across(tiles_across), total((int)items), per_xcd((int)((items + 7) / 8))
    {
    }
    unsigned grid() const { return (unsigned)per_xcd * 8; }
    __device__ int item() const { return (int)(blockIdx.x % 8) * per_xcd + (int)(blockIdx.x / 8); }  // (past the end from `total` on)

    struct Tile {
        int n_img, row, col;
    };
    __host__ __device__ Tile tile(int n) const  // of the n-th over all images
    {
        Tile t;
        t.n_img = per_image.quotient(n);
        const int at = per_image.remainder(n, t.n_img);
        t.row = across.quotient(at);
        t.col = across.remainder(at, t.row);
        return t;
    }
};

}  // namespace rtoss
