// How output rows leave a workgroup: in pieces of 16 bytes, past the L2's write-back where memory is written in whole sectors.
#pragma once

namespace rtoss {

// Memory is written in sectors of 64 bytes: a store past the L2's write-back (store16_through) of a part of one makes memory read and
// write it, where the L2 would have put the parts together.  us before such stores, with them at every pitch (tensors not in any
// cache): 1x1 40 -> 1000 channels on 28 028 positions, rows of 2000 bytes, 26.2 32.3, fp32 results, 4000 bytes, 30.3 40.2; 72 -> 2104,
// 4208 bytes, 53.2 65.1; 72 -> 1024, 2048 bytes, 29.8 28.3, into a slice of rows of 2080 bytes 37.5 42.0, fp32 results of 4160 bytes 38.1 32.3.
constexpr int kSector = 64;

// Whether every piece of every row is whole and starts at a multiple of `unit` bytes: blocks of `row` bytes, `first` bytes into rows that
// are `pitch` bytes apart, in a tensor at address `at`.
constexpr bool aligned_pieces(unsigned long long at, int row, int first, long long pitch, int unit)
{
    return ((at | (unsigned)row | (unsigned)first | (unsigned long long)pitch) & (unsigned)(unit - 1)) == 0;
}

// ... of the whole output of a layer of `channels` channels
inline bool whole_sectors(const void* y, int channels, int pitch, int elem)
{
    return aligned_pieces((unsigned long long)y, channels * elem, 0, (long long)pitch * elem, kSector);
}

}  // namespace rtoss
