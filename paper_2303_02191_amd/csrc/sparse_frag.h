// Layout of the 2-of-4 compressed weight fragments that the packer writes and the 3x3 kernels on the
// sparse matrix instruction stream (conv3x3_sparse.hip, conv3x3_rows.hip).
#pragma once
#include "common.h"
#include "mma.h"

namespace rtoss {

// How the 9 taps of a kernel are laid onto the matrix instructions: `groups` sets of 4 taps, each a 2-of-4
// group of the sparse instruction (legal for a dictionary when no pattern has more than 2 live taps in any set),
// and optionally the centre tap as a dense K-slot.  Per 32 input channels a layout costs 2 sparse steps per group
// + 1 dense step for the centre, against 9 dense steps.
//   Layout 0, corners / edge midpoints / centre: 5 steps.  Fits the edge-connected patterns of 2 and 3 entries
//   (the T shapes of 4 entries have 3 edge midpoints).
//   Layout 1, three groups: 6 steps.  Three groups of four have twelve slots for nine taps: the last slot of a group
//   repeats a tap that stands in another group, and the packer takes it from there where the pattern needs that (tap_choice).
//   An exhaustive search over three sets of four taps: with every tap in one group {0,4,8} {1,5,6} {2,3,7} place all 36
//   edge-connected patterns of 4 entries, none places the 49 of 5; with repeats, 451 of the 512 masks fit the best choices, those 49 and
//   everything that {0,4,8} {1,5,6} {2,3,7} place among them.  (6 entries: the matrix instruction's 6 live taps a channel, but not all 48 fit.)
struct TapLayout {
    int groups;     // sparse groups
    int centre;     // 1: tap 4 is a dense step of its own
    int repeats;    // 1: the last slot of every group repeats a tap of another group
    int tap[3][4];  // taps of each group's 4 slots
};
constexpr int kNumLayouts = 2;
constexpr TapLayout kLayouts[kNumLayouts] = {
    {2, 1, 0, {{0, 2, 6, 8}, {1, 3, 5, 7}, {-1, -1, -1, -1}}},
    {3, 0, 1, {{0, 4, 8, 7}, {1, 5, 6, 8}, {2, 3, 7, 5}}},
};
// A choice: bit g set = group g takes the tap of its last slot from the group that it stands in first.  The taps that a group has
// under a choice, as a mask.
constexpr int kTapChoices = 8;
__host__ __device__ constexpr unsigned group_taps(const TapLayout& l, int g, int choice)
{
    unsigned taps = 0;
    for (int f = 0; f < 4; ++f) {
        bool here = !l.repeats || f < 3 || (choice >> g & 1);
        if (l.repeats && f < 3)
            for (int o = 0; o < l.groups; ++o) here = here && !(l.tap[o][3] == l.tap[g][f] && (choice >> o & 1));
        if (here) taps |= 1u << l.tap[g][f];
    }
    return taps;
}
// The first choice under which a pattern has at most two live taps in every group; -1: none.
constexpr int tap_choice(const TapLayout& l, unsigned mask)
{
    for (int c = 0; c < (l.repeats ? kTapChoices : 1); ++c) {
        bool fits = true;
        for (int g = 0; g < l.groups; ++g) {
            int live = 0;
            for (unsigned m = mask & group_taps(l, g, c); m; m &= m - 1) ++live;
            fits = fits && live <= 2;
        }
        if (fits) return c;
    }
    return -1;
}
// Packed weight fragments: per (stage of 32 input channels, tile of 16 output channels)
//   operand fragments of 64 lanes x 16 bytes: [group][step 0/1] ..., then the centre's if the layout has one
//   then one index word per lane and group: [group][lane]; low half = step 0, high = step 1
// (which output channel a row of a tile is: tile_row_channel)
constexpr int kFragBytes = 1024;
constexpr int layout_fragments(const TapLayout& l) { return 2 * l.groups + l.centre; }
constexpr int layout_tile_bytes(const TapLayout& l) { return layout_fragments(l) * kFragBytes + l.groups * 64 * 4; }

// Output channel held by row r of channel tile mt.  Within a group of 4 tiles (64 channels) the rows
// are dealt so that the accumulator values one lane holds after the multiplication -- rows
// 4q .. 4q+3 of each of the 4 tiles -- are the 16 consecutive channels 64*(mt/4) + 16q .. +15:
// the epilogues store runs of 16 channels without exchanging data between lanes.
__device__ __forceinline__ int tile_row_channel(int mt, int r)
{
    return 64 * (mt >> 2) + 16 * (r >> 2) + 4 * (mt & 3) + (r & 3);
}
// first of the 4 consecutive channels that quarter q of a lane holds of tile mm (counted from the
// first channel of mm's group of 4 tiles when mm < 4; mm may run over several groups)
__device__ __forceinline__ int tile_quarter_offset(int mm, int q)
{
    return 64 * (mm >> 2) + 16 * q + 4 * (mm & 3);
}

// B operand of a sparse step from 16-byte reads of the group's four taps (8 channels each): element 4*c + f = channel c of
// the step's four, tap slot f.  A 4x4 (tap, channel) transposition of byte pairs.  `half`: channels 0-3 or 4-7 of the reads.
__device__ __forceinline__ u32x8 sparse_operand(const u32x4 (&r)[4], int half)
{
    u32x8 b;
#pragma unroll
    for (int p = 0; p < 2; ++p) {  // channel pair: one dword of each tap
        const int d = 2 * half + p;
        b[4 * p + 0] = __builtin_amdgcn_perm(r[1][d], r[0][d], 0x05040100u);  // first channel: taps 0,1
        b[4 * p + 1] = __builtin_amdgcn_perm(r[3][d], r[2][d], 0x05040100u);  // ... taps 2,3
        b[4 * p + 2] = __builtin_amdgcn_perm(r[1][d], r[0][d], 0x07060302u);  // second channel
        b[4 * p + 3] = __builtin_amdgcn_perm(r[3][d], r[2][d], 0x07060302u);
    }
    return b;
}

// Channel tiles per stage in the packed section: padded so that every block of 8 tiles is complete.
inline int padded_m_tiles(int Co) { return ((Co + 15) / 16 + 7) / 8 * 8; }
// The section is [fragments][block of zeros]; the zeros feed the copy lanes that fill padding.
// Stages of 32 input channels; a last stage with fewer channels is filled with zero weights.
inline int sparse_stages(const rtoss_wdesc& d) { return (d.Ci + 31) / 32; }
inline size_t fragment_bytes(const rtoss_wdesc& d, int layout = 0)
{
    return (size_t)sparse_stages(d) * padded_m_tiles(d.Co) * layout_tile_bytes(kLayouts[layout]);
}
inline size_t zero_block_bytes(const rtoss_wdesc& d) { return align_up((size_t)64 * sparse_stages(d) + 16, 256); }

}  // namespace rtoss
