// Geometry of the private sections that the packer (pack.hip) writes and the convolution kernels read.
#pragma once
#include "common.h"
#include "sparse_frag.h"

namespace rtoss {

// 64 bytes of input channels per stage; a last stage with fewer channels is filled with zero weights.
__host__ __device__ inline int stage_channels(rtoss_dtype dt) { return dt == RTOSS_F32 ? 16 : 32; }
inline int stage_count(const rtoss_wdesc& d) { return (d.Ci + stage_channels(d.dt) - 1) / stage_channels(d.dt); }
// Every section ends with a block of zeros: source of the copy lanes that fill padding.
__host__ __device__ inline int zero_section_bytes(int stages) { return (64 * stages + 16 + 255) / 256 * 256; }

// ---- 3x3, one dense step per tap: blocks of 4 channel tiles, [stage][block][tile][tap][lane] ----
constexpr int kDenseTileBytes = 9 * kFragBytes;
inline int dense_channel_blocks(int Co) { return (Co + 63) / 64; }

// ---- 1x1, streaming kernel: [channel block][wave slice][fragment][stage][lane] ----
constexpr int stream_mt_of(int KS) { return KS <= 8 ? 4 : (KS == 16 ? 2 : 1); }  // fragments per wave along output channels
inline int stream_wm_of(int KS, int Co)                                           // waves along output channels
{
    const int tiles = (Co + 15) / 16, groups = (tiles + stream_mt_of(KS) - 1) / stream_mt_of(KS);
    const int by_channels = groups >= 3 ? 4 : groups;  // 1, 2 or 4
    // deep layers: fewer waves along positions, so that a buffer (16 positions per such wave x Ci) stays <= 32 KB
    const int by_depth = KS >= 32 ? 4 : (KS == 16 ? 2 : 1);
    return by_channels > by_depth ? by_channels : by_depth;
}
inline int stream_co_blocks_of(int KS, int Co)
{
    const int span = 16 * stream_mt_of(KS) * stream_wm_of(KS, Co);
    return (Co + span - 1) / span;
}

// ---- 1x1, ring kernel: [stage][channel tile, padded to 8][lane] ----
inline int ring_padded_tiles(int Co) { return ((Co + 15) / 16 + 7) / 8 * 8; }

}  // namespace rtoss
