// Rows of the image stem's input tile as aligned 4-byte words (conv3x3_stem.hip).
#pragma once
#include <stdint.h>

namespace rtoss {

// A row of the tile begins at half number `at` of a tensor of more than one half (in front of it where the tile hangs over the left edge of
// the image); its halves [lo, hi) lie inside the image.  Word i of the row is halves 2i and 2i + 1 from at - odd on, odd = at & 1.
// cut: half hi - 1 is the tensor's last, and the lower one of its word: the word ends behind the tensor and is left out.
struct StemRow {
    int odd;
    int first, last;  // the words with halves of [lo, hi); a word of the row before where the cut one is the only one
    __host__ __device__ StemRow(int odd, int lo, int hi, bool cut) : odd(odd), first((lo + odd) / 2), last((hi - 1 + odd) / 2 - cut) {}
    __host__ __device__ int word(int i) const  // the nearest one to word i
    {
        const int from = i < first ? first : i;
        return from > last ? last : from;
    }
};

}  // namespace rtoss
