// Every word the image stem reads lies inside its tensor (csrc/stem_rows.h), for small images, both strides and all tiles, and the
// words cover the tile's part of every row.  Prints the calls looked at; the first one that is wrong ends it with status 1.
#define __host__
#define __device__
#include "stem_rows.h"

#include <algorithm>
#include <cstdio>

int main()
{
    long rows = 0, cut = 0;
    for (int S = 1; S <= 2; ++S)
        for (int Ci = 1; Ci <= 3; ++Ci)
            for (int N = 1; N <= 3; ++N)
                for (int H = 1; H <= 5; ++H)
                    for (int W = 1; W <= 140; ++W) {
                        const int64_t total = (int64_t)N * H * W * Ci;
                        if (total == 1) continue;  // (another kernel's)
                        const int Wo = (W - 1) / S + 1, IW = 31 * S + 3;
                        for (int n = 0; n < N; ++n)
                            for (int h = 0; h < H; ++h)
                                for (int ow0 = 0; ow0 < Wo; ow0 += 32) {
                                    const int iw0 = ow0 * S - 1, lo = iw0 < 0 ? Ci : 0, hi = std::min(IW, W - iw0) * Ci;
                                    const int64_t at = (((int64_t)n * H + h) * W + iw0) * Ci;
                                    const bool is_cut = total % 2 && n == N - 1 && h == H - 1 && W - iw0 <= IW;
                                    const rtoss::StemRow row((int)at & 1, lo, hi, is_cut);
                                    const int end = row.last + is_cut;  // the cut word is read by itself
                                    bool ok = 2 * row.first <= lo + row.odd && 2 * end + 1 >= hi - 1 + row.odd;
                                    for (int i = 0; i < 256; ++i) {
                                        const int64_t half = at - row.odd + 2 * row.word(i);
                                        ok = ok && half >= 0 && half % 2 == 0 && half + 1 < total;
                                        ok = ok && (i < row.first || i > row.last || row.word(i) == i);
                                    }
                                    if (is_cut) ok = ok && at + hi == total;
                                    ++rows, cut += is_cut;
                                    if (!ok) {
                                        printf("stride %d Ci %d N %d H %d W %d: image %d row %d column %d\n", S, Ci, N, H, W, n, h, iw0);
                                        return 1;
                                    }
                                }
                    }
    printf("%ld rows, %ld whose last word is cut\n", rows, cut);
    return 0;
}
