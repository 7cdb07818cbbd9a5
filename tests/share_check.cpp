// The ranges of a streaming 1x1 launch (csrc/share.h) cover its buffers in order, none is empty or more than one buffer longer than
// another, and where they divide into eighths (an XCD's each) no eighth has more than one buffer more than another.  Ends with
// status 1 at the first launch that is wrong.
#define __host__
#define __device__
#include "share.h"

#include <algorithm>
#include <cstdio>

int main()
{
    const int ranges[] = {1, 2, 3, 7, 8, 9, 16, 24, 31, 40, 96, 100, 128, 256, 341, 512, 768, 1024, 1536, 2048, 4096, 65528};
    for (const int n : ranges)
        for (int64_t i = 0; i < 700; ++i) {
            const int64_t buffers = i < 600 ? n + i * n / 100 + i : (int64_t)0x7fffffff - (i - 600) * 37;
            const rtoss::Share share(buffers, n);
            int64_t at = 0, eighth[8] = {};
            bool ok = true;
            for (int r = 0; r < n; ++r) {
                const rtoss::Range range = share.of(r);
                const int64_t length = (int64_t)range.end - range.first;
                ok = ok && range.first == at && (length == buffers / n || length == buffers / n + 1);
                at = range.end;
                if (n % 8 == 0) eighth[r / (n / 8)] += length;
            }
            ok = ok && at == buffers;
            if (n % 8 == 0) ok = ok && *std::max_element(eighth, eighth + 8) - *std::min_element(eighth, eighth + 8) <= 1;
            if (!ok) {
                printf("%lld buffers, %d ranges\n", (long long)buffers, n);
                return 1;
            }
        }
    return 0;
}
