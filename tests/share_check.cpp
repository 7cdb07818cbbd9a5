// The shares of a streaming 1x1 launch (csrc/share.h) hold every buffer once, none is empty or more than one buffer longer than
// another, and where they divide into eighths (an XCD's each) no eighth has more than one buffer more than another.  Ends with
// status 1 at the first launch that is wrong.
#define __host__
#define __device__
#include "share.h"

#include <algorithm>
#include <cstdio>
#include <vector>

int main()
{
    const int shares[] = {1, 2, 3, 7, 8, 9, 16, 24, 31, 40, 96, 100, 128, 256, 341, 512, 768, 1024, 1536, 2048, 4096, 65528};
    for (const int n : shares)
        for (int64_t i = 0; i < 400; ++i) {
            const int64_t buffers = i < 300 ? n + i * n / 100 + i : (int64_t)0x7fffffff - (i - 300) * 37;
            const rtoss::Share share(buffers, n);
            int64_t eighth[8] = {};
            std::vector<bool> taken(n);
            bool ok = true;
            for (int s = 0; s < n && ok; ++s) {
                // every n-th buffer from one of the first n on, up to the last
                const rtoss::Buffers b = share.of(s);
                ok = b.step == n && b.first >= 0 && b.first < n && !taken[b.first] && b.count >= 1;
                ok = ok && b.at(b.count - 1) < buffers && b.at(b.count) >= buffers;
                if (ok) taken[b.first] = true;
                if (n % 8 == 0) eighth[s / (n / 8)] += b.count;
            }
            if (n % 8 == 0) ok = ok && *std::max_element(eighth, eighth + 8) - *std::min_element(eighth, eighth + 8) <= 1;
            if (!ok) {
                printf("%lld buffers, %d shares\n", (long long)buffers, n);
                return 1;
            }
        }
    return 0;
}
