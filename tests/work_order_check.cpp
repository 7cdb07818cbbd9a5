// Divisor against the division: every divisor up to 3000 and around powers of two, dividends around their multiples and at both ends of the range; and
// tiles of every item of small launches, each once.  Prints the number of differences.
#include <cstdio>
#include <set>
#include <tuple>
#include <vector>

#define __host__
#define __device__
static struct { unsigned x; } blockIdx;
#include "work_order.h"

int main()
{
    long wrong = 0;
    std::vector<int> divisors;
    for (int d = 1; d <= 3000; ++d) divisors.push_back(d);
    for (int s = 12; s < 31; ++s)
        for (int e = -2; e <= 2; ++e) divisors.push_back((1 << s) + e);
    divisors.push_back(0x7fffffff);
    for (const int d : divisors) {
        const rtoss::Divisor by(d);
        const auto check = [&](int64_t n) {
            if (n < 0 || n > 0x7fffffff) return;
            const int q = by.quotient((int)n);
            wrong += q != (int)(n / d) || by.remainder((int)n, q) != (int)(n % d);
        };
        const int64_t last = 0x7fffffff / d;
        for (int64_t m = 0; m <= last; m += 1 + last / 2000)
            for (int e = -1; e <= 1; ++e) check(m * d + e);
        for (int e = -1; e <= 1; ++e) check(last * d + e);
        check(0x7fffffff);
    }
    for (int images = 1; images <= 5; ++images)
        for (int rows = 1; rows <= 9; ++rows)
            for (int across = 1; across <= 11; ++across) {
                const rtoss::WorkOrder order((int64_t)images * rows * across, 1, rows * across, across);
                std::set<std::tuple<int, int, int>> seen;
                for (int n = 0; n < order.total; ++n) {
                    const auto t = order.tile(n);
                    wrong += t.n_img >= images || t.row >= rows || t.col >= across || t.n_img < 0 || t.row < 0 || t.col < 0;
                    seen.insert({t.n_img, t.row, t.col});
                }
                wrong += (int)seen.size() != order.total || order.grid() < (unsigned)order.total;
            }
    printf("%ld\n", wrong);
    return wrong != 0;
}
