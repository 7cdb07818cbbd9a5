// The cut of a launch shape into tiles (csrc/rows_cut.h): the busiest workgroup's cost is what walking every slot's tiles gives, the chosen cut
// covers every row, no cut of a search without short cuts costs less, and images of any height take a bounded search.  Ends with status 1 at
// the first that is wrong.
#include "rows_cut.h"

#include <chrono>
#include <cstdio>
#include <random>

using namespace rtoss;

static double walked(const RowPlan& p, int slots, int stages)
{
    double worst = 0;
    for (int xcd = 0; xcd < 8; ++xcd)
        for (int s = 0; s < slots; ++s) {
            int tall = 0, low = 0;
            for (int e = xcd * p.tall_per_xcd + s; e < std::min((xcd + 1) * p.tall_per_xcd, p.tall_total); e += slots) ++tall;
            for (int e = xcd * p.short_per_xcd + slots - 1 - s; e < std::min((xcd + 1) * p.short_per_xcd, p.short_total); e += slots) ++low;
            worst = std::max(worst, tall * tile_cost(kTall, stages) + low * tile_cost(kShort, stages));
        }
    return worst;
}

static double every_cut(int N, int H, int W, int blocks, int stages, int slots)
{
    const int all = (H + 19) / 20, strips = N * ((W + 15) / 16);
    double least = 1e300;
    for (int a = 0; a <= all; ++a)
        for (int b = a; b <= all; ++b)
            for (int sa = a == b ? strips : 0; sa <= strips; sa += std::max(1, strips / 64))
                least = std::min(least, plan_cost(make_plan(N, H, W, blocks, sa, a, std::max(0, (H - 20 * a + 15) / 16), b,
                                                            std::max(0, (H - 20 * b + 15) / 16)), slots, stages));
    return least;
}

int main()
{
    std::mt19937 rng(1);
    const auto upto = [&](int n) { return (int)(rng() % n); };
    for (int i = 0; i < 20000; ++i) {
        RowPlan p{};
        p.tall_total = upto(1 << upto(13)), p.short_total = upto(1 << upto(13));
        p.tall_per_xcd = (p.tall_total + 7) / 8, p.short_per_xcd = (p.short_total + 7) / 8;
        const int slots = 1 + upto(32), stages = 3 + upto(30);
        if (plan_cost(p, slots, stages) != walked(p, slots, stages)) return printf("cost of %d %d over %d\n", p.tall_total, p.short_total, slots), 1;
    }
    for (int i = 0; i < 300; ++i) {
        const int N = 1 + upto(20), H = 1 + upto(i % 10 ? 250 : 900), W = 1 + upto(400), blocks = 1 + upto(4), stages = 3 + upto(14), slots = 1 + upto(32);
        double cost = 0;
        const RowPlan p = cut_rows(N, H, W, blocks, stages, slots, &cost);
        const bool covers = (p.sa == 0 || 20 * p.a5 + 16 * p.a4 >= H) && (p.sa == p.strips || 20 * p.b5 + 16 * p.b4 >= H);
        if (!covers || cost != plan_cost(p, slots, stages) || cost > every_cut(N, H, W, blocks, stages, slots))
            return printf("%dx%dx%d %d %d %d\n", N, H, W, blocks, stages, slots), 1;
    }
    // (the search without short cuts is quadratic in H: minutes for the first of these, hours for the last)
    const auto start = std::chrono::steady_clock::now();
    const int tall[][4] = {{1, 100000, 17, 2}, {3, 1 << 20, 9, 1}, {1, 10000000, 64, 2}, {1, 40000000, 1, 1}};
    for (const auto& t : tall) {
        double cost = 0;
        const RowPlan p = cut_rows(t[0], t[1], t[2], t[3], 3, 32, &cost);
        const double even = (double)p.strips * t[3] / 256 * (t[1] / 20.0) * tile_cost(kTall, 3);
        if (!((p.sa == 0 || 20ll * p.a5 + 16ll * p.a4 >= t[1]) && 20ll * p.b5 + 16ll * p.b4 >= t[1]) || cost > 1.05 * even + 40) return printf("%d rows: %f, %f\n", t[1], cost, even), 1;
    }
    if (std::chrono::steady_clock::now() - start > std::chrono::seconds(2)) return printf("slow\n"), 1;
    return 0;
}
