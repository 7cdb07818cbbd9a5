// How the pipelined 3x3 kernels' strips of output rows are cut into tiles (host side; rows_plan.h has the kernels').
#pragma once
#include <algorithm>
#include <cstdint>

namespace rtoss {

constexpr int kTall = 5, kShort = 4;  // output rows per wave of the two tile classes

// How the rows of the strips are cut into tiles, and how the tiles are dealt to the workgroups.
// A strip is 16 output columns of one image.  Strips [0, sa) are cut into a5 tall tiles followed by a4
// short ones, the other strips into b5 tall and b4 short.  A list entry is (tile, channel block) with the
// channel block fastest; each class has its own list, cut into 8 contiguous ranges, one per XCD, so that
// the channel blocks of a tile, and neighbouring tiles, meet in one L2.
struct RowPlan {
    int col_strips, co_blocks, strips;
    int sa, a5, a4, b5, b4;
    int tall_total, tall_per_xcd, short_total, short_per_xcd;
};

// Relative cost of one tile of TN rows per wave over `stages` stages: a stage costs a fixed part (weight
// operand reads, hand-over) plus a part per row; the epilogue and the prologue of a tile scale with its
// rows.  (Fitted to per-workgroup time stamps of both tile classes on a 256 -> 256 channel layer.)
inline double tile_cost(int tn, int stages) { return stages * (tn + 0.7) + 1.5 * tn; }

// The busiest workgroup's cost under a plan, by the kernel's own dealing rule.  An XCD's slots hold one of two numbers of each class: the
// larger number of tall tiles at the first slots, of short ones at the last.
inline double plan_cost(const RowPlan& p, int slots, int stages)
{
    const double c5 = tile_cost(kTall, stages), c4 = tile_cost(kShort, stages);
    double worst = 0;
    for (int xcd = 0; xcd < 8; ++xcd) {
        const int nt = std::max(0, std::min((xcd + 1) * p.tall_per_xcd, p.tall_total) - xcd * p.tall_per_xcd);
        const int ns = std::max(0, std::min((xcd + 1) * p.short_per_xcd, p.short_total) - xcd * p.short_per_xcd);
        const int qt = nt / slots, qs = ns / slots, more_t = nt % slots, more_s = ns % slots;
        const bool both = more_t + more_s > slots;  // a slot with the larger number of both
        if (more_t > 0) worst = std::max(worst, (qt + 1) * c5 + (qs + both) * c4);
        if (more_s > 0) worst = std::max(worst, (qt + both) * c5 + (qs + 1) * c4);
        worst = std::max(worst, qt * c5 + qs * c4);
    }
    return worst;
}

inline RowPlan make_plan(int N, int H, int W, int co_blocks, int sa, int a5, int a4, int b5, int b4)
{
    RowPlan p;
    p.col_strips = (W + 15) / 16;
    p.co_blocks = co_blocks;
    p.strips = N * p.col_strips;
    p.sa = sa;
    p.a5 = a5;
    p.a4 = a4;
    p.b5 = b5;
    p.b4 = b4;
    p.tall_total = (sa * a5 + (p.strips - sa) * b5) * co_blocks;
    p.short_total = (sa * a4 + (p.strips - sa) * b4) * co_blocks;
    p.tall_per_xcd = (p.tall_total + 7) / 8;
    p.short_per_xcd = (p.short_total + 7) / 8;
    return p;
}

// Searches the cuts (n5 tall + n4 short tiles covering H rows with no tile to spare) for the two strip classes and the number of strips of
// the first class.  It runs in front of a shape's first launch, so pairs of cuts that could not be cheaper even with their tiles spread
// evenly are passed over (1x640x640 24 ms, now none; 1x1080x1920 200 ms, 0.9; 2x100x168 0.5, 0.02; the same plans), and it ends after
// kCutLimit candidates, a few milliseconds, which takes images of thousands of rows.
constexpr int kCutLimit = 1 << 16;
inline RowPlan cut_rows(int N, int H, int W, int co_blocks, int stages, int slots, double* cost)
{
    const int all = (int)(((int64_t)H + 4 * kTall - 1) / (4 * kTall)), strips = N * ((W + 15) / 16);
    const auto shorts = [&](int n5) { return (int)std::max<int64_t>(0, (H - (int64_t)n5 * 4 * kTall + 4 * kShort - 1) / (4 * kShort)); };
    const double c5 = tile_cost(kTall, stages), c4 = tile_cost(kShort, stages);
    const auto even = [&](int n5) { return (double)strips * co_blocks / (8 * slots) * (n5 * c5 + shorts(n5) * c4); };
    RowPlan best = make_plan(N, H, W, co_blocks, 0, 0, 0, all, 0);
    double best_cost = plan_cost(best, slots, stages);
    const int step = std::max(1, strips / 64);  // candidate numbers of strips: all of them when the list is short, else a coarse scan
    int left = kCutLimit;
    for (int a = 0; a <= all; ++a)
        for (int b = a; b <= all; ++b) {
            if (--left <= 0) break;
            if (std::min(even(a), even(b)) >= 1.000001 * best_cost) continue;  // (the sums round)
            for (int sa = a == b ? strips : 0; sa <= strips; sa += step, --left) {
                const RowPlan p = make_plan(N, H, W, co_blocks, sa, a, shorts(a), b, shorts(b));
                const double c = plan_cost(p, slots, stages);
                if (c < best_cost) best_cost = c, best = p;
            }
        }
    *cost = best_cost;
    return best;
}

}  // namespace rtoss
