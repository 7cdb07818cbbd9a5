// 3x3 stride-1 pattern-sparse convolution for large layers: the cut of the rows into tiles, and the pipelined kernel (rows_kernel.h) for
// layout 0.  (Layout 1: conv3x3_rows_groups.hip, compiled beside this one.)
#include <algorithm>
#include <map>
#include <mutex>
#include <tuple>
#include <vector>

#include "rows_kernel.h"

namespace rtoss {

// ---------------------------------------------------------------------------------------------------------
// Host: cutting the rows into tiles.
// ---------------------------------------------------------------------------------------------------------
// Relative cost of one tile of TN rows per wave over `stages` stages: a stage costs a fixed part (weight
// operand reads, hand-over) plus a part per row; the epilogue and the prologue of a tile scale with its
// rows.  (Fitted to per-workgroup time stamps of both tile classes on a 256 -> 256 channel layer.)
namespace {

inline double tile_cost(int tn, int stages) { return stages * (tn + 0.7) + 1.5 * tn; }

struct PlanKey {
    int N, H, W, co_blocks, stages, slots;
    bool operator<(const PlanKey& o) const
    {
        return std::tie(N, H, W, co_blocks, stages, slots) < std::tie(o.N, o.H, o.W, o.co_blocks, o.stages, o.slots);
    }
};

// The busiest workgroup's cost under a plan, by the kernel's own dealing rule.
double plan_makespan(const RowPlan& p, int slots, int stages)
{
    const double c5 = tile_cost(kTall, stages), c4 = tile_cost(kShort, stages);
    double worst = 0;
    for (int xcd = 0; xcd < 8; ++xcd) {
        const int nt = std::max(0, std::min((xcd + 1) * p.tall_per_xcd, p.tall_total) - xcd * p.tall_per_xcd);
        const int ns = std::max(0, std::min((xcd + 1) * p.short_per_xcd, p.short_total) - xcd * p.short_per_xcd);
        for (int s = 0; s < slots; ++s) {
            const int mine_t = nt > s ? (nt - s + slots - 1) / slots : 0;
            const int rs = slots - 1 - s;
            const int mine_s = ns > rs ? (ns - rs + slots - 1) / slots : 0;
            worst = std::max(worst, mine_t * c5 + mine_s * c4);
        }
    }
    return worst;
}

RowPlan make_plan(int N, int H, int W, int co_blocks, int sa, int a5, int a4, int b5, int b4)
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

}  // namespace

// Searches the cuts (n5 tall + n4 short tiles covering H rows with no tile to spare) for the two strip
// classes and the number of strips of the first class; results are remembered per launch shape.
RowPlan plan_rows(int N, int H, int W, int co_blocks, int stages, int slots, double* cost)
{
    static std::mutex mu;
    static std::map<PlanKey, std::pair<RowPlan, double>> cache;
    const PlanKey key{N, H, W, co_blocks, stages, slots};
    {
        std::lock_guard<std::mutex> lock(mu);
        auto it = cache.find(key);
        if (it != cache.end()) {
            if (cost) *cost = it->second.second;
            return it->second.first;
        }
    }
    struct Cut {
        int n5, n4;
    };
    std::vector<Cut> cuts;
    for (int n5 = 0; n5 * 4 * kTall < H + 4 * kTall; ++n5) {
        const int rest = H - n5 * 4 * kTall;
        cuts.push_back(Cut{n5, rest > 0 ? (rest + 4 * kShort - 1) / (4 * kShort) : 0});
        if (rest <= 0) break;
    }
    const int strips = N * ((W + 15) / 16);
    RowPlan best = make_plan(N, H, W, co_blocks, 0, 0, 0, cuts.back().n5, cuts.back().n4);
    double best_cost = plan_makespan(best, slots, stages);
    for (const Cut& a : cuts)
        for (const Cut& b : cuts) {
            if (&a > &b) continue;
            // candidate numbers of first-class strips: all of them when the list is short, else a coarse scan
            const int step = std::max(1, strips / 64);
            for (int sa = (&a == &b ? strips : 0); sa <= strips; sa += step) {
                const RowPlan p = make_plan(N, H, W, co_blocks, sa, a.n5, a.n4, b.n5, b.n4);
                const double c = plan_makespan(p, slots, stages);
                if (c < best_cost) {
                    best_cost = c;
                    best = p;
                }
            }
        }
    std::lock_guard<std::mutex> lock(mu);
    if (cache.size() > 4096) cache.clear();
    cache[key] = {best, best_cost};
    if (cost) *cost = best_cost;
    return best;
}

RowPlan plan_rows_for_device(int N, int H, int W, int co_blocks, int stages, int cus, int* slots_out, double* cost)
{
    // one workgroup per compute unit (a workgroup owns nearly all of a unit's LDS)
    const int full = std::max(8, cus) / 8;
    RowPlan plan = plan_rows(N, H, W, co_blocks, stages, full, cost);
    // (fewer entries than workgroups: launch only as many slots per XCD as the longer list needs)
    const int slots = std::max(1, std::min(full, std::max(plan.tall_per_xcd, plan.short_per_xcd)));
    if (slots != full) plan = plan_rows(N, H, W, co_blocks, stages, slots, cost);
    *slots_out = slots;
    return plan;
}

bool rows3x3_needs_fused_stage(const ConvParams& c) { return c.ep.scale || c.ep.bias || c.ep.residual || c.ep.act > 1; }

rtoss_status launch_conv3x3_rows(const rtoss_wdesc& d, const ConvParams& c, int layout, const void* section, const void* x, void* y,
                                 hipStream_t s)
{
    return layout == 1 ? launch_conv3x3_rows_groups(d, c, section, x, y, s) : launch_rows_typed<0>(d, c, section, x, y, s);
}

}  // namespace rtoss
