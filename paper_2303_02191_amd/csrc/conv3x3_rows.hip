// 3x3 stride-1 pattern-sparse convolution for large layers: the cut of the rows into tiles, and the pipelined kernel (rows_kernel.h) for
// layout 0.  (Layout 1: conv3x3_rows_groups.hip, compiled beside this one.)
#include <algorithm>
#include <map>
#include <mutex>
#include <new>
#include <tuple>

#include "rows_kernel.h"

namespace rtoss {

namespace {

struct PlanKey {
    int N, H, W, co_blocks, stages, slots;
    bool operator<(const PlanKey& o) const
    {
        return std::tie(N, H, W, co_blocks, stages, slots) < std::tie(o.N, o.H, o.W, o.co_blocks, o.stages, o.slots);
    }
};

}  // namespace

// (results are remembered per launch shape)
RowsLaunch plan_rows_for_device(int N, int H, int W, int Co, int stages, int cus)
{
    static std::mutex mu;
    static std::map<PlanKey, RowsLaunch> cache;
    // one workgroup per compute unit (a workgroup owns nearly all of a unit's LDS)
    const int co_blocks = ((Co + 15) / 16 + kRowsTM - 1) / kRowsTM, full = std::max(8, cus) / 8;
    const PlanKey key{N, H, W, co_blocks, stages, full};
    {
        std::lock_guard<std::mutex> lock(mu);
        auto it = cache.find(key);
        if (it != cache.end()) return it->second;
    }
    RowsLaunch r;
    r.plan = cut_rows(N, H, W, co_blocks, stages, full, &r.cost);
    // (fewer entries than workgroups: launch only as many slots per XCD as the longer list needs)
    r.slots = std::max(1, std::min(full, std::max(r.plan.tall_per_xcd, r.plan.short_per_xcd)));
    if (r.slots != full) r.plan = cut_rows(N, H, W, co_blocks, stages, r.slots, &r.cost);
    std::lock_guard<std::mutex> lock(mu);
    try {
        if (cache.size() > 4096) cache.clear();
        cache[key] = r;
    } catch (const std::bad_alloc&) {  // (not remembered: nothing may leave the C interface)
    }
    return r;
}

bool rows3x3_needs_fused_stage(const ConvParams& c) { return c.ep.scale || c.ep.bias || c.ep.residual || c.ep.act > 1; }

rtoss_status launch_conv3x3_rows(const rtoss_wdesc& d, const ConvParams& c, int layout, const RowsLaunch* planned, const void* section,
                                 const void* x, void* y, hipStream_t s)
{
    return layout == 1 ? launch_conv3x3_rows_groups(d, c, planned, section, x, y, s) : launch_rows_typed<0>(d, c, planned, section, x, y, s);
}

}  // namespace rtoss
