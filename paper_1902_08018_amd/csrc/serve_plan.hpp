// serve_plan.hpp -- the launch plans behind a serving slot's graphs and the
// workspace the graphs share, with no device calls.  serve.hip sizes a slot
// and captures its graphs through these functions alone, so that no graph's
// plan can need more than the slot holds; the host tests run them too.
#pragma once

#include <algorithm>
#include <utility>
#include <vector>

#include "../../include/wh.h"
#include "serve_policy.hpp"
#include "wh_internal.hpp"

namespace wh {

// The plan of the graph for k right-hand sides over rows [chunk.first,
// chunk.second), and the doubles of workspace its launches use: FP64 slab
// partials, and B^T U for the multi-RHS kernel.
struct ServePlan {
    GemvPlan plan;
    size_t workspace;
};

// The workspace (doubles) of a matrix's slot.  Its graphs run one after
// another (one launch stream), so they share it.
inline size_t serve_workspace(const wh_matrix_desc& d, const std::vector<std::pair<uint32_t, uint32_t>>& chunks,
                              int num_cus, const GemvTuning& tune)
{
    size_t n = 0;
    for (const auto& c : chunks)
        n = std::max(n, whz_serve_workspace(d.rate, d.cols, c.first, c.second, num_cus, &tune));
    return n;
}

// A graph's plan within a slot's workspace.  The slab count the planner likes
// best depends on k in either direction (fewer right-hand sides make partials
// cheaper), so every bucket's plan is held to the workspace on its own.
inline ServePlan serve_plan(const wh_matrix_desc& d, const std::pair<uint32_t, uint32_t>& chunk, uint32_t k,
                            int num_cus, const GemvTuning& tune, size_t workspace)
{
    if (k == 1) { // as without launch-shape overrides, which are wh_gemv's
        const GemvPlan pl =
            whz_gemv_plan(d.rate, d.rows, d.cols, chunk.first, chunk.second, num_cus, nullptr, workspace);
        return ServePlan{pl, pl.nslab > 1 ? (size_t)pl.nslab * pl.part_rows() : 0};
    }
    const MrhsPlan pl =
        whz_mrhs_plan(d.rate, d.rows, d.cols, chunk.first, chunk.second, num_cus, k, false, &tune, workspace);
    return ServePlan{pl, mrhs_workspace(pl, k).total};
}

} // namespace wh
