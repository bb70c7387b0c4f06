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

inline ServePlan serve_plan(const wh_matrix_desc& d, const std::pair<uint32_t, uint32_t>& chunk, uint32_t k,
                            int num_cus, const GemvTuning& tune)
{
    if (k == 1) {
        const GemvPlan pl = whz_gemv_plan(d.rate, d.rows, d.cols, chunk.first, chunk.second, num_cus);
        return ServePlan{pl, pl.nslab > 1 ? (size_t)pl.nslab * pl.part_rows() : 0};
    }
    const MrhsPlan pl =
        whz_mrhs_plan(d.rate, d.rows, d.cols, chunk.first, chunk.second, num_cus, k, false, &tune);
    return ServePlan{pl, mrhs_workspace(pl, k).total};
}

// The workspace (doubles) of a matrix's slot: the most any of its graphs
// uses.  Graphs run one after another (one launch stream), so they share it.
// The slab count depends on k in either direction (fewer right-hand sides
// make partials cheaper), so no bucket stands for another.
inline size_t serve_workspace(const wh_matrix_desc& d, const std::vector<std::pair<uint32_t, uint32_t>>& chunks,
                              int num_cus, const GemvTuning& tune)
{
    size_t n = 0;
    for (const auto& c : chunks)
        for (uint32_t k : policy::kBuckets)
            n = std::max(n, serve_plan(d, c, k, num_cus, tune).workspace);
    return n;
}

} // namespace wh
