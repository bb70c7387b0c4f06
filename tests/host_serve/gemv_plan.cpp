// Host driver of the fused GEMV's planner with launch-shape overrides.
//
// usage: gemv_plan <rate> <rows> <cols> <lanes> <rows per group> <slabs>
//            (0: the planner's choice); prints what the plan holds
#include "planner.hpp"

#include <cstdio>
#include <cstdlib>

int main(int argc, char** argv)
{
    if (argc != 7)
        return 2;
    uint32_t v[6];
    for (int i = 0; i < 6; ++i)
        v[i] = (uint32_t)atoi(argv[1 + i]);
    wh::GemvTuning t;
    t.lanes = v[3];
    t.rows = v[4];
    t.slabs = v[5];
    const wh::GemvPlan pl = wh::whz_gemv_plan(v[0], v[1], v[2], 0, v[1], 256, &t);
    printf("%u %u %u %u %d\n", 1u << pl.lg, pl.rpg, pl.nslab, pl.slab_bc, (int)pl.uncapturable);
    return 0;
}
