// whz_dispatch.hip -- rate dispatch and launch planning for the WHZ1 kernels.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "../../include/wh.h"
#include "wh_internal.hpp"

#define WH_FOR_EACH_NW(X) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(10) X(12) X(16)

namespace wh {

#define X(k)                                                                                                         \
    namespace nw##k {                                                                                                \
    hipError_t decode_blocks(const void*, uint64_t, uint64_t, float*, hipStream_t);                                  \
    hipError_t decode_matrix(const void*, uint32_t, uint32_t, float*, hipStream_t);                                  \
    hipError_t encode(const float*, uint32_t, uint32_t, void*, uint32_t*, hipStream_t);                              \
    hipError_t gemv(const GemvPlan&, AccMode, const void*, const float*, float*, double*, hipStream_t);              \
    hipError_t mrhs(const MrhsPlan&, const void*, const void*, uint32_t, uint32_t, float*, uint32_t, double*,           \
                    hipStream_t);                                                                                      \
    }
WH_FOR_EACH_NW(X)
#undef X

bool whz_rate_supported(uint32_t rate)
{
    if (rate % 2)
        return false;
    switch (rate / 2) {
#define X(nw) case nw:
        WH_FOR_EACH_NW(X)
#undef X
        return true;
    default:
        return false;
    }
}

hipError_t whz_decode_blocks(uint32_t rate, const void* stream, uint64_t b0, uint64_t n, float* out, hipStream_t st)
{
    switch (rate / 2) {
#define X(k)                                                                                                         \
    case k:                                                                                                          \
        return nw##k::decode_blocks(stream, b0, n, out, st);
        WH_FOR_EACH_NW(X)
#undef X
    default:
        return hipErrorInvalidValue;
    }
}

hipError_t whz_decode_matrix(uint32_t rate, const void* stream, uint32_t rows, uint32_t cols, float* out,
                             hipStream_t st)
{
    switch (rate / 2) {
#define X(k)                                                                                                         \
    case k:                                                                                                          \
        return nw##k::decode_matrix(stream, rows, cols, out, st);
        WH_FOR_EACH_NW(X)
#undef X
    default:
        return hipErrorInvalidValue;
    }
}

hipError_t whz_encode(uint32_t rate, const float* M, uint32_t rows, uint32_t cols, void* stream, uint32_t* bad,
                      hipStream_t st)
{
    switch (rate / 2) {
#define X(k)                                                                                                         \
    case k:                                                                                                          \
        return nw##k::encode(M, rows, cols, stream, bad, st);
        WH_FOR_EACH_NW(X)
#undef X
    default:
        return hipErrorInvalidValue;
    }
}

namespace {

uint32_t ceil_div(uint64_t a, uint64_t b) { return (uint32_t)((a + b - 1) / b); }

GemvPlan range_plan(uint32_t cols, uint32_t row_begin, uint32_t row_end)
{
    GemvPlan pl{};
    pl.nbc = (cols + 3) / 4;
    pl.bi_begin = row_begin / 4;
    pl.bi_end = (row_end + 3) / 4;
    pl.cols = cols;
    pl.nrows = row_end - row_begin;
    pl.skip = row_begin & 3u;
    return pl;
}

// Slab width for `nslab` slabs of whole groups of `width` block columns;
// returns the slab count that width gives.
uint32_t set_slabs(GemvPlan& pl, uint32_t nslab, uint32_t width)
{
    uint32_t slab_bc = ceil_div(pl.nbc, nslab ? nslab : 1);
    slab_bc = ceil_div(slab_bc, width) * width;
    pl.slab_bc = slab_bc ? slab_bc : width;
    pl.nslab = ceil_div(pl.nbc, pl.slab_bc);
    if (pl.nslab < 1)
        pl.nslab = 1;
    return pl.nslab;
}

} // namespace

// Launch shape of the fused GEMV, chosen from sweeps of every shape over
// matrices from 378 x 256000 to 65536^2 on MI355X:
//  * 8 lanes per block row (14 % faster than 512 on 65536^2).  A wave then
//    decodes an 8 x 8 patch of blocks instead of 64 blocks of one row, and a
//    workgroup's slab of u is small and reused by its 64 block rows.  Wider
//    groups only where a tile of 512 / G block rows would be mostly empty
//    (few rows); narrower where a row has fewer than 8 block columns.
//  * One block row per group and tile.
//  * Column slabs of 1 to 16 blocks per lane and row, by gemv_shape_cost (the
//    fixed rule's below where gemv_rounds_cost favours them); or
//    no slabs, with groups wide enough to take a whole block row at a block a
//    lane, where that costs less (up to 1024 columns: no partial sums, no
//    second kernel, no ordering of the workspace's users; 256 x 1024 at rate
//    16 16.3 -> 10.9 us).  Past
//    2^27 blocks, about 8192 workgroups of up to 48 blocks per lane, which
//    keeps the FP64 partial sums small (the times differ by under 1 % there).
namespace {

// Column slabs by a fixed rule: about 2048 workgroups of 3 to 16 blocks per
// lane, and past 2^27 blocks about 8192 of up to 48.
uint32_t split_slabs(uint64_t blocks, uint32_t nbc, uint32_t lanes, uint32_t G)
{
    uint64_t iters = std::min<uint64_t>(16, std::max<uint64_t>(3, (blocks + (uint64_t)lanes * 1024) / ((uint64_t)lanes * 2048)));
    if (blocks > (1ull << 27))
        iters = std::min<uint64_t>(48, blocks / ((uint64_t)lanes * 8192));
    return ceil_div(nbc, (uint64_t)G * iters);
}

// log2 of the narrowest groups, from 8 lanes (fewer where a row has fewer block
// columns), whose tiles are at least 90 % full.
uint32_t patch_group(uint32_t nbr, uint32_t nbc, uint32_t lanes)
{
    uint32_t lg = 3;
    while (lg > 2 && (1u << lg) > nbc)
        --lg;
    for (;;) {
        const uint64_t tile = lanes >> lg;
        const uint64_t span = (uint64_t)ceil_div(nbr, tile) * tile;
        if (lg >= gemv_max_lg(lanes) || 10 * (uint64_t)nbr >= 9 * span)
            return lg;
        ++lg;
    }
}

// log2 of the groups a WH_GEMV_LANES value asks for.
uint32_t group_of(uint32_t group_lanes, uint32_t lanes)
{
    uint32_t lg = 2;
    while ((1u << lg) < group_lanes && lg < gemv_max_lg(lanes))
        ++lg;
    return lg;
}

// The workgroup lanes that rule counts with.
uint32_t rule_lanes(uint32_t rate) { return rate <= 16 ? 1024u : 768u; }

// The slabs that rule gives, under launch-shape overrides (`tune` may be null)
// the ones they ask for.  Where it splits the columns, calls use the context's
// workspace and are not captured into graphs, whatever the plan's own slabs
// are; where it does not, the plan has one slab.
uint32_t rule_slabs(uint32_t rate, uint32_t nbr, uint32_t nbc, const GemvTuning* tune)
{
    const uint32_t lanes = rule_lanes(rate);
    uint32_t lg = patch_group(nbr, nbc, lanes);
    if (tune && tune->lanes)
        lg = group_of(tune->lanes, lanes);
    uint32_t nslab = split_slabs((uint64_t)nbr * nbc, nbc, lanes, 1u << lg);
    if (tune && tune->slabs)
        nslab = std::min(tune->slabs, ceil_div(nbc, 1u << lg));
    GemvPlan pl{};
    pl.nbc = nbc;
    return set_slabs(pl, nslab, 1u << lg);
}

// Whether a plan's partial sums fit `most` doubles.
bool fits_partials(uint32_t nslab, uint32_t nbr, uint64_t most) { return nslab <= 1 || (uint64_t)nslab * nbr * 4 <= most; }

// The slab partials' price in the unit of gemv_shape_cost: the reduce kernel
// (4 us) and ordering the workspace's users (3 us).
constexpr double kSlabReduceCost = 1.2;

// What a block costs in a wave that takes 2^lg block columns of each of its
// rows, against 8: neighbouring blocks in two dimensions need more alike
// numbers of planes and lookups (65536^2: 16 lanes 2 %, 64 and more 14 %).
// Wider groups are taken for a clear gain only: 6 % on top of that.
double row_group_cost(uint32_t lg)
{
    return lg <= 3 ? 1.0 : (lg == 4 ? 1.02 : (lg == 5 ? 1.06 : 1.14)) * 1.06;
}

// What a launch of `wgs` workgroups with `iters` blocks a lane takes, in the
// time of one block a lane at two workgroups a CU (`resident` = 2 x the CUs).
// A workgroup costs its blocks and 0.8 of one for its start (section table,
// slab of u, sums).  The last workgroups run in a device that empties, about
// 0.3 of their blocks; and a launch is never shorter than its longest
// workgroup, whose blocks take two thirds of the time with the CU to itself.
// Measured against full sweeps (us): 4096^2 at rate 8 with 1024 / 512 / 344 /
// 256 workgroups (1 to 4 blocks) 29.7 / 26.4 / 32.3 / 26.7, the 378 x 256000
// slit with 3 / 4 / 6 / 8 / 12 blocks 87.4 / 83.0 / 84.2 / 86.3 / 90.0, 10000^2
// with 3 / 4 / 5 / 6 / 8 blocks 108.3 / 106.7 / 101.7 / 107.2 / 110.8, and
// 256 x 1024 at rate 16 with 1 / 3 blocks 16.3 / 26.1.
double gemv_shape_cost(uint32_t wgs, uint32_t iters, uint32_t resident)
{
    const double start = 0.8;
    const double work = (double)wgs / resident * (start + iters) + 0.3 * iters;
    const double longest = start + iters * (2 * wgs <= resident ? 2.0 / 3.0 : 1.0);
    return std::max(work, longest);
}

// The same with rounds, where the columns are split: a workgroup's start costs
// 1.2 blocks (2.4 where a CU holds one workgroup), a last round of at most one
// workgroup a CU half of a full round (0.6 in workgroups of 12 waves) and less
// the fewer they are, a fuller last round all of it; a tenth of the time goes as
// if rounds had no edges.  The cost above alone gave some shapes up to 27 % more
// time than the rule's slabs take (us, its choice and the rule's: 241 x 45201 at
// rate 4 28.4 / 22.4, 188 x 54946 at rate 6 25.1 / 20.5, 52783 x 627 at rate 16
// 52.6 / 44.9).  Where this one says that the rule's are 1 % cheaper they stand:
// of 576 swept shapes (2^14 to 2^29 values, every rate, smooth and random data)
// none is then more than 8 % slower than with the rule.  How much blocks of a
// wave differ is not known here, and a few smooth matrices would do better with
// the choice (143 x 53955 at rate 14: 25.1 us, the rule's 29.8).
double gemv_rounds_cost(uint64_t wgs, uint32_t iters, uint32_t lanes, uint32_t num_cus, uint32_t per_cu)
{
    const uint64_t resident = (uint64_t)per_cu * num_cus, full = wgs / resident, rest = wgs % resident;
    const double start = per_cu == 2 ? 1.2 : 2.4, alone = per_cu == 1 ? 1.0 : (lanes == 768u ? 0.6 : 0.5);
    double last = rest == 0 ? 0.0 : 1.0;
    if (rest > 0 && rest <= num_cus)
        last = alone * (full ? 0.75 + 0.25 * (double)rest / num_cus : 1.0);
    return (0.9 * ((double)full + last) + 0.1 * (double)wgs / (double)resident + 0.4) * (start + iters);
}
constexpr double kSlabReduceRounds = 1.7; // the slab partials' price in its unit

// A slab whose B^T u does not fit a workgroup's LDS makes it at every block:
// about 5 % (the kernel's kSlabVectors).
double slab_width_cost(uint64_t slab_bc, uint32_t rate) { return slab_bc > gemv_slab_vectors(rate) ? 1.05 : 1.0; }

} // namespace

GemvPlan whz_gemv_plan(uint32_t rate, uint32_t rows, uint32_t cols, uint32_t row_begin, uint32_t row_end,
                       int num_cus, const GemvTuning* tune, size_t most_workspace)
{
    (void)rows;
    GemvPlan pl = range_plan(cols, row_begin, row_end);
    const uint64_t most = std::min<uint64_t>(most_workspace, WH_NOALLOC_SCRATCH_BYTES / sizeof(double));
    const uint32_t lanes = gemv_wg_lanes(rate), max_lg = gemv_max_lg(lanes);
    pl.lanes = lanes;
    const uint32_t nbr = pl.bi_end - pl.bi_begin;
    uint32_t lg = patch_group(nbr, pl.nbc, lanes);
    const uint32_t by_rule = rule_slabs(rate, nbr, pl.nbc, nullptr);
    pl.uncapturable = rule_slabs(rate, nbr, pl.nbc, tune) > 1;
    const uint64_t blocks = (uint64_t)nbr * pl.nbc;
    const uint32_t per_cu = rate > 24 ? 1u : 2u; // workgroups (gemv_wg_lanes)
    const uint32_t cus = num_cus > 0 ? (uint32_t)num_cus : 256u, resident = per_cu * cus;
    uint32_t rpg = 1, per_lane = 0; // blocks a lane and row; 0: not chosen yet
    if (tune && tune->lanes) {
        lg = group_of(tune->lanes, lanes);
    } else if (!(tune && (tune->rows || tune->slabs)) && blocks <= (1ull << 27) && fits_partials(by_rule, nbr, most)) {
        // (the choice below keeps to plans that fit where the rule's does, so
        // wh_gemv_noalloc takes and refuses the calls that it would with it)
        double best = 1e300;
        if (pl.uncapturable) {
            for (uint32_t it = 1; it <= 16; ++it) {
                const uint32_t nslab = ceil_div(pl.nbc, ((uint64_t)it) << lg);
                if (!fits_partials(nslab, nbr, most))
                    continue;
                const double cost = gemv_shape_cost(ceil_div(nbr, lanes >> lg) * nslab, it, resident) *
                                        slab_width_cost((uint64_t)it << lg, rate) +
                                    (nslab > 1 ? kSlabReduceCost : 0.0);
                if (cost < best) {
                    best = cost;
                    per_lane = it;
                }
            }
        }
        const uint32_t patch_lg = lg;
        for (uint32_t g = patch_lg; g <= max_lg; ++g) { // one slab: the group takes whole block rows
            const uint32_t it = ceil_div(pl.nbc, 1u << g);
            if (pl.uncapturable && (g > patch_lg ? it > 1 || g > 8 : it > 16))
                // A block a lane, four waves: with 256 x 2048 and larger a call
                // keeps its workspace, which callers and tests of its sharing
                // count on.  The times cross further out (us, one slab of two
                // blocks a lane and the plan taken: 4096^2 at rate 16 28.6 /
                // 32.1, 50818 x 231 at rate 12 22.0 / 26.4)
                continue;
            const double cost = gemv_shape_cost(ceil_div(nbr, lanes >> g), it, resident) * row_group_cost(g);
            if (cost < best) {
                best = cost;
                per_lane = it;
                lg = g;
            }
        }
        if (pl.uncapturable && per_lane && lg == patch_lg) {
            GemvPlan ruled = pl;
            const uint32_t rule_n =
                set_slabs(ruled, split_slabs(blocks, pl.nbc, rule_lanes(rate), 1u << lg), 1u << lg);
            const uint32_t rule_it = ruled.slab_bc >> lg, n = ceil_div(pl.nbc, (uint64_t)per_lane << lg);
            const uint32_t tiles = ceil_div(nbr, lanes >> lg);
            const auto rounds = [&](uint32_t nslab, uint32_t it) {
                return gemv_rounds_cost((uint64_t)tiles * nslab, it, lanes, cus, per_cu) *
                           slab_width_cost((uint64_t)it << lg, rate) +
                       (nslab > 1 ? kSlabReduceRounds : 0.0);
            };
            if (n > 1 && fits_partials(rule_n, nbr, most) && rounds(rule_n, rule_it) < 0.99 * rounds(n, per_lane))
                per_lane = rule_it;
        }
    }
    if (tune && tune->rows && gemv_slots(lg, lanes) * 4 * tune->rows <= lanes && !gemv_one_tile_row(rate))
        rpg = tune->rows;
    pl.lg = lg;
    pl.rpg = rpg;
    pl.ntiles = ceil_div(nbr, (uint64_t)(lanes >> lg) * rpg);
    const uint32_t G = 1u << lg;
    uint32_t nslab = per_lane              ? ceil_div(pl.nbc, (uint64_t)G * per_lane)
                     : tune && tune->lanes ? split_slabs(blocks, pl.nbc, rule_lanes(rate), G)
                                           : by_rule;
    if (tune && tune->slabs)
        nslab = tune->slabs;
    const uint32_t max_slabs = ceil_div(pl.nbc, G);
    set_slabs(pl, std::max(1u, std::min(nslab, max_slabs)), G);
    return pl;
}

GemvPlan block_slab_plan(uint32_t cols, uint32_t row_begin, uint32_t row_end, int num_cus, uint32_t lanes,
                         uint32_t tile_rows)
{
    GemvPlan pl = range_plan(cols, row_begin, row_end);
    pl.lanes = lanes;
    const uint32_t nbr = pl.bi_end - pl.bi_begin;
    pl.ntiles = ceil_div(nbr, tile_rows);
    // enough workgroups to fill the chip several times over
    const uint64_t want = (uint64_t)(num_cus > 0 ? num_cus : 256) * 8;
    const uint32_t max_slabs = ceil_div(pl.nbc, lanes);
    uint32_t nslab = pl.ntiles ? ceil_div(want, pl.ntiles) : 1;
    if (nslab > max_slabs)
        nslab = max_slabs;
    set_slabs(pl, nslab ? nslab : 1, lanes);
    return pl;
}

hipError_t whz_gemv(uint32_t rate, const GemvPlan& pl, AccMode mode, const void* stream, const float* u, float* y,
                    double* part, hipStream_t st)
{
    if (pl.ntiles == 0)
        return hipSuccess;
    switch (rate / 2) {
#define X(k)                                                                                                         \
    case k:                                                                                                          \
        return nw##k::gemv(pl, mode, stream, u, y, part, st);
        WH_FOR_EACH_NW(X)
#undef X
    default:
        return hipErrorInvalidValue;
    }
}

// What a multi-RHS call of `nslab` column slabs takes, in the time of a step of
// 16 block columns at two workgroups a CU (`resident` of them; about 7 us).
// The workgroups of a launch are of one length, so they go in rounds: a last
// round of at most one a CU takes 0.6 of a full one's time, a fuller last round
// all of it.  But workgroups drift apart: six tenths of the time go as if
// rounds had no edges.  Partials (`per_slab` doubles each) are written and read
// at 3 TB/s.
double mrhs_shape_cost(uint32_t nslab, uint32_t ntiles, uint32_t steps, uint64_t per_slab, uint32_t resident)
{
    const uint32_t it = ceil_div(steps, nslab);
    const uint64_t wgs = (uint64_t)ntiles * nslab, rest = wgs % resident;
    const double alone = 0.3 + 0.6 * it, full = 0.3 + it;
    const double rounds = (double)(wgs / resident) * full + (rest == 0 ? 0.0 : 2 * rest <= resident ? alone : full);
    const double even = std::max((double)wgs / resident * full + 0.3 * it, alone);
    return 0.4 * rounds + 0.6 * even + (nslab > 1 ? 0.2 + (double)nslab * (double)per_slab * 8.0 / 21e6 : 0.0);
}

namespace {

// The rows, columns and contraction of a multi-RHS plan; its slabs are to be set.
MrhsPlan mrhs_range_plan(uint32_t cols, uint32_t row_begin, uint32_t row_end, uint32_t k, bool bf16,
                         const GemvTuning* tune)
{
    MrhsPlan pl = range_plan(cols, row_begin, row_end);
    pl.math = (uint32_t)mrhs_math(k, bf16, tune && tune->mrhs_fp32);
    return pl;
}

uint32_t mrhs_tiles(uint32_t nbr, uint32_t waves) { return ceil_div(nbr, 4 * waves); }

// The FP64 partials (slabs x k x rows) stay within 256 MiB: 8 slabs of up to
// 64 right-hand sides over 65536 rows (at k = 64, 8 slabs take 7.27 ms where 2
// took 7.60); short row ranges (few tiles, which need the slabs to fill the
// device) keep theirs.
uint32_t mrhs_slab_cap(uint64_t per_slab)
{
    return (uint32_t)std::max<uint64_t>(1, (32ull << 20) / std::max<uint64_t>(per_slab, 1));
}

// Slabs by a fixed rule: about two rounds of workgroups in a multiple of 8
// slabs (65536^2 with up to 16 right-hand sides: 8 slabs 5.4 ms where 3 take
// 6.2).
uint32_t mrhs_rule_slabs(uint32_t ntiles, uint32_t steps, uint32_t cap, uint32_t resident)
{
    uint32_t nslab = ntiles ? ceil_div(2 * (uint64_t)resident, ntiles) : 1;
    if (steps >= 8)
        nslab = (nslab + 7) / 8 * 8;
    return std::max(1u, std::min(std::min(nslab, cap), steps));
}

} // namespace

MrhsPlan whz_mrhs_plan(uint32_t rate, uint32_t rows, uint32_t cols, uint32_t row_begin, uint32_t row_end,
                       int num_cus, uint32_t k, bool bf16, const GemvTuning* tune, size_t most_workspace)
{
    (void)rows;
    const uint32_t slabs = tune ? tune->mrhs_slabs : 0;
    MrhsPlan pl = mrhs_range_plan(cols, row_begin, row_end, k, bf16, tune);
    const uint32_t nbr = pl.bi_end - pl.bi_begin;
    pl.ntiles = mrhs_tiles(nbr, (uint32_t)mrhs_waves((int)((k + 15) / 16), (int)rate / 2));
    const uint64_t per_slab = (uint64_t)std::max<uint32_t>(k, 1) * nbr * 4;
    const uint32_t cap = mrhs_slab_cap(per_slab);
    const uint32_t steps = (pl.nbc + 15) / 16, resident = 2u * (num_cus > 0 ? (uint32_t)num_cus : 256u);
    const auto fits = [&](uint32_t n) {
        MrhsPlan p = pl;
        set_slabs(p, n, 16);
        return mrhs_workspace(p, k).total <= most_workspace;
    };
    // the rule's count, unless the cost above says that another one is 2 %
    // better.  From sweeps over 22 shapes (us, the rule's count and the chosen
    // one): 48573 x 660 BF16 with 42 vectors 81 / 58, 4096^2 with 64 67 / 55,
    // 30000 x 700 with 20 59 / 51, 300 x 40000 at rate 16 with 12 58 / 49,
    // 1500 x 20000 BF16 with 64 76 / 65; none slower
    uint32_t nslab = mrhs_rule_slabs(pl.ntiles, steps, cap, resident);
    const auto cost_of = [&](uint32_t n) { return mrhs_shape_cost(n, pl.ntiles, steps, per_slab, resident); };
    double best = fits(nslab) ? 0.98 * cost_of(nslab) : 1e300;
    for (uint32_t it = 1; it < steps; it += std::max(1u, it / 16)) { // steps a slab
        const uint32_t n = ceil_div(steps, it);
        if (n <= cap && cost_of(n) < best && fits(n)) {
            best = cost_of(n);
            nslab = n;
        }
    }
    if (cost_of(1) < best)
        nslab = 1;
    if (slabs)
        nslab = slabs;
    if (nslab > steps)
        nslab = steps ? steps : 1;
    set_slabs(pl, nslab, 16);
    return pl;
}

size_t whz_serve_workspace(uint32_t rate, uint32_t cols, uint32_t row_begin, uint32_t row_end, int num_cus,
                           const GemvTuning* tune)
{
    const GemvPlan one = range_plan(cols, row_begin, row_end);
    const uint32_t nbr = one.bi_end - one.bi_begin;
    const uint32_t by_rule = rule_slabs(rate, nbr, one.nbc, nullptr);
    size_t most = by_rule > 1 ? (size_t)by_rule * one.part_rows() : 0;
    const uint32_t steps = (one.nbc + 15) / 16, resident = 2u * (num_cus > 0 ? (uint32_t)num_cus : 256u);
    for (uint32_t k = 16; k <= kMaxRhs; k += 16) {
        MrhsPlan pl = mrhs_range_plan(cols, row_begin, row_end, k, false, tune);
        const uint32_t cap = mrhs_slab_cap((uint64_t)k * nbr * 4);
        uint32_t nslab = mrhs_rule_slabs(mrhs_tiles(nbr, k <= 16 ? 16 : 8), steps, cap, resident);
        if (tune && tune->mrhs_slabs)
            nslab = std::max(1u, std::min(tune->mrhs_slabs, steps));
        set_slabs(pl, nslab, 16);
        most = std::max(most, mrhs_workspace(pl, k).total);
    }
    return most;
}

hipError_t whz_mrhs(uint32_t rate, const MrhsPlan& pl, const void* stream, const void* U, uint32_t ldu, uint32_t k,
                    float* Y, uint32_t ldy, double* part, hipStream_t st)
{
    if (pl.ntiles == 0)
        return hipSuccess;
    switch (rate / 2) {
#define X(kw)                                                                                                        \
    case kw:                                                                                                         \
        return nw##kw::mrhs(pl, stream, U, ldu, k, Y, ldy, part, st);
        WH_FOR_EACH_NW(X)
#undef X
    default:
        return hipErrorInvalidValue;
    }
}

} // namespace wh
