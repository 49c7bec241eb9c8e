// Host build of the planner (plan.hpp): which blocks, groups and runs a call takes.
#include "../paper_2508_00441_amd/csrc/plan.hpp"

using namespace ozaki;

extern "C" {

// The route of a DGEMM call without rounding modes of its own (one word per running sum) in `bytes` of work memory (0: the
// documented size, -1: the documented minimum).  route: small_tiles, group_len, run_limit, measured, bounds from the slices,
// products per pass.  Returns the planner's status.
int plan_route(int64_t m, int64_t n, int64_t k, int fmt, int s, int64_t k_block, int full, int chained, int64_t bytes, int64_t route[6]) {
    Plan plan;
    const int st = make_plan(m, n, k, fmt, s, k_block, full != 0, plan);
    if (st != 0) return st;
    const size_t size = bytes > 0 ? (size_t)bytes : bytes < 0 ? minimum_bytes(plan) : recommended_bytes(plan);
    Route r;
    if (!place_call(plan, false, 1, chained != 0, true, WorkMem{reinterpret_cast<uint8_t*>((uintptr_t)1 << 40), size}, r))
        return OZAKI_STATUS_WORKSPACE;
    route[0] = r.pl.small_tiles;
    route[1] = r.pl.group_len;
    route[2] = r.pl.run_limit;
    route[3] = r.check.starts != nullptr;
    route[4] = r.check.bound_a != nullptr;
    route[5] = r.c.chunk_pairs;
    return 0;
}

// How a call in the documented work memory (with room for a scaled call's product) begins.  route: with launch_ladder_sums?, vectors off the ladder
// that it leaves out, does it look at the vectors itself?, is there a launch_deltas?, bytes at the end of the products' memory.
int ladder_route(int64_t m, int64_t n, int64_t k, int fmt, int s, int64_t k_block, int full, int exact, int64_t route[5]) {
    Plan plan;
    const int st = make_plan(m, n, k, fmt, s, k_block, full != 0, plan);
    if (st != 0) return st;
    Route r;
    const size_t size = recommended_bytes(plan) + product_bytes(plan);
    if (!place_call(plan, false, exact ? SUM_WORDS_MAX : 1, true, true, WorkMem{reinterpret_cast<uint8_t*>((uintptr_t)1 << 40), size}, r))
        return OZAKI_STATUS_WORKSPACE;
    if (!exact || ladder_exact_fits(fmt, s, full != 0)) place_ladder(r);
    route[0] = r.off.counts != nullptr;
    route[1] = r.off.limit;
    route[2] = r.off.uncounted != nullptr;
    route[3] = r.c.A.deltas != nullptr && r.off.uncounted == nullptr;
    route[4] = r.c.A.off_ladder ? reinterpret_cast<uint8_t*>(r.c.P) + (size_t)r.c.chunk_pairs * stored_bytes(r.pl) - r.c.A.off_ladder : 0;
    return 0;
}

// 1: strips, 0: the plain order, for a launch of groups of `len` pairs and less over the anti-diagonals of s slices, in blocks_m x blocks_n
// blocks of 256 (small: 128)
int order_of_launch(int small, int s, int full, int len, int64_t blocks_m, int64_t blocks_n, int64_t chunks) {
    const PairOrder o{s, full, len};
    Pass ps{order_top_diag(o), 2, 0, 0};
    for (int g = ps.g_hi; g >= 2; --g) { ps.npairs += diag_len(o, g); ps.ngroups += diag_groups(o, g); }
    return work_order(ps.npairs, ps.ngroups, longest_group(o, ps), small ? 64 : 32, blocks_m, blocks_n, chunks).unit != 0;
}

}  // extern "C"
