// Launch of the slice-pair GEMMs in 128 x 128 blocks (pair_gemm_small.hpp).
#include "pair_gemm_small.hpp"

namespace ozaki {

hipError_t launch_pair_gemm_small(const Plan& pl, const Operand& A, const Operand& B, const PairOrder& order, const Pass& ps,
                                  bool allow_chain, const RunCheck& check, const OffLadder& off, int64_t t, float* P, hipStream_t st) {
    SmallGemmArgs a;
    const size_t slice_a = (size_t)pl.chunks * A.rows_pad * pl.row_bytes, slice_b = (size_t)pl.chunks * B.rows_pad * pl.row_bytes;
    a.sa = A.slices + (size_t)t * pl.s * slice_a;
    a.sb = B.slices + (size_t)t * pl.s * slice_b;
    a.P = P;
    a.rows_pad_a = A.rows_pad; a.rows_pad_b = B.rows_pad; a.chunks = (int)pl.chunks;
    a.tiles_m = (int)pl.tiles_m; a.tiles_n = (int)pl.tiles_n;
    a.quads_m = (int)pl.quads_m; a.quads_n = (int)pl.quads_n;
    a.allow_chain = allow_chain ? 1 : 0;
    a.da = A.deltas != nullptr ? A.deltas + (size_t)t * (A.rows_pad / LINK_ROWS) * pl.s : nullptr;
    a.db = B.deltas != nullptr ? B.deltas + (size_t)t * (B.rows_pad / LINK_ROWS) * pl.s : nullptr;
    a.ea = A.exps + (size_t)t * pl.s * A.rows_pad;
    a.eb = B.exps + (size_t)t * pl.s * B.rows_pad;
    a.m = pl.m; a.n = pl.n;
    a.order = order; a.pass = ps;
    list_groups(order, ps, a.groups);
    a.starts = check.starts;
    a.ba = check.bound_a != nullptr ? check.bound_a + (size_t)t * (A.rows_pad / LINK_ROWS) * pl.s : nullptr;
    a.bb = check.bound_b != nullptr ? check.bound_b + (size_t)t * (B.rows_pad / LINK_ROWS) * pl.s : nullptr;
    a.pair_bound = pl.pair_bound;
    a.sure = pl.run_limit;
    a.unit = ldexpf(1.0f, -pl.p_frac);
    a.off = off;
    const int64_t blocks = (int64_t)ps.ngroups * a.quads_m * a.quads_n;
    if (blocks > 0x7FFFFFFF || pl.chunks * MAX_SLICES > 0x7FFFFFFF) return hipErrorInvalidValue;
    a.work = work_order(ps.npairs, ps.ngroups, longest_group(order, ps), 64, a.quads_m, a.quads_n, pl.chunks);
    const dim3 grid((unsigned)blocks);
    return off.counts != nullptr ? launch_pair_gemm_small_behind(a, pl.fmt, grid, st) : launch_small_kernel<false>(a, pl.fmt, grid, st);
}

}  // namespace ozaki
