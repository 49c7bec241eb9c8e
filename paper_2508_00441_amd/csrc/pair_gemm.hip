// The 256 x 256 slice-pair GEMM kernels (pair_gemm_body.hpp) and the choice among the GEMM kernels.
#include "pair_gemm_body.hpp"

namespace ozaki {

namespace {

template <int FMT>
__global__ void __launch_bounds__(256) pair_gemm_kernel(const GemmArgs a) { pair_gemm_body<FMT, false>(a); }

}  // namespace

hipError_t launch_pair_gemm(const Plan& pl, const Operand& A, const Operand& B, const PairOrder& order, const Pass& ps,
                            bool allow_chain, const RunCheck& check, int64_t t, float* P, hipStream_t st) {
    if (ps.ngroups <= 0 || pl.tiles_m == 0 || pl.tiles_n == 0 || pl.chunks == 0) return hipSuccess;
    if (pl.small_tiles) return launch_pair_gemm_small(pl, A, B, order, ps, allow_chain, check, t, P, st);
    GemmArgs a;
    const size_t slice_a = (size_t)pl.chunks * A.rows_pad * pl.row_bytes, slice_b = (size_t)pl.chunks * B.rows_pad * pl.row_bytes;
    a.sa = A.slices + (size_t)t * pl.s * slice_a;
    a.sb = B.slices + (size_t)t * pl.s * slice_b;
    a.P = P;
    a.rows_pad_a = A.rows_pad; a.rows_pad_b = B.rows_pad; a.chunks = pl.chunks;
    a.tiles_m = (int)pl.tiles_m; a.tiles_n = (int)pl.tiles_n;
    a.quads_m = (int)pl.quads_m; a.quads_n = (int)pl.quads_n;
    a.allow_chain = allow_chain ? 1 : 0;
    a.da = A.deltas + (size_t)t * (A.rows_pad / LINK_ROWS) * pl.s;
    a.db = B.deltas + (size_t)t * (B.rows_pad / LINK_ROWS) * pl.s;
    a.order = order; a.pass = ps;
    list_groups(order, ps, a.groups);
    a.starts = check.starts;
    a.ba = check.bound_a != nullptr ? check.bound_a + (size_t)t * (A.rows_pad / LINK_ROWS) * pl.s : nullptr;
    a.bb = check.bound_b != nullptr ? check.bound_b + (size_t)t * (B.rows_pad / LINK_ROWS) * pl.s : nullptr;
    a.pair_bound = pl.pair_bound;
    a.sure = pl.run_limit;
    a.unit = ldexpf(1.0f, -pl.p_frac);
    const int64_t blocks = (int64_t)ps.ngroups * pl.tiles_m * pl.tiles_n;
    if (blocks > 0x7FFFFFFF || pl.chunks > 0x7FFFFFFF) return hipErrorInvalidValue;
    a.work = work_order(ps.npairs, ps.ngroups, longest_group(order, ps), 32, a.tiles_m, a.tiles_n, pl.chunks);
    if (check.starts != nullptr) return launch_pair_gemm_measured(a, pl.fmt, (unsigned)blocks, st);
    if (pl.fmt == FMT_FP16) hipLaunchKernelGGL((pair_gemm_kernel<FMT_FP16>), dim3((unsigned)blocks), dim3(256), 0, st, a);
    else if (pl.fmt == FMT_FP6) hipLaunchKernelGGL((pair_gemm_kernel<FMT_FP6>), dim3((unsigned)blocks), dim3(256), 0, st, a);
    else if (pl.fmt == FMT_FP6_E3M2) hipLaunchKernelGGL((pair_gemm_kernel<FMT_FP6_E3M2>), dim3((unsigned)blocks), dim3(256), 0, st, a);
    else if (pl.fmt == FMT_INT8) hipLaunchKernelGGL((pair_gemm_kernel<FMT_INT8>), dim3((unsigned)blocks), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((pair_gemm_kernel<FMT_FP8>), dim3((unsigned)blocks), dim3(256), 0, st, a);
    return hipGetLastError();
}

}  // namespace ozaki
