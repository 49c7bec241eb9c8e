// The 256 x 256 slice-pair GEMM kernels (pair_gemm_body.hpp) and the choice among the GEMM kernels.
#include "pair_gemm_body.hpp"

namespace ozaki {

namespace {

template <int FMT>
__global__ void __launch_bounds__(256) pair_gemm_kernel(const GemmArgs a) { pair_gemm_body<FMT, false>(a); }

// FP8: the kernel of pair_gemm_fp8.hip, whose k-steps take two stages.  GEMM, us, pair_gemm_kernel and that one:
//   stages per pair  4096^2, 13 slices: 2 stages 289 and 303, 4 stages 391 and 389, 8 stages 603 and 598, 64 stages 3880 and 3830; 8192^2:
//                    930 and 983, 1380 and 1375, 2357 and 2347.  A pair of one long step has no second one to fetch for.
//   odd numbers      are filled up to even ones.  4096^2, 9 slices: 97 stages 2920 and 2970, 129 stages 3940 and 3940, 161 stages 4940 and
//                    4890, 257 stages 7800 and 7710; 8192 x 4096: 6040 and 6080, 8066 and 8040, 10010 and 9930, 15740 and 15570.
//   tiles            64 stages, 13 slices: 16 tiles 2 to 6 % slower, 32 tiles 526 and 528, 64 tiles 1027 and 1009, 132 tiles 2017 and
//                    1994, 224 tiles 3420 and 3393, 240 tiles 3665 and 3619.  Below 256 the length of the groups and the size of
//                    the blocks are chosen by estimates that are pair_gemm_kernel's (choose_gemm), so the line stays there.
bool fp8_long_steps(int64_t tiles, int64_t chunks) { return tiles >= 256 && (chunks % 2 == 0 ? chunks >= 4 : chunks >= 160); }

// Products of this size pass the caches on their way to the accumulation whatever the kernel does: their stores need not push the slices
// out of the L2s.  16384 x 8192 x 1024 FP8: GEMM 8.83 -> 8.39 ms; 4096^2 FP6, all pairs: GEMM 4.11 -> 4.07, accumulation 0.594 -> 0.564 ms;
// smaller ones are read back from the caches (2048^2 FP16: accumulation 55 -> 62 us with such stores).
constexpr double STREAMED_PRODUCT_BYTES = 512.0 * (1 << 20);

}  // namespace

hipError_t launch_pair_gemm(const Plan& pl, const Operand& A, const Operand& B, const PairOrder& order, const Pass& ps,
                            bool allow_chain, const RunCheck& check, const OffLadder& off, int64_t t, float* P, hipStream_t st) {
    if (ps.ngroups <= 0 || pl.tiles_m == 0 || pl.tiles_n == 0 || pl.chunks == 0) return hipSuccess;
    if (pl.small_tiles) return launch_pair_gemm_small(pl, A, B, order, ps, allow_chain, check, off, t, P, st);
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
    a.off = off;
    const int64_t blocks = (int64_t)ps.ngroups * pl.tiles_m * pl.tiles_n;
    if (blocks > 0x7FFFFFFF || pl.chunks > 0x7FFFFFFF) return hipErrorInvalidValue;
    a.work = work_order(ps.npairs, ps.ngroups, longest_group(order, ps), 32, a.tiles_m, a.tiles_n, pl.chunks);
    a.streamed = (double)ps.ngroups * (double)(pl.quads_m * pl.quads_n) * QUAD_ELEMS * 4.0 >= STREAMED_PRODUCT_BYTES;
    if (pl.fmt == FMT_FP8 && fp8_long_steps(pl.tiles_m * pl.tiles_n, pl.chunks)) return launch_pair_gemm_fp8(a, check.starts != nullptr, (unsigned)blocks, st);
    if (check.starts != nullptr) return launch_pair_gemm_measured(a, pl.fmt, (unsigned)blocks, st);
    if (pl.fmt == FMT_FP16) hipLaunchKernelGGL((pair_gemm_kernel<FMT_FP16>), dim3((unsigned)blocks), dim3(256), 0, st, a);
    else if (pl.fmt == FMT_FP6) hipLaunchKernelGGL((pair_gemm_kernel<FMT_FP6>), dim3((unsigned)blocks), dim3(256), 0, st, a);
    else if (pl.fmt == FMT_FP6_E3M2) hipLaunchKernelGGL((pair_gemm_kernel<FMT_FP6_E3M2>), dim3((unsigned)blocks), dim3(256), 0, st, a);
    else if (pl.fmt == FMT_INT8) hipLaunchKernelGGL((pair_gemm_kernel<FMT_INT8>), dim3((unsigned)blocks), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((pair_gemm_kernel<FMT_FP8>), dim3((unsigned)blocks), dim3(256), 0, st, a);
    return hipGetLastError();
}

}  // namespace ozaki
