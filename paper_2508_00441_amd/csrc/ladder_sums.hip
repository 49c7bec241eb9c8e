// Launches of the kernels of ladder_sums.hpp.
#include <string.h>

#include "ladder_sums.hpp"

namespace ozaki {

extern template hipError_t launch_ladder_kernel<FMT_FP8, ACC_HW>(const LadderArgs&, int, int, unsigned, hipStream_t);
extern template hipError_t launch_ladder_kernel<FMT_FP8, ACC_EMU>(const LadderArgs&, int, int, unsigned, hipStream_t);
extern template hipError_t launch_ladder_kernel<FMT_FP8, ACC_EXACT>(const LadderArgs&, int, int, unsigned, hipStream_t);
extern template hipError_t launch_ladder_kernel<FMT_FP6, ACC_HW>(const LadderArgs&, int, int, unsigned, hipStream_t);
extern template hipError_t launch_ladder_kernel<FMT_FP6, ACC_EMU>(const LadderArgs&, int, int, unsigned, hipStream_t);
extern template hipError_t launch_ladder_kernel<FMT_FP6, ACC_EXACT>(const LadderArgs&, int, int, unsigned, hipStream_t);
extern template hipError_t launch_ladder_kernel<FMT_FP6_E3M2, ACC_HW>(const LadderArgs&, int, int, unsigned, hipStream_t);
extern template hipError_t launch_ladder_kernel<FMT_FP6_E3M2, ACC_EMU>(const LadderArgs&, int, int, unsigned, hipStream_t);
extern template hipError_t launch_ladder_kernel<FMT_FP6_E3M2, ACC_EXACT>(const LadderArgs&, int, int, unsigned, hipStream_t);
extern template hipError_t launch_ladder_kernel<FMT_INT8, ACC_HW>(const LadderArgs&, int, int, unsigned, hipStream_t);
extern template hipError_t launch_ladder_kernel<FMT_INT8, ACC_EMU>(const LadderArgs&, int, int, unsigned, hipStream_t);
extern template hipError_t launch_ladder_kernel<FMT_INT8, ACC_EXACT>(const LadderArgs&, int, int, unsigned, hipStream_t);

namespace {

template <int FMT>
hipError_t launch_mode(const LadderArgs& a, int S, int accum_mode, int part, unsigned blocks, hipStream_t st) {
    if (accum_mode == ACC_EXACT) return launch_ladder_kernel<FMT, ACC_EXACT>(a, S, part, blocks, st);
    if (accum_mode == ACC_EMU) return launch_ladder_kernel<FMT, ACC_EMU>(a, S, part, blocks, st);
    return launch_ladder_kernel<FMT, ACC_HW>(a, S, part, blocks, st);
}

}  // namespace

hipError_t launch_ladder_sums(const Plan& pl, const Operand& A, const Operand& B, int64_t t, const OffLadder& off, uint64_t* S, double* C,
                              int64_t ldc, const ScaledResult* scaled, int accum_mode, hipStream_t st) {
    if (!ladder_possible(pl)) return hipErrorInvalidValue;
    LadderArgs a;
    const size_t slice_a = (size_t)pl.chunks * A.rows_pad * pl.row_bytes, slice_b = (size_t)pl.chunks * B.rows_pad * pl.row_bytes;
    a.sa = A.slices + (size_t)t * pl.s * slice_a;
    a.sb = B.slices + (size_t)t * pl.s * slice_b;
    a.ea = A.exps + (size_t)t * pl.s * A.rows_pad;
    a.eb = B.exps + (size_t)t * pl.s * B.rows_pad;
    a.rows_pad_a = A.rows_pad; a.rows_pad_b = B.rows_pad;
    a.chunks = (int)pl.chunks; a.s = pl.s;
    const int64_t bm = ladder_blocks(pl.m), bn = ladder_blocks(pl.n);
    a.blocks_m = (int)bm; a.blocks_n = (int)bn;
    a.work = WorkOrder{32, 4};                            // an XCD's 32 workgroups: 4 x 8 tiles, which share their slices
    a.m = pl.m; a.n = pl.n;
    a.add_to_C = t > 0;
    a.off = off;
    a.deltas = delta_args(pl, &A, &B);
    a.deltas_of = a.deltas.tiles * (unsigned)pl.T * (unsigned)pl.s;      // (with off.uncounted: of MOST_MARKS / 256 tiles at most)
    a.S = S;
    a.C = C; a.ldc = ldc;
    a.W = C; a.ldw = ldc;
    a.alpha = a.beta = 0; a.use_beta = 0;
    a.scaled = scaled != nullptr;
    if (scaled != nullptr) {
        a.C = scaled->C; a.ldc = scaled->ldc;
        memcpy(&a.alpha, &scaled->alpha, 8);
        memcpy(&a.beta, &scaled->beta, 8);
        a.use_beta = scaled->beta != 0.0;
    }
    for (int part = pl.full ? LESSER_HALF : WHOLE; part <= (pl.full ? GREATER_HALF : WHOLE); ++part) {
        const int S_kernel = part == LESSER_HALF ? pl.s - 1 : pl.s;
        if (t > 0 || part == GREATER_HALF) a.off.uncounted = nullptr;      // the call's first launch has left its answer
        const unsigned blocks = (unsigned)(bm * bn);
        hipError_t e;
        if (pl.fmt == FMT_FP6) e = launch_mode<FMT_FP6>(a, S_kernel, accum_mode, part, blocks, st);
        else if (pl.fmt == FMT_FP6_E3M2) e = launch_mode<FMT_FP6_E3M2>(a, S_kernel, accum_mode, part, blocks, st);
        else if (pl.fmt == FMT_INT8) e = launch_mode<FMT_INT8>(a, S_kernel, accum_mode, part, blocks, st);
        else e = launch_mode<FMT_FP8>(a, S_kernel, accum_mode, part, blocks, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace ozaki
