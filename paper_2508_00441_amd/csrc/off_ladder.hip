// Launches of the kernels of off_ladder.hpp.
#include <string.h>

#include "off_ladder.hpp"

namespace ozaki {

extern template hipError_t launch_off_ladder_format<FMT_FP8>(const OffLadderArgs&, int, bool, unsigned, hipStream_t);
extern template hipError_t launch_off_ladder_format<FMT_INT8>(const OffLadderArgs&, int, bool, unsigned, hipStream_t);

hipError_t launch_off_ladder(const Plan& pl, const Operand& A, const Operand& B, const OffLadder& off, double* C, int64_t ldc,
                             const ScaledResult* scaled, int accum_mode, hipStream_t st) {
    if (!ladder_possible(pl) || pl.full || pl.T != 1 || off.limit % 32 != 0) return hipErrorInvalidValue;
    OffLadderArgs a;
    a.off = off;
    a.sa = A.slices; a.sb = B.slices;
    a.ea = A.exps; a.eb = B.exps;
    a.rows_pad_a = A.rows_pad; a.rows_pad_b = B.rows_pad;
    a.chunks = (int)pl.chunks;
    const int64_t bm = (pl.m + 31) / 32, bn = (pl.n + 31) / 32, blocks = off.limit / 32 * (bm + bn);
    if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
    a.blocks_m = (int)bm; a.blocks_n = (int)bn;
    a.m = pl.m; a.n = pl.n;
    a.two_b = 2 * pl.b; a.p_frac = pl.p_frac; a.run_limit = pl.run_limit;
    a.exact = accum_mode == ACC_EXACT ? 1 : 0;
    a.C = C; a.ldc = ldc;
    a.alpha = a.beta = 0; a.use_beta = 0;
    a.scaled = scaled != nullptr;
    if (scaled != nullptr) {
        a.C = scaled->C; a.ldc = scaled->ldc;
        memcpy(&a.alpha, &scaled->alpha, 8);
        memcpy(&a.beta, &scaled->beta, 8);
        a.use_beta = scaled->beta != 0.0;
    }
    const bool integer_only = accum_mode != ACC_HW;
    return pl.fmt == FMT_INT8 ? launch_off_ladder_format<FMT_INT8>(a, pl.s, integer_only, (unsigned)blocks, st)
                              : launch_off_ladder_format<FMT_FP8>(a, pl.s, integer_only, (unsigned)blocks, st);
}

}  // namespace ozaki
