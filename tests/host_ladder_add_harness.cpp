// Host build of LadderAdd (fp64_emu.hpp), for CPU-side unit tests: sums of integer terms at rising scales, with and without a branch.
#include "../paper_2508_00441_amd/csrc/fp64_emu.hpp"
#include <stddef.h>

extern "C" {
// v: [sums][terms] integers, term i at the scale 2^(first + i * step).  Writes the FP64 bits of each sum as RoundedSum and as LadderAdd give
// them; narrow: for chains whose scales span 60 bits at most.
void host_ladder_sums(const int* v, size_t sums, int terms, int first, int step, int narrow, uint64_t* by_rounded, uint64_t* by_ladder) {
    using namespace ozaki;
    for (size_t j = 0; j < sums; ++j) {
        RoundedSum r;
        r.start_at_zero();
        LadderAdd l{0, first};
        for (int i = 0; i < terms; ++i) {
            r.add((int64_t)v[j * terms + i], first + i * step);
            if (narrow) l.add<60>(v[j * terms + i], first + i * step);
            else l.add<250>(v[j * terms + i], first + i * step);
        }
        by_rounded[j] = fp64_scale_pow2_emulated(r.value(), 7);
        by_ladder[j] = l.value(7);
    }
}
}
