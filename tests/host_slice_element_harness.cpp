// Host build of the slicer's per-element routines, for CPU-side unit tests (no GPU involved): one vector is sliced with the
// exponents of its slices given, as split_stream_kernel does it, in "waves" of `chunk` consecutive elements that drop the waiting
// rule once none of their elements waits.
#include "../paper_2508_00441_amd/csrc/slice_element.hpp"
#include <stddef.h>
#include <vector>

extern "C" {
// x: n FP64 bit patterns, c: [s] exponents.  q_out: [s][n] slice integers.  Returns the number of (element, slice) that waited.
int host_slice_vector_narrow(const uint64_t* x, size_t n, int b, int s, int chunk, const int* c, int* q_out) {
    using namespace ozaki;
    const int F = 60 - b, pos = F - 32, bias = (1 << (pos - 1)) - 1;
    const uint32_t keep = ~((1u << pos) - 1u);
    int waited = 0;
    for (size_t i0 = 0; i0 < n; i0 += chunk) {
        const size_t i1 = i0 + chunk < n ? i0 + chunk : n;
        std::vector<int> wait(i1 - i0);
        std::vector<uint64_t> T(i1 - i0);
        for (size_t i = i0; i < i1; ++i) decode_narrow(x[i], F, T[i - i0], wait[i - i0]);
        int unit_prev = 0;
        bool settled = false;
        for (int p = 0; p < s; ++p) {
            const int unit = c[p] - b, step = unit_prev - unit;
            unit_prev = unit;
            bool waits = false;
            for (size_t i = i0; i < i1; ++i) {
                int& q = q_out[(size_t)p * n + i];
                if (settled) {
                    q = slice_narrow_active(T[i - i0], step, pos, bias, keep) >> pos;
                } else {
                    q = slice_narrow(T[i - i0], wait[i - i0], step, pos, bias, keep) >> pos;
                    waits |= wait[i - i0] < 0;
                    waited += wait[i - i0] < 0;
                }
            }
            settled |= !waits;
        }
    }
    return waited;
}
}
