// Host build of slice_digits.hpp, for CPU-side unit tests (no GPU involved): one vector sliced ladder by ladder, as the slicing
// kernel does it.
#include "../paper_2508_00441_amd/csrc/slice_digits.hpp"
#include <stddef.h>

extern "C" {
// x: n FP64 bit patterns.  q_out: [s][n] slice integers, c_out: [s] exponents.  Returns the number of ladders taken.
int host_slice_vector_digits(const uint64_t* x, size_t n, int b, int s, int* q_out, int* c_out) {
    using namespace ozaki;
    const DigitLadder l = digit_ladder(b);
    uint32_t top = 0;
    for (size_t i = 0; i < n; ++i) top = magnitude_key(x[i]) > top ? magnitude_key(x[i]) : top;
    auto exact = [&](int unit) {
        uint32_t key = 0;
        for (size_t i = 0; i < n; ++i) key = remainder_key(x[i], unit) > key ? remainder_key(x[i], unit) : key;
        return key;
    };
    bool left = top != 0;
    int c = left ? (top >= 0x100000u ? magnitude_exponent(top) : (int)exact(2000) - CD_BIAS) : 0, ladders = 0;
    for (int p = 0; p < s;) {
        if (!left) {
            for (; p < s; ++p) {
                c_out[p] = 0;
                for (size_t i = 0; i < n; ++i) q_out[(size_t)p * n + i] = 0;
            }
            break;
        }
        ++ladders;
        uint32_t proof[3] = {0, 0, 0};
        auto limbs = [&](size_t i, uint32_t (&w)[3]) {
            uint32_t y[3];
            if (p > 0 || c < -1021) digit_number<true>(x[i], c, l, y);
            else digit_number<false>(x[i], c, l, y);
            digit_limbs(y, l, w);
        };
        uint32_t w[3];
        for (size_t i = 0; i < n; ++i) {
            limbs(i, w);
            for (int j = 0; j < 3; ++j) proof[j] |= digit_proof(w[j]);
        }
        int levels = digit_levels(proof, l);
        if (levels > s - p) levels = s - p;
        for (int j = 0; j < levels; ++j) {
            c_out[p + j] = c - j * l.step;
            for (size_t i = 0; i < n; ++i) {
                limbs(i, w);
                q_out[(size_t)(p + j) * n + i] = digit_of(w[j / l.per_limb], j % l.per_limb, l.step);
            }
        }
        p += levels;
        const uint32_t key = exact(c - (levels - 1) * l.step - b);
        left = key != 0;
        c = (int)key - CD_BIAS;
    }
    return ladders;
}
}
