// Host build of slice_digits.hpp, for CPU-side unit tests (no GPU involved): one vector sliced number by number, as the slicing
// kernel does it.
#include "../paper_2508_00441_amd/csrc/slice_digits.hpp"
#include <stddef.h>
#include <vector>

static int numbers;

extern "C" {
// How often the elements of the last vector had to be read for their 96-bit numbers.
int host_numbers_of_last_vector() { return numbers; }

// x: n FP64 bit patterns.  q_out: [s][n] slice integers, c_out: [s] exponents.  Returns the number of regular ladders of units, each unit
// b + 1 bits below the one before it, that the slices take.
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
    numbers = 0;
    int c = left ? (top >= 0x100000u ? magnitude_exponent(top) : (int)exact(2000) - CD_BIAS) : 0, ladders = 0;
    struct Number { uint32_t x[3]; };
    std::vector<Number> y(n);
    for (int p = 0; p < s;) {
        if (!left) {
            for (; p < s; ++p) {
                c_out[p] = 0;
                for (size_t i = 0; i < n; ++i) q_out[(size_t)p * n + i] = 0;
            }
            break;
        }
        ++numbers;
        ++ladders;
        uint32_t turns[3] = {0, 0, 0};
        for (size_t i = 0; i < n; ++i) {
            if (p > 0 || c < -1021) digit_number<true>(x[i], c, y[i].x, turns);
            else digit_number<false>(x[i], c, y[i].x, turns);
        }
        auto move_up = [&](int places) {
            for (; places > 0; places -= 31)
                for (size_t i = 0; i < n; ++i) digit_shift(y[i].x[2], y[i].x[1], y[i].x[0], places < 31 ? places : 31);
        };
        int at = 0, last = 0;
        bool more = true;
        while (true) {
            int run = digit_run(turns, at, l);
            run = run < s - p ? run : s - p;
            last = at + (run - 1) * l.step;
            int moved = 0;
            for (int d = 0; d < run; ++d) {
                if (d > 0 && d % l.fields == 0) {
                    move_up(l.fields * l.step);
                    moved += l.fields * l.step;
                }
                c_out[p + d] = c - at - d * l.step;
                for (size_t i = 0; i < n; ++i) q_out[(size_t)(p + d) * n + i] = digit_of(y[i].x[2], d % l.fields, l.step);
            }
            p += run;
            if (p == s) break;
            const int next = digit_next(turns, run, l.step);
            more = next != NUMBER_BITS;
            if (!digit_in_number(at + next, l.step)) break;
            ladders += next != run * l.step;
            at += next;
            move_up(next - moved);
            for (int rest = next; rest > 0; rest -= 31) digit_shift(turns[2], turns[1], turns[0], rest < 31 ? rest : 31);
        }
        if (p == s) break;
        const uint32_t key = more ? exact(c - last - b) : 0u;
        left = key != 0;
        c = (int)key - CD_BIAS;
    }
    return ladders;
}
}
