// All slices of an element read off ONE fixed-point number, the units of a vector's slices off one OR.
//
// The nested roundings to nearest of Eq. 5-7 at units u_0 > u_1 > ... are a signed-digit recoding of the element: every remainder
// is x less x rounded to a multiple of the last unit (a remainder is at most half a unit, so each unit is an even multiple of the next).
// Write x in two's complement.  Before slice j, whose exponent is c_j and whose unit is 2^(c_j - b), the remainder is the bits from 2^c_j
// down as a signed number, and with step = b + 1
//     q_j = (g + 1) >> 1,   g = the step + 1 bits from 2^c_j down, signed: the digit and the half below it.
// That is rounding half up.  An exact half (which only the lowest set bit of x can be) rounds to the even neighbour; where that is the
// lower one, the bit above the lowest set one is 0, and subtracting one from the lowest bit of the number makes every digit right
// (0 1111...: the half is not rounded up, the next digit is 0 111..1 + 1 = +2^b, the others are -1 + 1 = 0).  So one is subtracted
// wherever that bit is 0: at units where the element is no exact half it changes no digit.  It also serves x = +2^c before the first slice.
//
// Eq. 4 after a slice whose unit is bit k: the largest remainder lies in (2^m, 2^(m+1)], where m is the highest place below k-1 whose bit
// differs from the one above it, and c = m + 1 (a positive power of two, which would be counted one place too high, has had one
// subtracted).  Over a vector that is the highest place at which ANY element has such a turn of bits.  So one OR of the turns of all
// elements gives the exponents of all slices, however the units lie.  (With enough elements each unit lies exactly `step` below the last;
// vectors of few non-zero elements, or whose elements run out of bits, leave that ladder all the time.)
//
// The number has 96 bits, bit 95 worth 2^c (c: exponent of slice 0), and places are counted from there down.  Bits below it are
// lost to the number and marked in its lowest bit and in that of the turns; a slice is taken while the half below its digit lies above
// that bit, and beyond it the vector's remainders start another number.
//
// Compiles for the device and, for CPU-side unit tests of this very code, for the host.
#pragma once
#include "slice_element.hpp"

namespace ozaki {

constexpr int NUMBER_BITS = 96;

// Digits are read off the upper word of the number, `fields` regular ones before the number has to move up.
struct DigitLadder {
    int step;                 // b + 1
    int fields;               // 31 / step: a field is step + 1 bits with the half below its digit
    uint32_t magic;           // ceil-like 2^16 / step: exact quotients below 96
    uint32_t tops[3];         // the places of regular exponents after the first, in a number's words
};
OZAKI_SLICE_HD DigitLadder digit_ladder(int b) {
    DigitLadder l;
    l.step = b + 1;
    l.fields = 31 / l.step;
    l.magic = 65536u / (uint32_t)l.step + 1u;
    l.tops[0] = l.tops[1] = l.tops[2] = 0;
    for (int at = l.step; at < NUMBER_BITS; at += l.step) l.tops[2 - at / 32] |= 0x80000000u >> (at % 32);
    return l;
}

// low word of (hi:lo) >> (n mod 32)
OZAKI_SLICE_HD uint32_t funnel_right(uint32_t hi, uint32_t lo, int n) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_alignbit(hi, lo, (uint32_t)n);
#else
    return (uint32_t)((((uint64_t)hi << 32) | lo) >> (n & 31));
#endif
}
// number of trailing zeros; 0xFFFFFFFF for 0
OZAKI_SLICE_HD uint32_t trailing_zeros(uint32_t v) {
#if defined(__HIP_DEVICE_COMPILE__)
    return (uint32_t)(__ffs((int)v) - 1);
#else
    return v ? (uint32_t)__builtin_ctz(v) : 0xFFFFFFFFu;
#endif
}
OZAKI_SLICE_HD uint32_t digit_min(uint32_t a, uint32_t b) { return a < b ? a : b; }

// The 96-bit number of an element, x[2] the upper word; its turns are ORed into `turns`.  The element modulo the bits above
// 2^c; BEYOND: the element may reach above 2^c (later numbers of a vector) or be a subnormal number (c below -1021).
template <bool BEYOND>
OZAKI_SLICE_HD void digit_number(uint64_t w, int c, uint32_t (&x)[3], uint32_t (&turns)[3]) {
    const uint32_t wh = (uint32_t)(w >> 32), wl = (uint32_t)w;
    const int e11 = (int)((wh >> 20) & 0x7FFu);
    const uint64_t neg = (uint64_t)((int64_t)w >> 63);
    const uint32_t mh = (wh & 0xFFFFFu) | (e11 != 0 ? 0x100000u : 0u);
    int r = c - ((e11 > 1 ? e11 : 1) - 1023);                        // places from bit 95 down to the leading bit of a normal number
    // trailing zeros of the significand; of zero so many that its lowest bit counts as one above the number
    const uint32_t tz = digit_min(trailing_zeros(wl), digit_min(trailing_zeros(mh), 4096u) + 32u);
    uint64_t S = ((((uint64_t)mh << 32) | wl) ^ neg) - neg;
    const uint32_t sg = (uint32_t)((int)(S >> 32) >> 31);            // (not the sign bit of x: -0.0 has no bits to fill up with)
    const int low = 52 + r - (int)tz;                                // places from bit 95 down to the lowest set bit
    const bool above = (((int64_t)S >> (tz & 63u)) & 2) != 0;        // the bit above the lowest set one
    const uint32_t one = !above && (uint32_t)low < (uint32_t)(NUMBER_BITS - 1) ? 1u : 0u;
    if (BEYOND) {
        S <<= digit_min((uint32_t)(r < 0 ? -r : 0), 63u);            // what is shifted out, or above bit 52, lies above 2^c
        r = r < 0 ? 0 : r;
    }
    const uint32_t h1 = funnel_right((uint32_t)(S >> 32), (uint32_t)S, 21), h0 = (uint32_t)S << 11;
    const uint32_t y2 = funnel_right(sg, h1, r), y1 = funnel_right(h1, h0, r), y0 = funnel_right(h0, 0u, r);
    const uint32_t x2 = r < 32 ? y2 : sg;
    const uint32_t x1 = r < 32 ? y1 : r < 64 ? y2 : sg;
    uint32_t x0 = r < 32 ? y0 : r < 64 ? y1 : r < 96 ? y2 : sg;
    x0 |= low >= NUMBER_BITS - 1 ? 1u : 0u;                          // something lies in the lowest bit or below the number
    const uint32_t b0 = x0 < one ? 1u : 0u;
    const uint64_t up = (((uint64_t)x2 << 32) | x1) - b0;
    x[0] = x0 - one;
    x[1] = (uint32_t)up;
    x[2] = (uint32_t)(up >> 32);
    turns[2] |= x[2] ^ funnel_right(x[2], x[1], 31);
    turns[1] |= x[1] ^ funnel_right(x[1], x[0], 31);
    turns[0] |= x[0] ^ ((x[0] << 1) | one);                          // (below a number from which one was subtracted the ones go on)
}

// A number, or the turns, moved up by n < 32 places, n > 0.
OZAKI_SLICE_HD void digit_shift(uint32_t& x2, uint32_t& x1, uint32_t& x0, int n) {
    x2 = funnel_right(x2, x1, 32 - n);
    x1 = funnel_right(x1, x0, 32 - n);
    x0 <<= n;
}

// Slice integer of field d of the upper word.
OZAKI_SLICE_HD int digit_of(uint32_t word, int d, int step) {
    const int off = 31 - (d + 1) * step;
#if defined(__HIP_DEVICE_COMPILE__)
    const int g = __builtin_amdgcn_sbfe((int)word, off, step + 1);
#else
    const int g = (int)(word << (d * step)) >> (31 - step);
    (void)off;
#endif
    return (g + 1) >> 1;
}

// Can a slice whose exponent is `at` places below 2^c be read off the number?
OZAKI_SLICE_HD bool digit_in_number(int at, int step) { return at + step <= NUMBER_BITS - 2; }

// Places from the top down to the first bit set; NUMBER_BITS if there is none.
OZAKI_SLICE_HD int digit_first(uint32_t w2, uint32_t w1, uint32_t w0) {
    const uint64_t up = ((uint64_t)w2 << 32) | w1;
    return up != 0 ? 64 - bit_length_u64(up) : NUMBER_BITS - bit_length_u32(w0);
}

// The vector's turns moved up by `at` places: how many slices from there on lie `step` apart inside the number (one at least).
OZAKI_SLICE_HD int digit_run(const uint32_t (&turns)[3], int at, const DigitLadder& l) {
    const uint32_t lead = (uint32_t)digit_first(l.tops[2] & ~turns[2], l.tops[1] & ~turns[1], l.tops[0] & ~turns[0]);
    return (int)((digit_min(lead, (uint32_t)(NUMBER_BITS - 2 - at)) * l.magic) >> 16);
}

// Eq. 4 after the first `run` of them: places from the first one's exponent down to that of the next slice, at least run * step;
// NUMBER_BITS where no remainder is left.  Where that is not in the number, the remainders have to be looked at.
OZAKI_SLICE_HD int digit_next(const uint32_t (&turns)[3], int run, int step) {
    const int d = run * step;                                        // < NUMBER_BITS
    return d < 64 ? digit_first(turns[2] & (uint32_t)((~0ull >> d) >> 32), turns[1] & (uint32_t)(~0ull >> d), turns[0])
                  : digit_first(0, 0, turns[0] & (~0u >> (d - 64)));
}

// |x| as a key whose maximum over a vector gives Eq. 4: the upper word, its lowest bit sticky.
OZAKI_SLICE_HD uint32_t magnitude_key(uint64_t w) {
    return ((uint32_t)(w >> 32) & 0x7FFFFFFFu) | digit_min((uint32_t)w, 1u);
}
// ceil(log2) of the vector's largest element, for keys of 2^20 and more (some element is not subnormal)
OZAKI_SLICE_HD int magnitude_exponent(uint32_t key) { return (int)(key >> 20) - 1023 + ((key & 0xFFFFFu) != 0 ? 1 : 0); }

// |remainder| at unit 2^(E + sh) of mm * 2^E, in units of 2^E: exact
OZAKI_SLICE_HD uint64_t remainder_abs(uint64_t mm, int sh) {
    if (sh <= 0) return 0;
    if (sh > 54) return mm;
    const uint64_t low = mm & ((1ull << sh) - 1), up = (1ull << sh) - low;
    return low < up ? low : up;
}
// ceil(log2) of a non-zero mm * 2^E, biased; 0 for zero
OZAKI_SLICE_HD uint32_t exponent_key(uint64_t mm, int E) {
    return mm == 0 ? 0u : (uint32_t)(E + bit_length_u64(mm) - (((mm & (mm - 1)) == 0) ? 1 : 0) + CD_BIAS);
}
// the same of the remainder of an FP64 number at unit 2^unit
OZAKI_SLICE_HD uint32_t remainder_key(uint64_t w, int unit) {
    const int e11 = (int)((w >> 52) & 0x7FF);
    uint64_t mm = w & 0x000FFFFFFFFFFFFFull;
    if (e11 != 0) mm |= 0x0010000000000000ull;
    const int E = e11 != 0 ? e11 - 1075 : -1074;
    return exponent_key(remainder_abs(mm, unit - E), E);
}

}  // namespace ozaki
