// Slices of at most 7 bits while the units follow the regular ladder: all slices of an element read off ONE fixed-point number.
//
// Every remainder of Eq. 7 is at most half a unit, so the next unit lies at least b+1 bits below; with enough elements some
// remainder is larger than a quarter of the unit, and then (Eq. 4) it lies exactly b+1 =: step bits below.  Along such a ladder of
// units u_0 > u_1 > ... the nested roundings to nearest of Eq. 5-7 are a signed-digit recoding of the element: with R_j = x / u_j
// rounded to nearest, q_j = R_j - 2^step R_(j-1), and R_j is the floor of x / u_j plus the bit below it.  Cut the two's complement
// fixed-point form of x into fields f_j of `step` bits that end at the units:
//     q_j = (f_j as a signed number) + (the top bit of f_(j+1))  =  (g + 1) >> 1  with g = f_j and that bit, signed.
// That is rounding half up.  An exact half (which only the lowest set bit of x can be) rounds to the even neighbour: where that
// is the lower one, subtracting one from the lowest bit of the number makes every digit right (0 1111...: the half is not rounded up, the
// next digit is 0 111..1 + 1 = +2^b, the others are -1 + 1 = 0).  The same subtraction serves x = +2^c before the first slice.
//
// Whether a unit follows the ladder is read off the same number: the remainder before slice j, as a fraction of u_(j-1), is f_j and
// what is below it as a signed fraction; it is larger than a quarter in magnitude if its bits begin with 10 or 011 (01 alone may be
// exactly a quarter).  One such element in the vector proves c_j = c_(j-1) - step.  So a vector needs one OR over its elements for
// all slices, instead of one maximum after another.
//
// The number has 96 bits, bit 95 worth 2^c (c: exponent of slice 0 of the ladder; the unit of slice j ends at bit 95 - b - j step),
// the lowest bit sticky.  It is cut into three limbs of 32 bits that each begin at a field, D = 31 / step fields per limb (the
// bit below a limb's last field is in it too).
//
// Compiles for the device and, for CPU-side unit tests of this very code, for the host.
#pragma once
#include "slice_element.hpp"

namespace ozaki {

struct DigitLadder {
    int step;                 // b + 1
    int per_limb;             // D
    uint32_t magic;           // ceil-like 2^16 / step: exact quotients and divisibility tests below 96
    uint32_t tops;            // the top bits of a limb's fields
};
OZAKI_SLICE_HD DigitLadder digit_ladder(int b) {
    DigitLadder l;
    l.step = b + 1;
    l.per_limb = 31 / l.step;
    l.magic = 65536u / (uint32_t)l.step + 1u;
    l.tops = 0;
    for (int d = 0; d < l.per_limb; ++d) l.tops |= 0x80000000u >> (d * l.step);
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
// number of trailing zeros; at least 32 for 0
OZAKI_SLICE_HD uint32_t trailing_zeros(uint32_t v) {
#if defined(__HIP_DEVICE_COMPILE__)
    return (uint32_t)(__ffs((int)v) - 1);
#else
    return v ? (uint32_t)__builtin_ctz(v) : 0xFFFFFFFFu;
#endif
}
OZAKI_SLICE_HD uint32_t digit_min(uint32_t a, uint32_t b) { return a < b ? a : b; }

// The 96-bit number of an element, x[2] the upper word.  |element| modulo the bits above 2^c; BEYOND: the element may reach above
// 2^c (later ladders of a vector) or be a subnormal number (c below -1021).
template <bool BEYOND>
OZAKI_SLICE_HD void digit_number(uint64_t w, int c, const DigitLadder& l, uint32_t (&x)[3]) {
    const uint32_t wh = (uint32_t)(w >> 32), wl = (uint32_t)w;
    const int e11 = (int)((wh >> 20) & 0x7FFu);
    const uint64_t neg = (uint64_t)((int64_t)w >> 63);
    const uint32_t mh = (wh & 0xFFFFFu) | (e11 != 0 ? 0x100000u : 0u);
    int r = c - ((e11 > 1 ? e11 : 1) - 1023);                        // places from bit 95 down to the leading bit of a normal number
    const uint32_t tz = digit_min(trailing_zeros(wl), digit_min(trailing_zeros(mh), 63u - 32u) + 32u);
    const uint64_t S = ((((uint64_t)mh << 32) | wl) ^ neg) - neg;
    const uint32_t sg = (uint32_t)((int)(S >> 32) >> 31);            // (not the sign bit of x: -0.0 has no bits to fill up with)
    const int low = 52 + r - (int)tz;                                // places from bit 95 down to the lowest set bit
    const bool above = (((int64_t)S >> tz) & 2) != 0;                // the bit above the lowest set one
    const bool half = (uint32_t)low < 96u && (((uint32_t)low * l.magic) & 0xFFFFu) < l.magic;
    const uint32_t one = half && !above ? 1u : 0u;
    uint32_t h1 = funnel_right((uint32_t)(S >> 32), (uint32_t)S, 21), h0 = (uint32_t)S << 11;
    if (BEYOND) {
        if (r < 0) {
            const uint64_t h = r > -64 ? (((uint64_t)h1 << 32) | h0) << -r : 0ull;
            h1 = (uint32_t)(h >> 32);
            h0 = (uint32_t)h;
            r = 0;
        }
    }
    const uint32_t y2 = funnel_right(sg, h1, r), y1 = funnel_right(h1, h0, r), y0 = funnel_right(h0, 0u, r);
    const uint32_t x2 = r < 32 ? y2 : sg;
    const uint32_t x1 = r < 32 ? y1 : r < 64 ? y2 : sg;
    uint32_t x0 = r < 32 ? y0 : r < 64 ? y1 : r < 96 ? y2 : sg;
    x0 |= low >= 96 ? 1u : 0u;                                       // something lies below the number
    const uint32_t b0 = x0 < one ? 1u : 0u;
    const uint64_t up = (((uint64_t)x2 << 32) | x1) - b0;
    x[0] = x0 - one;
    x[1] = (uint32_t)up;
    x[2] = (uint32_t)(up >> 32);
}

// The limbs: 32 bits from field 0, D and 2D on.
OZAKI_SLICE_HD void digit_limbs(const uint32_t (&x)[3], const DigitLadder& l, uint32_t (&w)[3]) {
    const int o = l.per_limb * l.step;                               // 24 .. 31
    w[0] = x[2];
    w[1] = funnel_right(x[2], x[1], 32 - o);
    w[2] = funnel_right(x[1], x[0], 64 - 2 * o);
}

// Bit at the top of field j: the remainder before slice j is larger than a quarter of the unit before it.  (At the last field of a
// limb of one-bit steps the third bit is missing and taken as 0: then only 10 counts.)
OZAKI_SLICE_HD uint32_t digit_proof(uint32_t w) {
    const uint32_t a = w << 1, b = w << 2;
    return (w & ~a) | (~w & a & b);
}

// Slice integer of field d of a limb.
OZAKI_SLICE_HD int digit_of(uint32_t limb, int d, int step) {
    const int off = 31 - (d + 1) * step;
#if defined(__HIP_DEVICE_COMPILE__)
    const int g = __builtin_amdgcn_sbfe((int)limb, off, step + 1);
#else
    const int g = (int)(limb << (d * step)) >> (31 - step);
    (void)off;
#endif
    return (g + 1) >> 1;
}

// How many slices of the ladder the vector's proofs confirm: slice 0 is given, the first unconfirmed one ends it.  `first`: the
// top bit of field 0 of limb 0 is not asked for.
OZAKI_SLICE_HD int digit_levels(const uint32_t (&proof)[3], const DigitLadder& l) {
    int n = 0;
    for (int i = 0; i < 3; ++i) {
        const uint32_t missing = l.tops & ~(i == 0 ? proof[0] | 0x80000000u : proof[i]);
        if (missing != 0) {
            const uint32_t lead = 32u - (uint32_t)bit_length_u32(missing);
            return n + (int)((lead * l.magic) >> 16);
        }
        n += l.per_limb;
    }
    return n;
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
