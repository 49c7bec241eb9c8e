// The per-element step of the slicer that carries remainders from slice to slice (blocks beyond 16384 elements whose units leave the
// ladder of slice_digits.hpp), for slices at most 7 bits wide: Eq. 5-7 of the paper, with the exponents of all slices known, on a 64-bit
// fixed-point number held as two 32-bit words, so that the rounding and the subtraction are 32-bit integer operations.
//
// With F = 60 - b fraction bits (F >= 53 here) an element of slice p is T = x^(p) / 2^(c_p - b) * 2^F, |T| <= 2^60.
// The unit of the slice sits at bit F of T, i.e. at bit pos = F - 32 of the upper word:
//     q        = nearest integer to T / 2^F, ties to even: (hi + (2^(pos-1) - 1) + carry) >> pos, where the carry out
//                of the lower word of T + (2^(F-1) - 1) + (unit bit of T) is (lo != 0) | unit bit
//     T - q 2^F  changes the upper word only
//
// An element whose lowest bit lies below 2^-F of the current unit cannot be written this way yet (it is then smaller
// than an eighth of the unit: q = 0).  It waits with its significand in T and, in `wait`, E + F - u: the left shift that would bring
// x = significand * 2^E to the unit 2^u of the current slice, negative while waiting.  Every slice adds u_previous - u to it; for
// an element that is already in fixed-point form (0 there) that is exactly the left shift from the previous unit to this one, so one
// rule serves both.  Once no element of a wave waits any more, the shift is the same for all (slice_narrow_active).
//
// Compiles for the device and, for CPU-side unit tests of this very code, for the host.
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define OZAKI_SLICE_HD __host__ __device__ __forceinline__
#else
#define OZAKI_SLICE_HD inline
#endif

namespace ozaki {

constexpr int CD_BIAS = 2048;             // ceil(log2 |x|) of a finite FP64 number is in [-1074, 1024]

OZAKI_SLICE_HD int bit_length_u64(uint64_t v) {            // 0 for v == 0
#if defined(__HIP_DEVICE_COMPILE__)
    return 64 - __clzll((long long)v);
#else
    return v ? 64 - __builtin_clzll(v) : 0;
#endif
}
OZAKI_SLICE_HD int bit_length_u32(uint32_t v) {
#if defined(__HIP_DEVICE_COMPILE__)
    return 32 - __clz((int)v);
#else
    return v ? 32 - __builtin_clz(v) : 0;
#endif
}

// FP64 bits -> waiting element.  Zero is in fixed-point form whatever the first unit is.
OZAKI_SLICE_HD void decode_narrow(uint64_t w, int F, uint64_t& T, int& wait) {
    const int e11 = (int)((w >> 52) & 0x7FF);
    uint64_t mm = w & 0x000FFFFFFFFFFFFFull;
    int E = -1074;
    if (e11 != 0) { mm |= 0x0010000000000000ull; E = e11 - 1075; }
    T = (w >> 63) ? 0ull - mm : mm;                                  // two's complement
    wait = mm == 0 ? 2047 : E + F;
}

// An element in fixed-point form whose remainder is still in units of the previous slice: `shift` brings it to this slice's
// unit.  pos = F - 32, bias = 2^(pos-1) - 1, keep = ~(2^pos - 1).  Returns q * 2^pos (the slice integer where it sits in the
// upper word).
OZAKI_SLICE_HD int slice_narrow_active(uint64_t& T, int shift, int pos, int bias, uint32_t keep) {
    const uint64_t t = T << (shift & 63);                           // nothing is shifted out: |T| <= 2^60 afterwards
    int hi = (int)(uint32_t)(t >> 32);
    const uint32_t lo = (uint32_t)t;
#if defined(__HIP_DEVICE_COMPILE__)
    uint32_t nz;                                                    // lo != 0 as 0 / 1: one 32-bit minimum (written out because
    asm("v_min_u32 %0, 1, %1" : "=v"(nz) : "v"(lo));                // the compiler turns the C form into a 64-bit compare and a select)
#else
    const uint32_t nz = lo != 0 ? 1u : 0u;
#endif
    const uint32_t carry = nz | (((uint32_t)hi >> pos) & 1u);       // (lo != 0) | unit bit
    const int sum = hi + bias + (int)carry;
    const int q_at_pos = (int)((uint32_t)sum & keep);
    hi -= q_at_pos;
    T = ((uint64_t)(uint32_t)hi << 32) | lo;
    return q_at_pos;
}

// One element that may still be waiting, one slice.  step = previous unit - this unit (minus this unit for the first slice).
OZAKI_SLICE_HD int slice_narrow(uint64_t& T, int& wait, int step, int pos, int bias, uint32_t keep) {
    wait += step;
    int q_at_pos = 0;
    if (wait >= 0) {
        q_at_pos = slice_narrow_active(T, wait, pos, bias, keep);
        wait = 0;
    }
    return q_at_pos;
}

}  // namespace ozaki
