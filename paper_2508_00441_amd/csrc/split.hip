// Slicing of the FP64 operands into Type2 slices (paper Section 3, Eq. 4-8), integer arithmetic only.
//
// For a vector x (a row of A or a column of B restricted to one k-block) and p = 1..s:
//     c   = smallest integer with max|x^(p)| <= 2^c   (Eq. 4, evaluated exactly; 0 for a zero vector)
//     q_i = x^(p)_i / 2^(c-b) rounded to the nearest integer, ties to even       (Eq. 5-6)
//     x^(p+1)_i = x^(p)_i - q_i 2^(c-b)                                            (Eq. 7, exact)
//     slice^(p)_i = q_i 2^-b stored in Type2                                       (Eq. 8)
// Eq. 5-6 obtain q through (x + sigma) - sigma with sigma = 0.75 * 2^(rho+c) in FP64: x + sigma lies in the
// binade whose unit in the last place is 2^(rho+c-53) = 2^(c-b), sigma is an even multiple of that unit,
// so the FP64 addition rounds x to the nearest multiple of 2^(c-b) with ties to even q, and the
// subtraction of sigma is exact.  The kernel computes the same q with integers: once an element is within
// reach of the current unit it is kept as the signed 64-bit fixed-point number x^(p) / 2^(c-b) with 60-b
// fraction bits, which holds the element and every later remainder exactly (|x^(p)| <= 2^c bounds it by 2^60);
// q is its rounding to an integer, the remainder is what is left, and moving to the next slice is a left shift
// by c_p - c_(p+1).  Until then the element waits with its significand and exponent: with b <= 7 it is then smaller
// than half the unit (q = 0); with wider slices it can already reach the unit, and is rounded in its integer form.
// No FP64 instruction is executed.  Two forms of this element step: slices of at most 7 bits (FP8, FP6, INT8, and FP16 in
// blocks of 1024 elements and more) work on the upper 32-bit word of the fixed-point number (slice_element.hpp); wider FP16
// slices, whose fixed-point form has fewer than 53 fraction bits, take the 64-bit step below (decode_element,
// slice_element).  4096 + 4096 vectors of 4096 elements, nine FP16 slices of 6 bits: 0.33 ms with the 64-bit step, 0.24 ms with the 32-bit one.
//
// A vector is held in the registers of TPR threads (8*U consecutive elements per thread in U groups of
// eight) for all s slices, so HBM sees each input element once and each slice code once.
#include <string.h>

#include "layout.hpp"
#include "slice_element.hpp"

namespace ozaki {

namespace {

__global__ void __launch_bounds__(256) transpose_kernel(const double* __restrict__ A, int64_t lda, int64_t m, int64_t k,
                                                        double* __restrict__ At) {
    __shared__ double tile[32][33];
    const int64_t i0 = (int64_t)blockIdx.x * 32, k0 = (int64_t)blockIdx.y * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    for (int j = ty; j < 32; j += 8) {
        int64_t i = i0 + tx, kk = k0 + j;
        if (i < m && kk < k) tile[j][tx] = A[i + kk * lda];
    }
    __syncthreads();
    for (int j = ty; j < 32; j += 8) {
        int64_t i = i0 + j, kk = k0 + tx;
        if (i < m && kk < k) At[i * k + kk] = tile[tx][j];
    }
}

// Two consecutive FP64 bit patterns, loaded with one 16-byte access.  Vectors with an odd leading dimension, or a base address
// that is only a multiple of 8, put them 8 bytes off a 16-byte boundary: global loads of the GPU need 4-byte alignment only,
// and the type says 8 to the compiler.  (Eight 8-byte loads per thread, 64 bytes apart from lane to lane, took twice the time.)
typedef uint64_t two_doubles __attribute__((ext_vector_type(2), aligned(8)));

// One operand of a split launch.
struct SplitVectors {
    const double* X;       // vector r starts at X + r*ldv, its elements are `es` apart
    int64_t ldv, es;
    int64_t rows, rows_pad;
    uint8_t* slices;       // null: count only, nothing is stored
    int32_t* exps;
    int32_t* l1;           // sum |q| per slice, or null (FP16 slices only)
};

// A launch splits the vectors of up to two operands (same k, block length, format and slice count): the first wg_first
// workgroups of the grid belong to v[0], the rest to v[1].
struct SplitArgs {
    SplitVectors v[2];
    unsigned wg_first;     // a multiple of 64
    int64_t k, kb;
    int64_t chunks;        // chunks per block
    int s, b;
    int* flags;            // [0]: non-finite input seen; [1]: slice count (count-only mode)
};

constexpr int NO_ELEM = -(1 << 30);
static_assert(NO_ELEM == NO_CANDIDATE, "the two slicers share the reduction");

// Type2 codes of the two values q0 * 2^-b and q1 * 2^-b (|q| <= 2^b), packed low/high.  The hardware FP32 -> FP8
// (OCP E4M3 on gfx950) and FP32 -> FP16 conversions are exact here because every such value is a normal number of
// the format; FP32 arithmetic is not FP64 arithmetic, so the integer-only property of the slicer is about FP64.
template <int FMT>
__device__ __forceinline__ uint32_t encode_type2_pair(int q0, int q1, int b) {
    if (FMT == FMT_INT8) return ((uint32_t)q0 & 0xFFu) | (((uint32_t)q1 & 0xFFu) << 8);     // the integers themselves, |q| <= 64
    const float f0 = ldexpf((float)q0, -b), f1 = ldexpf((float)q1, -b);
    if (FMT == FMT_FP16) {
        typedef _Float16 h2 __attribute__((ext_vector_type(2)));
        const h2 h = {(_Float16)f0, (_Float16)f1};
        return __builtin_bit_cast(uint32_t, h);                       // q = 0 gives +0.0, code 0
    } else {
        const uint32_t w = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(f0, f1, 0, false) & 0xFFFFu;
        return w;
    }
}

// FP6 E2M3 code of q * 2^-(b-1), twice the slice value (|q| <= 2^b, b <= 4): with q' = q * 2^(4-b) the value is q'/8,
// and for magnitudes 0..16 the code (subnormals 0..7, normals 8..15 with exponent field 1, 16 = 2.0) is the magnitude
// itself; bit 5 is the sign.
__device__ __forceinline__ uint32_t encode_e2m3(int q, int b) {
    const int v = q << (4 - b);
    const uint32_t mag = (uint32_t)(v < 0 ? -v : v);
    return mag | (v < 0 ? 32u : 0u);
}

// FP6 E3M2 code of q * 2^-b (|q| <= 2^b, b <= 3): with q' = q * 2^(3-b) the value is q'/8; the codes (exponent field
// << 2 | fraction) of the magnitudes 0 .. 8 are 0 (zero), 2 (subnormal 2/16), 4, 6, 8, 9, 10, 11, 12; bit 5 is the sign.
__device__ __forceinline__ uint32_t encode_e3m2(int q, int b) {
    const int v = q << (3 - b);
    const uint32_t mag = (uint32_t)(v < 0 ? -v : v);
    return (uint32_t)((0xCBA986420ull >> (4 * mag)) & 0xFull) | (v < 0 ? 32u : 0u);
}

constexpr int ACTIVE = 0x7FFF;

// Element state shared by the two slicing kernels.  Dormant (not yet representable exactly with F fraction bits of
// the current unit): tv = signed 53-bit significand, pk = (E + F) | (cd << 16) with x = tv * 2^E and
// cd = ceil(log2 |x|).  Active: tv = T = x^(p) / 2^(c_p - b) * 2^F as a signed 64-bit integer (|x^(p)| <= 2^(c_p)
// bounds |T| by 2^(b+F) = 2^60), pk = ACTIVE.  An element becomes active at the first slice whose unit 2^u satisfies
// u <= E + F and stays so.
__device__ __forceinline__ void decode_element(uint64_t w, int F, int64_t& tv, int& pk, int& cmax, bool& nonfinite) {
    const int e11 = (int)((w >> 52) & 0x7FF);
    uint64_t mm = w & 0x000FFFFFFFFFFFFFull;
    nonfinite |= (e11 == 0x7FF);
    int E = -1074;
    if (e11 != 0) { mm |= 0x0010000000000000ull; E = e11 - 1075; }
    const int L = 64 - __clzll((long long)mm);                       // bit length (0 for mm == 0)
    const int cd = E + L - (((mm & (mm - 1)) == 0) ? 1 : 0);         // smallest c with |x| <= 2^c
    tv = (w >> 63) ? -(int64_t)mm : (int64_t)mm;
    pk = mm == 0 ? ACTIVE : (((E + F) & 0xFFFF) | (cd << 16));
    cmax = (mm != 0 && cd > cmax) ? cd : cmax;
}

// Eq. 5-8 for one element of an FP16 slicing and one slice whose unit is 2^unit: returns q, leaves the exact remainder
// in (T, st), and keeps track of the largest remainder of the active elements (rmax, in units of 2^(unit - F)) and of
// the largest ceil(log2 |x|) of the still dormant ones (cdorm).  rescale: left shift that brings an active remainder
// from the previous slice's unit to this one.  (Slices of at most 7 bits use slice_element.hpp instead.)
__device__ __forceinline__ int slice_element(int64_t& tv, int& pk, int unit, int rescale, int F, int64_t round_bias, uint64_t& rmax,
                                             int& cdorm) {
    // The bookkeeping of dormant elements is done with selects, the 64-bit arithmetic of active ones behind ONE
    // divergent branch: dormant elements (most of a wide-range vector during its first slices) and zeros skip it.
    const int st = pk;
    const bool was_active = st == ACTIVE;
    const int ef = (int)(short)(st & 0xFFFF);
    const bool wakes = !was_active && unit <= ef;          // representable from now on: x / 2^unit * 2^F
    const bool active = was_active || wakes;
    if (!active && unit - ef + F <= 53) {
        // With b >= 8 there are fewer than 53 fraction bits: the element reaches the unit but its low bits do not
        // fit the fixed-point form yet.  Round its integer form tv * 2^E directly, by sh = unit - E bits, and let the
        // remainder wait on as a dormant element with the same E.
        int64_t T = tv;
        const int sh = unit - ef + F;                      // F < sh <= 53
        const int64_t q64 = (T + (((int64_t)1 << (sh - 1)) - 1) + ((T >> sh) & 1)) >> sh;
        T -= q64 << sh;
        tv = T;
        const uint64_t ar = (uint64_t)(T < 0 ? -T : T);
        if (ar == 0) {
            pk = ACTIVE;                                   // nothing left: an active zero
        } else {
            const int L = 64 - __clzll((long long)ar);
            const int cd = ef - F + L - (((ar & (ar - 1)) == 0) ? 1 : 0);
            pk = (st & 0xFFFF) | (cd << 16);
            cdorm = cd > cdorm ? cd : cdorm;
        }
        return (int)q64;
    }
    const int cd = st >> 16;
    cdorm = (!active && cd > cdorm) ? cd : cdorm;          // still dormant: |x| < 2^(unit-1), q = 0, remainder = x
    pk = active ? ACTIVE : st;
    int q = 0;
    if (active) {
        // an active remainder is rescaled from the previous slice's unit, a waking element is brought to this unit
        int64_t T = tv << (was_active ? rescale : ef - unit);
        // nearest integer to T / 2^F, ties to even (two's complement form), and the exact remainder
        const int64_t q64 = (T + round_bias + ((T >> F) & 1)) >> F;
        q = (int)q64;
        T -= q64 << F;
        const uint64_t ar = (uint64_t)(T < 0 ? -T : T);
        rmax = ar > rmax ? ar : rmax;
        tv = T;
    }
    return q;
}

// Stores the Type2 codes of eight consecutive inner indices ke .. ke+7 of vector `row` into slice matrix dst_slice
// (internal layout, see layout.hpp).
template <int FMT>
__device__ __forceinline__ void store_codes(const int (&qs)[8], int64_t ke, uint8_t* dst_slice, int64_t v_rows_pad, int64_t row, int b) {
    constexpr bool FP16 = FMT == FMT_FP16;
    constexpr bool FP6 = fmt_is_fp6(FMT);
    constexpr int EPC = FP16 ? CHUNK_BYTES / 2 : CHUNK_BYTES;
    constexpr int ROWB = FP6 ? CHUNK_BYTES_FP6 : CHUNK_BYTES;
    if constexpr (FP6) {
        // eight 6-bit codes = 48 bits: octet j of the 24-byte string of k-group g, i.e. bytes
        // 6j .. 6j+5 of the string, whose first 16 bytes live in the 16-byte plane of g and the rest in the
        // 8-byte plane (see layout.hpp).  Written as one 32-bit and one 16-bit store, both naturally aligned.
        uint64_t w48 = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e)
            w48 |= (uint64_t)(FMT == FMT_FP6_E3M2 ? encode_e3m2(qs[e], b) : encode_e2m3(qs[e], b)) << (6 * e);
        const int64_t kc = ke / EPC;
        const int o = (int)((ke % EPC) / 8), g = o >> 2, j = o & 3;
        uint8_t* const chunk = dst_slice + (size_t)kc * v_rows_pad * ROWB;
        uint8_t* const p16 = chunk + ((size_t)g * v_rows_pad + row) * 16;
        uint8_t* const p8 = chunk + (size_t)v_rows_pad * 32 + ((size_t)g * v_rows_pad + row) * 8;
        uint8_t* d32 = j == 0 ? p16 : j == 1 ? p16 + 8 : j == 2 ? p16 + 12 : p8 + 4;
        uint8_t* d16 = j == 0 ? p16 + 4 : j == 1 ? p16 + 6 : j == 2 ? p8 : p8 + 2;
        const bool low32 = (j & 1) == 0;                   // bytes 6j.. start 4-byte aligned for even j
        *reinterpret_cast<uint32_t*>(d32) = low32 ? (uint32_t)w48 : (uint32_t)(w48 >> 16);
        *reinterpret_cast<uint16_t*>(d16) = low32 ? (uint16_t)(w48 >> 32) : (uint16_t)w48;
    } else {
        uint32_t c2[4];                                            // two codes each
#pragma unroll
        for (int e = 0; e < 4; ++e) c2[e] = encode_type2_pair<FMT>(qs[2 * e], qs[2 * e + 1], b);
        const int64_t kc = ke / EPC;
        uint8_t* dst = dst_slice + ((size_t)kc * v_rows_pad + row) * CHUNK_BYTES + (ke % EPC) * (FP16 ? 2 : 1);
        if (FP16) {
            uint4 w;
            w.x = c2[0];
            w.y = c2[1];
            w.z = c2[2];
            w.w = c2[3];
            *reinterpret_cast<uint4*>(dst) = w;
        } else {
            uint2 w;
            w.x = c2[0] | (c2[1] << 16);
            w.y = c2[2] | (c2[3] << 16);
            *reinterpret_cast<uint2*>(dst) = w;
        }
    }
}

// The same for FP8 codes of the eight values qs[e] / scale (integers times a power of two, scale a power of two): the
// scaled FP32 -> FP8 pair conversion of gfx950 divides by the scale, so the slice integer is converted from where it
// sits in the slicer's upper word, without a shift or a separate scaling.  Exact for the same reason as above.
__device__ __forceinline__ void store_fp8_codes_scaled(const int (&qs)[8], float scale, int64_t ke, uint8_t* dst_slice, int64_t v_rows_pad,
                                                       int64_t row) {
    typedef short short2v __attribute__((ext_vector_type(2)));
    uint32_t w[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        short2v r = {0, 0};
        r = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(r, (float)qs[4 * h], (float)qs[4 * h + 1], scale, false);
        r = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(r, (float)qs[4 * h + 2], (float)qs[4 * h + 3], scale, true);
        w[h] = __builtin_bit_cast(uint32_t, r);
    }
    const int64_t kc = ke / CHUNK_BYTES;
    uint8_t* dst = dst_slice + ((size_t)kc * v_rows_pad + row) * CHUNK_BYTES + (ke % CHUNK_BYTES);
    uint2 v;
    v.x = w[0];
    v.y = w[1];
    *reinterpret_cast<uint2*>(dst) = v;
}

// FP16 codes of eight slice values (exact: q 2^-b with |q| <= 2^b is a normal number of the format, or zero)
__device__ __forceinline__ void store_fp16_codes(const float (&f)[8], int64_t ke, uint8_t* dst_slice, int64_t v_rows_pad, int64_t row) {
    constexpr int EPC = CHUNK_BYTES / 2;
    uint4 w;
    w.x = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(f[0], f[1]));
    w.y = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(f[2], f[3]));
    w.z = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(f[4], f[5]));
    w.w = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(f[6], f[7]));
    *reinterpret_cast<uint4*>(dst_slice + ((size_t)(ke / EPC) * v_rows_pad + row) * CHUNK_BYTES + (ke % EPC) * 2) = w;
}

// Where the eight 6-bit codes of one octet of a vector go inside a slice matrix: a 32-bit and a 16-bit store (see
// store_codes).  The same for every slice, so a thread works it out once per octet.
struct Fp6Slot {
    size_t at32, at16;     // byte offsets from the slice matrix
    bool low32;            // the 32-bit store takes bits 0..31 of the 48 (else bits 16..47)
};
__device__ __forceinline__ Fp6Slot fp6_slot(int64_t ke, int64_t v_rows_pad, int64_t row) {
    const int64_t kc = ke / CHUNK_BYTES;
    const int o = (int)((ke % CHUNK_BYTES) / 8), g = o >> 2, j = o & 3;
    const size_t chunk = (size_t)kc * v_rows_pad * CHUNK_BYTES_FP6;
    const size_t p16 = chunk + ((size_t)g * v_rows_pad + row) * 16;
    const size_t p8 = chunk + (size_t)v_rows_pad * 32 + ((size_t)g * v_rows_pad + row) * 8;
    Fp6Slot s;
    s.at32 = j == 0 ? p16 : j == 1 ? p16 + 8 : j == 2 ? p16 + 12 : p8 + 4;
    s.at16 = j == 0 ? p16 + 4 : j == 1 ? p16 + 6 : j == 2 ? p8 : p8 + 2;
    s.low32 = (j & 1) == 0;
    return s;
}
// FP6 codes of the eight slice integers given as q * 2^pos (the slicer's upper word), stored at a precomputed slot.
// The code of the magnitude |q| 2^(K-b) (K = 4 for E2M3, 3 for E3M2) is the magnitude itself for E2M3 and a table
// entry for E3M2 (see encode_e2m3 / encode_e3m2); bit 5 is the sign.
template <int FMT>
__device__ __forceinline__ void store_fp6_codes_at_pos(const int (&qs)[8], int pos, int b, const Fp6Slot& slot, uint8_t* dst_slice) {
    constexpr int K = FMT == FMT_FP6_E3M2 ? 3 : 4;
    const int down = pos - (K - b);
    uint32_t c[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int x = qs[e];
        const uint32_t mag = (uint32_t)(x < 0 ? -x : x) >> down;
        const uint32_t sign = ((uint32_t)x >> 26) & 32u;
        c[e] = (FMT == FMT_FP6_E3M2 ? (uint32_t)((0xCBA986420ull >> (4 * mag)) & 0xFull) : mag) | sign;
    }
    const uint32_t lo32 = c[0] | (c[1] << 6) | (c[2] << 12) | (c[3] << 18) | (c[4] << 24) | (c[5] << 30);
    const uint32_t hi16 = (c[5] >> 2) | (c[6] << 4) | (c[7] << 10);
    *reinterpret_cast<uint32_t*>(dst_slice + slot.at32) = slot.low32 ? lo32 : (lo32 >> 16) | (hi16 << 16);
    *reinterpret_cast<uint16_t*>(dst_slice + slot.at16) = (uint16_t)(slot.low32 ? hi16 : lo32);
}

// INT8 codes of the eight slice integers given as q * 2^pos: the byte at bit pos of each
__device__ __forceinline__ void store_int8_codes_at_pos(const int (&qs)[8], int pos, int64_t ke, uint8_t* dst_slice, int64_t v_rows_pad, int64_t row) {
    uint32_t w[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        w[h] = __builtin_amdgcn_ubfe((uint32_t)qs[4 * h], pos, 8);
#pragma unroll
        for (int e = 1; e < 4; ++e) w[h] |= __builtin_amdgcn_ubfe((uint32_t)qs[4 * h + e], pos, 8) << (8 * e);
    }
    uint2 v;
    v.x = w[0];
    v.y = w[1];
    *reinterpret_cast<uint2*>(dst_slice + ((size_t)(ke / CHUNK_BYTES) * v_rows_pad + row) * CHUNK_BYTES + ke % CHUNK_BYTES) = v;
}

// smallest c with v * 2^(unit - F) <= 2^c, for v != 0
__device__ __forceinline__ int ceil_log2_scaled(uint64_t v, int unit, int F) {
    const int L = 64 - __clzll((long long)v);
    return unit - F + L - (((v & (v - 1)) == 0) ? 1 : 0);
}

// Maximum over the 64 lanes of a wave (of int or uint32_t), returned to all of them: data-parallel-primitive steps inside rows of 16 lanes
// (swap inside pairs, pairs inside quads, mirror the half rows, mirror the rows), then the last lane of a row is
// passed on to the next row(s), and lane 63 holds the maximum.
template <typename V>
__device__ __forceinline__ V wave_max(V v) {
    static_assert(sizeof(V) == 4, "one register per lane");
    auto step = [](V x, int y) { return (V)y > x ? (V)y : x; };
    v = step(v, __builtin_amdgcn_update_dpp((int)v, (int)v, 0xB1, 0xF, 0xF, false));      // quad_perm [1,0,3,2]
    v = step(v, __builtin_amdgcn_update_dpp((int)v, (int)v, 0x4E, 0xF, 0xF, false));      // quad_perm [2,3,0,1]
    v = step(v, __builtin_amdgcn_update_dpp((int)v, (int)v, 0x141, 0xF, 0xF, false));     // row_half_mirror
    v = step(v, __builtin_amdgcn_update_dpp((int)v, (int)v, 0x140, 0xF, 0xF, false));     // row_mirror
    v = step(v, __builtin_amdgcn_update_dpp((int)v, (int)v, 0x142, 0xA, 0xF, false));     // row_bcast15 into rows 1 and 3
    v = step(v, __builtin_amdgcn_update_dpp((int)v, (int)v, 0x143, 0xC, 0xF, false));     // row_bcast31 into rows 2 and 3
    return (V)__builtin_amdgcn_readlane((int)v, 63);
}

// The sum, in lane 63: the same steps; a row that a step leaves out adds zero.
__device__ __forceinline__ int wave_sum(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);
    return __builtin_amdgcn_readlane(v, 63);
}

// (At least four waves per SIMD, i.e. at most 128 registers: two 512-thread workgroups per CU, so that one computes while
// the other waits at its barrier.)
// A vector rarely fills its threads: a wave without elements in its second octet leaves that half of the work out, and with
// one octet per thread (U = 1, TPR = 256) the launch has only the waves that hold elements (4096 + 4096 vectors of 4097
// elements, nine FP8 slices: 0.40 ms with every octet worked on, 0.35 ms so; 0.36 ms with fewer waves per workgroup there too,
// whose number should stay a multiple of the four SIMDs).
template <int U, int TPR, int FMT>
__global__ void __launch_bounds__((TPR < 256 ? 256 : TPR)) __attribute__((amdgpu_waves_per_eu(4))) split_kernel(SplitArgs a) {
    constexpr bool FP16 = FMT == FMT_FP16;
    constexpr bool FP6 = fmt_is_fp6(FMT);
    constexpr int BLOCK = TPR < 256 ? 256 : TPR;
    constexpr int RPB = BLOCK / TPR;                  // vectors per workgroup
    constexpr int EPC = FP16 ? CHUNK_BYTES / 2 : CHUNK_BYTES;   // elements per chunk
    constexpr int ROWB = FP6 ? CHUNK_BYTES_FP6 : CHUNK_BYTES;   // bytes per vector and chunk
    constexpr bool WHOLE = RPB == 1;                  // the workgroup is one vector, of blockDim.x <= TPR threads
    constexpr int MAX_WAVES = TPR / 64;
    __shared__ int red[2][BLOCK / 64];

    const int tr = WHOLE ? threadIdx.x : threadIdx.x % TPR;
    const int threads = WHOLE ? blockDim.x : TPR;     // per vector
    // Workgroups are handed to the eight XCDs (each with an L2 of its own) round-robin by their index.  Neighbouring
    // vectors share the cache lines of the slice layout (a line holds the 16-byte pieces of eight vectors in the
    // FP6 planes, the 64-byte chunks of two vectors otherwise), so eight consecutive workgroups' worth of vectors go to the
    // SAME XCD, where the partial lines meet in one L2 before they are written back; the next eight go to the next XCD, so that
    // also an operand of few vectors is spread over all of them.  Each operand's share of the grid is a multiple of 64.
    const bool second = blockIdx.x >= a.wg_first;                    // which operand this workgroup works on
    const double* const vX = second ? a.v[1].X : a.v[0].X;
    const int64_t v_ldv = second ? a.v[1].ldv : a.v[0].ldv, es = second ? a.v[1].es : a.v[0].es;
    const int64_t v_rows = second ? a.v[1].rows : a.v[0].rows, v_rows_pad = second ? a.v[1].rows_pad : a.v[0].rows_pad;
    uint8_t* const v_slices = second ? a.v[1].slices : a.v[0].slices;
    int32_t* const v_exps = second ? a.v[1].exps : a.v[0].exps;
    int32_t* const v_l1 = second ? a.v[1].l1 : a.v[0].l1;
    const unsigned li = blockIdx.x - (second ? a.wg_first : 0u);     // index inside the operand's part of the grid
    const int64_t wg = (li & ~63u) + (li & 7) * 8 + ((li >> 3) & 7);
    const int64_t row = wg * RPB + threadIdx.x / TPR;
    const int64_t t = blockIdx.y;
    const int64_t k0 = t * a.kb;
    int64_t klen = a.k - k0;
    if (klen > a.kb) klen = a.kb;
    if (row >= v_rows) klen = 0;                      // padding vectors are all zero
    const int64_t padded = a.chunks * EPC;
    if (wg * RPB >= v_rows) {                         // padding vectors only: zero codes and c = 0 in every slice
        if (v_slices == nullptr) return;
        const int zero8[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        for (int p = 0; p < a.s; ++p) {
            uint8_t* const dst = v_slices + (size_t)((t * a.s + p) * a.chunks) * (size_t)v_rows_pad * ROWB;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t ke = 8 * ((int64_t)tr + (int64_t)threads * u);
                if (ke < padded) store_codes<FMT>(zero8, ke, dst, v_rows_pad, row, a.b);
            }
            if (tr == 0) v_exps[(t * a.s + p) * v_rows_pad + row] = 0;
            if (tr == 0 && v_l1 != nullptr) v_l1[(t * a.s + p) * v_rows_pad + row] = 0;
        }
        return;
    }
    if (WHOLE && MAX_WAVES > 1) {
        if (threadIdx.x < 2 * MAX_WAVES) red[threadIdx.x / MAX_WAVES][threadIdx.x % MAX_WAVES] = NO_ELEM;
        __syncthreads();
    }
    // Fixed-point scale of the working representation: an active element holds T = x^(p) / 2^(c_p - b) * 2^F as a
    // signed 64-bit integer.  |x^(p)| <= 2^(c_p) bounds |T| by 2^(b+F) = 2^60.
    const int F = 60 - a.b;

    bool nonfinite = false;
    int cmax = NO_ELEM;
    const double* src = vX + row * v_ldv + k0 * es;
    // the eight FP64 bit patterns of octet u of this thread (zeros beyond the block)
    auto load_octet = [&](int u, uint64_t (&bits)[8]) {
        const int64_t ke = 8 * ((int64_t)tr + (int64_t)threads * u);
        if (es == 1 && ke + 8 <= klen) {
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                const two_doubles w = *reinterpret_cast<const two_doubles*>(src + ke + 2 * h);
                bits[2 * h] = w.x;
                bits[2 * h + 1] = w.y;
            }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) bits[e] = (ke + e < klen) ? __double_as_longlong(src[(ke + e) * es]) : 0ull;
        }
    };
    // does this wave hold elements of the block in octet u?  (wave-uniform)
    auto wave_has = [&](int u) -> bool {
        return 8 * ((int64_t)__builtin_amdgcn_readfirstlane(tr & ~63) + (int64_t)threads * u) < padded;
    };
    // Eq. 4: c = max over the vector of ceil(log2 |x_i|); each thread contributes the maximum over its elements
    // (from the decoded inputs for the first slice, from the remainders afterwards)
    auto vector_max = [&](int val, int p) -> int {
        static_assert(TPR >= 64, "a wave never holds parts of two vectors");
        val = wave_max(val);
        if (MAX_WAVES > 1) {
            const int wave = threadIdx.x >> 6;
            if ((threadIdx.x & 63) == 0) red[p & 1][wave] = val;
            __syncthreads();
            const int w0 = (wave / MAX_WAVES) * MAX_WAVES;
#pragma unroll
            for (int w = 0; w < MAX_WAVES; ++w) {                    // entries of waves that are not there never change
                const int o = red[p & 1][w0 + w];
                val = o > val ? o : val;
            }
        }
        return val;
    };

    // FP16: sum |q| of the slices, if wanted.  A wave's share goes to LDS and is added up behind the barrier of the next exchange.
    __shared__ int l1_share[2][BLOCK / 64];
    auto share_l1 = [&](int p, int mine) {
        const int share = wave_sum(mine);
        if ((threadIdx.x & 63) == 0) l1_share[p & 1][threadIdx.x >> 6] = share;
    };
    auto store_l1 = [&](int p) {
        if (tr != 0) return;
        const int w0 = threadIdx.x >> 6;
        int sum = 0;
        for (int w = 0; w < threads / 64; ++w) sum += l1_share[p & 1][w0 + w];
        v_l1[(t * a.s + p) * v_rows_pad + row] = sum;
    };

    if (!FP16 || a.b <= 7) {
        // ---- slices of at most 7 bits: the element step on 32-bit words (slice_element.hpp)
        const int pos = F - 32, bias = (1 << (pos - 1)) - 1;
        const uint32_t keep = ~((1u << pos) - 1u);
        const float code_unit = ldexpf(1.0f, -(pos + a.b));            // q * 2^pos * code_unit = q * 2^-b, the slice value
        const float code_scale = ldexpf(1.0f, pos + a.b);              // q * 2^pos / code_scale = q * 2^-b, the slice value
        Fp6Slot slots[FP6 ? U : 1];                                    // FP6 only: where each octet's codes go inside a slice matrix
        if constexpr (FP6) {
#pragma unroll
            for (int u = 0; u < U; ++u) slots[u] = fp6_slot(8 * ((int64_t)tr + (int64_t)threads * u), v_rows_pad, row);
        }
        uint64_t T[8 * U];                                             // element state, see slice_element.hpp
        int pk[8 * U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            uint64_t bits[8];
            load_octet(u, bits);
#pragma unroll
            for (int e = 0; e < 8; ++e) decode_narrow(bits[e], F, T[8 * u + e], pk[8 * u + e], cmax, nonfinite);
        }
        if (nonfinite) atomicOr(a.flags, 1);
        int unit_prev = 0, unit = 0, c = 0, step = 0;
        uint8_t* dst_slice = nullptr;
        int kmax, kmin;
        uint32_t cd_wait;
        float l1 = 0.0f;                                               // FP16: sum |q| 2^-b of this thread's elements, exact
        // head of slice p: Eq. 4, the unit 2^(c-b) and the distance from the previous unit
        auto begin_slice = [&](int p) {
            cmax = vector_max(cmax, p);
            // count-only mode (slicing until the remainder is zero, paragraph before Eq. 4): something is left before
            // the (p+1)-th slice, so this vector needs at least p + 1 of them
            if (v_slices == nullptr && cmax != NO_ELEM && tr == 0) atomicMax(a.flags + 1, p + 1);
            c = (cmax == NO_ELEM) ? 0 : cmax;
            unit = c - a.b;
            step = unit_prev - unit;
            unit_prev = unit;
            dst_slice = v_slices + (size_t)((t * a.s + p) * a.chunks) * (size_t)v_rows_pad * ROWB;
            kmax = KEY_NONE_MAX;
            kmin = KEY_NONE_MIN;
            cd_wait = 0;
            if constexpr (FP16) {
                if (v_l1 != nullptr && p > 0) store_l1(p - 1);
                l1 = 0.0f;
            }
        };
        auto store_octet = [&](int u, int (&qs)[8]) {                   // qs: q * 2^pos
            const int64_t ke = 8 * ((int64_t)tr + (int64_t)threads * u);
            if constexpr (FMT == FMT_FP8) {
                if (ke < padded && v_slices != nullptr) store_fp8_codes_scaled(qs, code_scale, ke, dst_slice, v_rows_pad, row);
            } else if constexpr (FP16) {
                float f[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    f[e] = (float)qs[e] * code_unit;
                    l1 += fabsf(f[e]);
                }
                if (ke < padded && v_slices != nullptr) store_fp16_codes(f, ke, dst_slice, v_rows_pad, row);
            } else if constexpr (FP6) {
                if (ke < padded && v_slices != nullptr) store_fp6_codes_at_pos<FMT>(qs, pos, a.b, slots[u], dst_slice);
            } else {
                if (ke < padded && v_slices != nullptr) store_int8_codes_at_pos(qs, pos, ke, dst_slice, v_rows_pad, row);
            }
        };
        // tail of slice p: the exponent goes out, the thread forms its candidate for the next one
        auto end_slice = [&](int p, bool settled) {
            if (tr == 0 && v_slices != nullptr) v_exps[(t * a.s + p) * v_rows_pad + row] = c;
            if constexpr (FP16) {
                if (v_l1 != nullptr) share_l1(p, (int)ldexpf(l1, a.b));
            }
            bool needs_exact;
            cmax = narrow_candidate(kmax, kmin, unit, F, needs_exact);
            if (needs_exact) {                                         // the upper words cannot tell: all 64 bits of the remainders
                uint64_t mx = 0;
#pragma unroll
                for (int i = 0; i < 8 * U; ++i) {
                    const uint64_t ar = (settled || pk[i] == 0) ? narrow_abs(T[i]) : 0ull;
                    mx = ar > mx ? ar : mx;
                }
                cmax = narrow_candidate_exact(mx, unit, F);
            }
            const int cw = (int)cd_wait - CD_BIAS;
            cmax = (cd_wait != 0 && cw > cmax) ? cw : cmax;
        };
        // first the slices during which some element of this wave still waits ...
        int p = 0;
        for (bool settled = false; p < a.s && !settled; ++p) {
            begin_slice(p);
            const int step16 = step * 65536;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (u > 0 && !wave_has(u)) break;
                int qs[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) qs[e] = slice_narrow(T[8 * u + e], pk[8 * u + e], step16, pos, bias, keep, kmax, kmin, cd_wait);
                store_octet(u, qs);
            }
            settled = __ballot(cd_wait != 0) == 0ull;
            end_slice(p, false);
        }
        // ... then the rest: every element is in fixed-point form, one shift for all, no control words
        for (; p < a.s; ++p) {
            begin_slice(p);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (u > 0 && !wave_has(u)) break;
                int qs[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) qs[e] = slice_narrow_active(T[8 * u + e], step, pos, bias, keep, kmax, kmin);
                store_octet(u, qs);
            }
            end_slice(p, true);
        }
        if constexpr (FP16) {
            if (v_l1 != nullptr) {
                __syncthreads();
                store_l1(a.s - 1);
            }
        }
        return;
    }

    // ---- FP16 slices of more than 7 bits (blocks of fewer than 1024 elements): element state as described at decode_element
    int64_t tv[8 * U];
    int pk[8 * U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        uint64_t bits[8];
        load_octet(u, bits);
#pragma unroll
        for (int e = 0; e < 8; ++e) decode_element(bits[e], F, tv[8 * u + e], pk[8 * u + e], cmax, nonfinite);
    }
    if (nonfinite) atomicOr(a.flags, 1);

    int c_prev = 0;
    for (int p = 0; p < a.s; ++p) {
        cmax = vector_max(cmax, p);
        if (v_l1 != nullptr && p > 0) store_l1(p - 1);
        if (v_slices == nullptr) {
            if (cmax != NO_ELEM && tr == 0) atomicMax(a.flags + 1, p + 1);      // count-only mode
        }
        const int c = (cmax == NO_ELEM) ? 0 : cmax;
        const int unit = c - a.b;                                      // the slice's unit is 2^(c-b)
        // remainders of active elements were left in units of the previous slice: rescale them to this one (a
        // left shift, exact and inside 2^60 because every remainder is at most 2^c; 0 << anything stays 0)
        int rescale = p == 0 ? 0 : c_prev - c;
        rescale = rescale < 0 ? 0 : (rescale > 63 ? 63 : rescale);
        c_prev = c;

        // ---- Eq. 5-8 element by element, eight codes per store
        uint8_t* const dst_slice = v_slices + (size_t)((t * a.s + p) * a.chunks) * (size_t)v_rows_pad * ROWB;
        uint64_t rmax = 0;                                             // largest |remainder| of this thread's active elements
        int cdorm = NO_ELEM;                                           // largest cd of its still dormant elements
        int l1 = 0;
        const int64_t round_bias = ((int64_t)1 << (F - 1)) - 1;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (u > 0 && !wave_has(u)) break;
            int qs[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) qs[e] = slice_element(tv[8 * u + e], pk[8 * u + e], unit, rescale, F, round_bias, rmax, cdorm);
#pragma unroll
            for (int e = 0; e < 8; ++e) l1 += qs[e] < 0 ? -qs[e] : qs[e];
            const int64_t ke = 8 * ((int64_t)tr + (int64_t)threads * u);
            if (ke < padded && v_slices != nullptr) store_codes<FMT>(qs, ke, dst_slice, v_rows_pad, row, a.b);
        }
        if (tr == 0 && v_slices != nullptr) v_exps[(t * a.s + p) * v_rows_pad + row] = c;
        if (v_l1 != nullptr) share_l1(p, l1);
        // this thread's candidate for the next exponent: remainders are rmax * 2^(unit - F)
        cmax = cdorm;
        if (rmax != 0) {
            const int ca = ceil_log2_scaled(rmax, unit, F);
            cmax = ca > cmax ? ca : cmax;
        }
    }
    if (v_l1 != nullptr) {
        __syncthreads();
        store_l1(a.s - 1);
    }
}

// Blocks of at most 256 elements, slices of at most 7 bits: a wave per vector, four elements per lane.  (With eight, half the
// lanes of split_kernel are idle there and a thread's serial chain, which is what these launches take, is twice as long:
// 256 + 256 vectors of 256 elements, 12 FP8 slices: 13.5 -> 10 us; 256 + 8192 of 256: 50 -> 30 us.)  The steps are those of split_kernel.
template <int FMT>
__global__ void __launch_bounds__(256) slice_short_kernel(SplitArgs a) {
    constexpr bool FP6 = fmt_is_fp6(FMT);
    constexpr int ROWB = FP6 ? CHUNK_BYTES_FP6 : CHUNK_BYTES;
    const int lane = threadIdx.x & 63;
    const bool second = blockIdx.x >= a.wg_first;
    const SplitVectors& v = second ? a.v[1] : a.v[0];
    const unsigned li = blockIdx.x - (second ? a.wg_first : 0u);     // dealt to the XCDs as in split_kernel
    const int64_t row = ((int64_t)((li & ~63u) + (li & 7) * 8 + ((li >> 3) & 7))) * 4 + (threadIdx.x >> 6);
    const int64_t t = blockIdx.y;
    int64_t klen = a.k - t * a.kb;
    if (klen > a.kb) klen = a.kb;
    if (row >= v.rows) klen = 0;                                     // a padding vector: zero codes, c = 0
    const int ke = 4 * lane;
    const bool stores = ke < a.chunks * CHUNK_BYTES;
    const int F = 60 - a.b, pos = F - 32, bias = (1 << (pos - 1)) - 1;
    const uint32_t keep = ~((1u << pos) - 1u);
    const float code_scale = ldexpf(1.0f, pos + a.b);
    const double* const src = v.X + row * v.ldv + t * a.kb * v.es;
    uint64_t bits[4];
    if (v.es == 1 && ke + 4 <= klen) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const two_doubles w = *reinterpret_cast<const two_doubles*>(src + ke + 2 * h);
            bits[2 * h] = w.x;
            bits[2 * h + 1] = w.y;
        }
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) bits[e] = (ke + e < klen) ? (uint64_t)__double_as_longlong(src[(ke + e) * v.es]) : 0ull;
    }
    uint64_t T[4];
    int pk[4], cmax = NO_ELEM;
    bool nonfinite = false;
#pragma unroll
    for (int e = 0; e < 4; ++e) decode_narrow(bits[e], F, T[e], pk[e], cmax, nonfinite);
    if (nonfinite) atomicOr(a.flags, 1);

    const size_t slice_bytes = (size_t)a.chunks * v.rows_pad * ROWB;
    uint8_t* dst_slice = v.slices + (size_t)(t * a.s) * slice_bytes;
    // FP6: an even lane stores the 48 bits of its own four codes and its neighbour's
    const Fp6Slot slot = fp6_slot(ke & ~7, v.rows_pad, row);
    const size_t at = ((size_t)(ke / CHUNK_BYTES) * v.rows_pad + row) * CHUNK_BYTES + ke % CHUNK_BYTES;
    auto store = [&](const int (&qs)[4]) {                           // qs: q * 2^pos
        if constexpr (FP6) {
            constexpr int K = FMT == FMT_FP6_E3M2 ? 3 : 4;
            const int down = pos - (K - a.b);
            uint32_t w = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t mag = (uint32_t)(qs[e] < 0 ? -qs[e] : qs[e]) >> down, sign = ((uint32_t)qs[e] >> 26) & 32u;
                w |= ((FMT == FMT_FP6_E3M2 ? (uint32_t)((0xCBA986420ull >> (4 * mag)) & 0xFull) : mag) | sign) << (6 * e);
            }
            const uint32_t next = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0xB1, 0xF, 0xF, false);     // the other lane of the pair
            if (stores && (lane & 1) == 0) {
                const uint64_t w48 = (uint64_t)w | ((uint64_t)next << 24);
                *reinterpret_cast<uint32_t*>(dst_slice + slot.at32) = slot.low32 ? (uint32_t)w48 : (uint32_t)(w48 >> 16);
                *reinterpret_cast<uint16_t*>(dst_slice + slot.at16) = slot.low32 ? (uint16_t)(w48 >> 32) : (uint16_t)w48;
            }
        } else {
            uint32_t w = 0;
            if constexpr (FMT == FMT_FP8) {
                typedef short short2v __attribute__((ext_vector_type(2)));
                short2v r = {0, 0};
                r = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(r, (float)qs[0], (float)qs[1], code_scale, false);
                r = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(r, (float)qs[2], (float)qs[3], code_scale, true);
                w = __builtin_bit_cast(uint32_t, r);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) w |= __builtin_amdgcn_ubfe((uint32_t)qs[e], pos, 8) << (8 * e);
            }
            if (stores) *reinterpret_cast<uint32_t*>(dst_slice + at) = w;
        }
    };
    int unit_prev = 0, unit = 0, step = 0, kmax, kmin;
    uint32_t cd_wait;
    auto begin_slice = [&](int p) {
        cmax = wave_max(cmax);
        const int c = (cmax == NO_ELEM) ? 0 : cmax;
        unit = c - a.b;
        step = unit_prev - unit;
        unit_prev = unit;
        kmax = KEY_NONE_MAX;
        kmin = KEY_NONE_MIN;
        cd_wait = 0;
        if (lane == 0) v.exps[(t * a.s + p) * v.rows_pad + row] = c;
    };
    auto end_slice = [&](bool settled) {
        bool needs_exact;
        cmax = narrow_candidate(kmax, kmin, unit, F, needs_exact);
        if (needs_exact) {
            uint64_t mx = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint64_t ar = (settled || pk[i] == 0) ? narrow_abs(T[i]) : 0ull;
                mx = ar > mx ? ar : mx;
            }
            cmax = narrow_candidate_exact(mx, unit, F);
        }
        const int cw = (int)cd_wait - CD_BIAS;
        cmax = (cd_wait != 0 && cw > cmax) ? cw : cmax;
        dst_slice += slice_bytes;
    };
    int p = 0;
    for (bool settled = false; p < a.s && !settled; ++p) {
        begin_slice(p);
        int qs[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) qs[e] = slice_narrow(T[e], pk[e], step * 65536, pos, bias, keep, kmax, kmin, cd_wait);
        store(qs);
        settled = __ballot(cd_wait != 0) == 0ull;
        end_slice(false);
    }
    for (; p < a.s; ++p) {
        begin_slice(p);
        int qs[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) qs[e] = slice_narrow_active(T[e], step, pos, bias, keep, kmax, kmin);
        store(qs);
        end_slice(true);
    }
}

// ---- Blocks too long for the registers of one workgroup --------------------------------------------------------
// The remainders need not be carried from slice to slice: x^(p) differs from x by a multiple of the previous unit, which
// is an even multiple of this one (every remainder is at most half a unit, so the units 2^u_p shrink by b+1 bits or more),
// hence  x^(p+1) = x - (x rounded to a multiple of 2^u_p, ties to even)  directly from x.  So the exponents come first
// (long_exponents_kernel, remainder_key), from the elements alone, and with them known every element is sliced on its own
// (split_stream_kernel), with no exchange between threads and no state in memory: the block is read two or three times
// instead of once, plus 24 bytes of state, per slice.  256 + 320 vectors of 65536 elements, 11 FP8 slices: 6.3 ms with the
// state in memory, 0.49 ms so.

// How far an element's remainder at unit 2^u is from zero, in 2^-32 of the unit and rounded up: the key of the maximum in
// Eq. 4.  The remainder of mm * 2^E is the distance of its fraction f = mm 2^-sh mod 1 (sh = u - E) from the nearest
// integer; f is taken to 64 bits with the lowest one sticky.  With hi, lo its words, f < 1/2 gives hi + (lo != 0), f >= 1/2
// gives the same of 2^64 - f, which is -hi whether lo is zero or not.
__device__ __forceinline__ uint32_t fraction_key(uint64_t f) {
    const int hi = (int)(uint32_t)(f >> 32);
    const uint32_t up = (uint32_t)hi + ((uint32_t)f != 0 ? 1u : 0u);
    return hi < 0 ? 0u - (uint32_t)hi : up;
}
__device__ __forceinline__ uint64_t unit_fraction(uint64_t mm, int sh) {
    if (sh <= 0) return 0;                                           // a multiple of the unit
    if (sh <= 64) return mm << (64 - sh);
    const int r = sh - 64;                                           // far below the unit: cut, with a sticky lowest bit
    const uint64_t cut = r < 64 ? mm >> r : 0;
    return cut | ((r < 64 ? (cut << r) != mm : mm != 0) ? 1u : 0u);
}
// |remainder| at unit 2^(E + sh), in units of 2^E: exact
__device__ __forceinline__ uint64_t remainder_abs(uint64_t mm, int sh) {
    if (sh <= 0) return 0;
    if (sh > 54) return mm;
    const uint64_t low = mm & ((1ull << sh) - 1), up = (1ull << sh) - low;
    return low < up ? low : up;
}

constexpr int LEVELS = 12;            // units tried per reading of the block

// Eq. 4 for all slices of one vector and block.  With enough elements a unit's largest remainder is nearly half the unit, so
// that the next unit is b+1 bits down: the keys of the next LEVELS units of that ladder are formed in one reading, and the
// ladder is followed as far as the keys confirm it; the first exponent off it is known from them too, and another reading
// starts there.
__global__ void __launch_bounds__(1024) long_exponents_kernel(SplitArgs a) {
    __shared__ uint32_t red[LEVELS][16];
    const int tid = threadIdx.x, wave = tid >> 6;
    const bool second = blockIdx.x >= a.wg_first;
    const SplitVectors& v = second ? a.v[1] : a.v[0];
    const int64_t row = blockIdx.x - (second ? a.wg_first : 0u);
    const int64_t t = blockIdx.y;
    int64_t klen = a.k - t * a.kb;
    if (klen > a.kb) klen = a.kb;
    int32_t* const exps = v.exps != nullptr ? v.exps + t * a.s * v.rows_pad + row : nullptr;
    if (row >= v.rows) {                                             // a padding vector: c = 0 throughout
        if (exps != nullptr && tid < a.s) exps[(int64_t)tid * v.rows_pad] = 0;
        return;
    }
    const double* const src = v.X + row * v.ldv + t * a.kb;
    // maximum over the workgroup of `count` keys per thread, left in red[0 .. count-1][0]
    auto block_max = [&](uint32_t (&keys)[LEVELS], int count) {
        __syncthreads();                                             // the previous maxima have been read
#pragma unroll
        for (int j = 0; j < LEVELS; ++j) {
            if (j < count) {
                const uint32_t m = wave_max(keys[j]);
                if ((tid & 63) == 0) red[j][wave] = m;
            }
        }
        __syncthreads();
        if (tid < LEVELS) {
            uint32_t m = red[tid][0];
#pragma unroll
            for (int w = 1; w < 16; ++w) m = red[tid][w] > m ? red[tid][w] : m;
            red[tid][0] = m;
        }
        __syncthreads();
    };
    // f(mm, E) for every element of the block, four 16-byte loads in flight per thread
    auto for_each = [&](auto f) {
        auto one = [&](uint64_t w) {
            const int e11 = (int)((w >> 52) & 0x7FF);
            uint64_t mm = w & 0x000FFFFFFFFFFFFFull;
            if (e11 != 0) mm |= 0x0010000000000000ull;
            f(mm, e11 != 0 ? e11 - 1075 : -1074);
        };
        int64_t i = 0;
        for (; i + 8192 <= klen; i += 8192) {
            two_doubles w[4];
#pragma unroll
            for (int h = 0; h < 4; ++h) w[h] = *reinterpret_cast<const two_doubles*>(src + i + h * 2048 + 2 * tid);
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                one(w[h].x);
                one(w[h].y);
            }
        }
        for (i += tid; i < klen; i += 1024) one((uint64_t)__double_as_longlong(src[i]));
    };

    uint32_t keys[LEVELS];
#pragma unroll
    for (int j = 0; j < LEVELS; ++j) keys[j] = 0;
    bool nonfinite = false;
    auto exponent_key = [&](uint64_t mm, int E) -> uint32_t {         // ceil log2 of a non-zero mm * 2^E, biased; 0 for zero
        return mm == 0 ? 0u : (uint32_t)(E + bit_length_u64(mm) - (((mm & (mm - 1)) == 0) ? 1 : 0) + CD_BIAS);
    };
    for_each([&](uint64_t mm, int E) {
        nonfinite |= E == 0x7FF - 1075;
        const uint32_t key = exponent_key(mm, E);
        keys[0] = key > keys[0] ? key : keys[0];
    });
    if (nonfinite) atomicOr(a.flags, 1);
    block_max(keys, 1);
    int p = 0, c = 0;
    bool left = red[0][0] != 0;                                      // is there a remainder before slice p?
    const bool any = left;
    if (left) c = (int)red[0][0] - CD_BIAS;
    if (exps != nullptr && tid == 0) exps[0] = c;
    while (left && p + 1 < a.s) {
        const int unit0 = c - a.b, step = a.b + 1;
        const int levels = a.s - 1 - p < LEVELS ? a.s - 1 - p : LEVELS;
#pragma unroll
        for (int j = 0; j < LEVELS; ++j) keys[j] = 0;
        for_each([&](uint64_t mm, int E) {
            const int sh = unit0 - E;
            if (sh <= 64) {
                uint64_t f = unit_fraction(mm, sh);
#pragma unroll
                for (int j = 0; j < LEVELS; ++j) {
                    const uint32_t key = fraction_key(f);
                    keys[j] = key > keys[j] ? key : keys[j];
                    f <<= step;
                }
            } else {
#pragma unroll
                for (int j = 0; j < LEVELS; ++j) {
                    const uint32_t key = fraction_key(unit_fraction(mm, sh - j * step));
                    keys[j] = key > keys[j] ? key : keys[j];
                }
            }
        });
        block_max(keys, levels);
        for (int j = 0; j < levels; ++j) {
            const uint32_t key = red[j][0];
            const int unit = unit0 - j * step;
            left = key != 0;
            if (!left) break;
            if (key > 1) {
                c = unit - 32 + bit_length_u32(key - 1);             // smallest c with key * 2^(unit-32) <= 2^c
            } else {
                // every remainder is at most 2^-32 of the unit: look at all their bits
                uint32_t exact[LEVELS];
#pragma unroll
                for (int i = 0; i < LEVELS; ++i) exact[i] = 0;
                for_each([&](uint64_t mm, int E) {
                    const uint32_t k = exponent_key(remainder_abs(mm, unit - E), E);
                    exact[0] = k > exact[0] ? k : exact[0];
                });
                block_max(exact, 1);
                c = (int)red[0][0] - CD_BIAS;
            }
            ++p;
            if (exps != nullptr && tid == 0) exps[(int64_t)p * v.rows_pad] = c;
            if (key == 1 || c - a.b != unit - step) break;           // off the ladder (or its keys are overwritten): read again
        }
    }
    // nothing left: the remaining slices are zero (c := 0); without slices to write, report how many there are
    if (exps != nullptr && !left)
        for (int i = p + 1 + tid; i < a.s; i += 1024) exps[(int64_t)i * v.rows_pad] = 0;
    if (v.slices == nullptr && tid == 0 && any) atomicMax(a.flags + 1, p + 1);
}

// All slices of one chunk (64 inner indices; FP16: 32) of 32 (64) consecutive vectors, with the exponents known: eight
// elements per thread, whose state goes from slice to slice in registers; what the workgroup stores of a slice is 2 KiB
// (4 KiB) in one piece.
template <int FMT>
__global__ void __launch_bounds__(256) split_stream_kernel(SplitArgs a) {
    constexpr bool FP16 = FMT == FMT_FP16;
    constexpr int EPC = FP16 ? CHUNK_BYTES / 2 : CHUNK_BYTES;
    constexpr int ROWB = fmt_is_fp6(FMT) ? CHUNK_BYTES_FP6 : CHUNK_BYTES;
    constexpr int OCTETS = EPC / 8, ROWS = 256 / OCTETS;
    const int64_t wg = blockIdx.x;
    const bool second = wg >= a.wg_first;
    const SplitVectors& v = second ? a.v[1] : a.v[0];
    const int64_t li = wg - (second ? a.wg_first : 0u);
    const int64_t row_groups = v.rows_pad / ROWS;
    const int64_t kc = li / row_groups, row = (li - kc * row_groups) * ROWS + threadIdx.x / OCTETS;
    const int64_t t = blockIdx.y;
    int64_t klen = a.k - t * a.kb;
    if (klen > a.kb) klen = a.kb;
    if (row >= v.rows) klen = 0;                                     // padding vectors are all zero
    const int64_t ke = kc * EPC + (threadIdx.x % OCTETS) * 8;
    const double* const src = v.X + row * v.ldv + t * a.kb;
    const int F = 60 - a.b;
    const int32_t* const exps = v.exps + t * a.s * v.rows_pad + row;
    uint8_t* dst_slice = v.slices + (size_t)(t * a.s) * a.chunks * (size_t)v.rows_pad * ROWB;
    const size_t slice_bytes = (size_t)a.chunks * v.rows_pad * ROWB;
    uint64_t bits[8];
    if (ke + 8 <= klen) {
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const two_doubles w = *reinterpret_cast<const two_doubles*>(src + ke + 2 * h);
            bits[2 * h] = w.x;
            bits[2 * h + 1] = w.y;
        }
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) bits[e] = (ke + e < klen) ? (uint64_t)__double_as_longlong(src[ke + e]) : 0ull;
    }
    int cmax = NO_ELEM;
    bool nonfinite = false;                                          // long_exponents_kernel has reported it
    // Blocks this long leave FP16 slices 4 bits at most, so the 32-bit element step serves every format.
    const int pos = F - 32, bias = (1 << (pos - 1)) - 1;
    const uint32_t keep = ~((1u << pos) - 1u);
    const float code_scale = ldexpf(1.0f, pos + a.b), code_unit = ldexpf(1.0f, -(pos + a.b));
    const Fp6Slot slot = fp6_slot(ke, v.rows_pad, row);
    auto store = [&](const int (&qs)[8]) {                           // qs: q * 2^pos
        if constexpr (FMT == FMT_FP8) {
            store_fp8_codes_scaled(qs, code_scale, ke, dst_slice, v.rows_pad, row);
        } else if constexpr (FMT == FMT_INT8) {
            store_int8_codes_at_pos(qs, pos, ke, dst_slice, v.rows_pad, row);
        } else if constexpr (FP16) {
            float f[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) f[e] = (float)qs[e] * code_unit;
            store_fp16_codes(f, ke, dst_slice, v.rows_pad, row);
        } else {
            store_fp6_codes_at_pos<FMT>(qs, pos, a.b, slot, dst_slice);
        }
    };
    uint64_t T[8];
    int pk[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) decode_narrow(bits[e], F, T[e], pk[e], cmax, nonfinite);
    int unit_prev = 0, kmax = KEY_NONE_MAX, kmin = KEY_NONE_MIN, p = 0;
    // while some element of the wave waits for its unit, then one shift for all (as in split_kernel)
    for (bool settled = false; p < a.s && !settled; ++p, dst_slice += slice_bytes) {
        const int unit = exps[(int64_t)p * v.rows_pad] - a.b;
        const int step16 = (unit_prev - unit) * 65536;
        unit_prev = unit;
        int qs[8];
        uint32_t cd_wait = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) qs[e] = slice_narrow(T[e], pk[e], step16, pos, bias, keep, kmax, kmin, cd_wait);
        store(qs);
        settled = __ballot(cd_wait != 0) == 0ull;
    }
    for (; p < a.s; ++p, dst_slice += slice_bytes) {
        const int unit = exps[(int64_t)p * v.rows_pad] - a.b, step = unit_prev - unit;
        unit_prev = unit;
        int qs[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) qs[e] = slice_narrow_active(T[e], step, pos, bias, keep, kmax, kmin);
        store(qs);
    }
}

template <int FMT>
__global__ void __launch_bounds__(256) export_slices_kernel(const uint8_t* __restrict__ slices, int64_t rows, int64_t rows_pad,
                                                            int64_t k, int64_t kb, int64_t chunks, int s, void* out) {
    // plain layout: block t starts at s*rows*(t*kb) entries; inside, [p][row][kb_t]
    constexpr bool FP16 = FMT == FMT_FP16;
    constexpr bool FP6 = fmt_is_fp6(FMT);
    constexpr int EPC = FP16 ? CHUNK_BYTES / 2 : CHUNK_BYTES;
    constexpr int ROWB = FP6 ? CHUNK_BYTES_FP6 : CHUNK_BYTES;
    const int64_t t = blockIdx.z, p = blockIdx.y;
    int64_t klen = k - t * kb;
    if (klen > kb) klen = kb;
    const int64_t total = rows * klen;
    const uint8_t* src = slices + (size_t)((t * s + p) * chunks) * (size_t)rows_pad * ROWB;
    const size_t out_base = (size_t)s * rows * (t * kb) + (size_t)p * rows * klen;
    for (int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (int64_t)gridDim.x * 256) {
        const int64_t r = idx / klen, kk = idx % klen;
        if constexpr (FP6) {
            // code i of k-group g sits at bits 6i .. 6i+5 of a 24-byte string: bytes 0..15 in the 16-byte plane of g,
            // bytes 16..23 in its 8-byte plane
            const uint8_t* chunk = src + (size_t)(kk / EPC) * rows_pad * ROWB;
            const int e = (int)(kk % EPC), g = e >> 5, bit = (e & 31) * 6;
            const uint8_t* p16 = chunk + ((size_t)g * rows_pad + r) * 16;
            const uint8_t* p8 = chunk + (size_t)rows_pad * 32 + ((size_t)g * rows_pad + r) * 8;
            const int b0 = bit >> 3, b1 = (bit + 5) >> 3;
            const uint32_t lo = b0 < 16 ? p16[b0] : p8[b0 - 16], hi = b1 < 16 ? p16[b1] : p8[b1 - 16];
            reinterpret_cast<uint8_t*>(out)[out_base + idx] = (uint8_t)((((hi << 8) | lo) >> (bit & 7)) & 63u);
        } else {
            const size_t off = ((size_t)(kk / EPC) * rows_pad + r) * CHUNK_BYTES + (kk % EPC) * (FP16 ? 2 : 1);
            if (FP16) reinterpret_cast<uint16_t*>(out)[out_base + idx] = *reinterpret_cast<const uint16_t*>(src + off);
            else reinterpret_cast<uint8_t*>(out)[out_base + idx] = src[off];
        }
    }
}

// One workgroup per 256 vectors and block, one half-wave per group of 32 vectors: for every slice p, is c_p - c_(p+1)
// the same for all real vectors of the group?  The first tiles_first workgroups of a grid row belong to the first
// operand, the rest to the second.
struct DeltaOperand {
    const int32_t* exps;
    int32_t* deltas;
    const int32_t* l1;
    int32_t* bounds;
    int64_t rows, rows_pad;
};
__global__ void __launch_bounds__(256) delta_kernel(DeltaOperand o0, DeltaOperand o1, unsigned tiles_first, int s, int b) {
    const bool second = blockIdx.x >= tiles_first;
    const int32_t* const exps = second ? o1.exps : o0.exps;
    int32_t* const deltas = second ? o1.deltas : o0.deltas;
    const int64_t rows = second ? o1.rows : o0.rows, rows_pad = second ? o1.rows_pad : o0.rows_pad;
    const int64_t tile = blockIdx.x - (second ? tiles_first : 0u), groups = rows_pad / LINK_ROWS, t = blockIdx.y;
    const int64_t row = tile * TILE + threadIdx.x;
    const int64_t group = row / LINK_ROWS;
    const int lane = threadIdx.x & 63, half = lane & 32;
    const int32_t* e = exps + (size_t)t * s * rows_pad;
    int32_t* out = deltas + (size_t)t * s * groups + group;          // slice p of this group at out[p * groups]
    for (int p = 0; p + 1 < s; ++p) {
        const int d = e[(size_t)p * rows_pad + row] - e[(size_t)(p + 1) * rows_pad + row];
        // the first vector of a group is a real one, or the whole group is padding (then every d is 0)
        const int ref = __shfl(d, half, 64);
        const unsigned long long ok = __ballot(row >= rows || d == ref);
        const bool same = (uint32_t)(ok >> half) == 0xFFFFFFFFu;
        if ((lane & 31) == 0) out[(size_t)p * groups] = same ? ref : DELTA_IRREGULAR;
    }
    if ((lane & 31) == 0) out[(size_t)(s - 1) * groups] = DELTA_IRREGULAR;
    const int32_t* const l1 = second ? o1.l1 : o0.l1;
    if (l1 == nullptr) return;
    // Operand::bounds: 2^b times the largest sum |q| of the group
    int32_t* const bounds = (second ? o1.bounds : o0.bounds) + (size_t)t * s * groups + group;
    for (int p = 0; p < s; ++p) {
        int most = l1[(size_t)(t * s + p) * rows_pad + row];
#pragma unroll
        for (int off = 1; off < 32; off <<= 1) {
            const int o = __shfl_xor(most, off, 64);
            most = o > most ? o : most;
        }
        if ((lane & 31) == 0) bounds[(size_t)p * groups] = most << b;
    }
}

template <int U, int TPR>
hipError_t launch_split_cfg(const SplitArgs& a_in, int fmt, int64_t T, hipStream_t st) {
    constexpr int BLOCK = TPR < 256 ? 256 : TPR;
    constexpr int RPB = BLOCK / TPR;
    SplitArgs a = a_in;
    a.wg_first = (unsigned)(a.v[0].rows_pad / RPB);                     // rows_pad is a multiple of 256, RPB <= 4
    dim3 grid(a.wg_first + (unsigned)(a.v[1].rows_pad / RPB), (unsigned)T);
    const int64_t octets = a.chunks * (fmt == FMT_FP16 ? CHUNK_BYTES / 2 : CHUNK_BYTES) / 8;
    const unsigned threads = RPB == 1 && U == 1 ? (unsigned)((octets + 64 * U - 1) / (64 * U)) * 64u : BLOCK;
    if (fmt == FMT_FP16) hipLaunchKernelGGL((split_kernel<U, TPR, FMT_FP16>), grid, dim3(threads), 0, st, a);
    else if (fmt == FMT_FP6) hipLaunchKernelGGL((split_kernel<U, TPR, FMT_FP6>), grid, dim3(threads), 0, st, a);
    else if (fmt == FMT_FP6_E3M2) hipLaunchKernelGGL((split_kernel<U, TPR, FMT_FP6_E3M2>), grid, dim3(threads), 0, st, a);
    else if (fmt == FMT_INT8) hipLaunchKernelGGL((split_kernel<U, TPR, FMT_INT8>), grid, dim3(threads), 0, st, a);
    else hipLaunchKernelGGL((split_kernel<U, TPR, FMT_FP8>), grid, dim3(threads), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_split_short(const SplitArgs& a_in, int fmt, int64_t T, hipStream_t st) {
    SplitArgs a = a_in;
    a.wg_first = (unsigned)(a.v[0].rows_pad / 4);
    const dim3 grid(a.wg_first + (unsigned)(a.v[1].rows_pad / 4), (unsigned)T), block(256);
    if (fmt == FMT_FP6) hipLaunchKernelGGL((slice_short_kernel<FMT_FP6>), grid, block, 0, st, a);
    else if (fmt == FMT_FP6_E3M2) hipLaunchKernelGGL((slice_short_kernel<FMT_FP6_E3M2>), grid, block, 0, st, a);
    else if (fmt == FMT_INT8) hipLaunchKernelGGL((slice_short_kernel<FMT_INT8>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((slice_short_kernel<FMT_FP8>), grid, block, 0, st, a);
    return hipGetLastError();
}

// blocks too long for the register-resident kernel: exponents first (one workgroup per vector and block), then the slices
hipError_t launch_split_long(const SplitArgs& a_in, int fmt, int64_t T, hipStream_t st) {
    SplitArgs a = a_in;
    a.wg_first = (unsigned)a.v[0].rows_pad;
    hipLaunchKernelGGL(long_exponents_kernel, dim3(a.wg_first + (unsigned)a.v[1].rows_pad, (unsigned)T), dim3(1024), 0, st, a);
    if (a.v[0].slices == nullptr && a.v[1].slices == nullptr) return hipGetLastError();      // count only
    const int rows = fmt == FMT_FP16 ? 64 : 32;                                              // vectors per workgroup
    const int64_t first = a.v[0].rows_pad / rows * a.chunks, rest = a.v[1].rows_pad / rows * a.chunks;
    if (first + rest > 0x7FFFFFFF) return hipErrorInvalidValue;
    a.wg_first = (unsigned)first;
    const dim3 grid((unsigned)(first + rest), (unsigned)T), block(256);
    if (fmt == FMT_FP16) hipLaunchKernelGGL((split_stream_kernel<FMT_FP16>), grid, block, 0, st, a);
    else if (fmt == FMT_FP6) hipLaunchKernelGGL((split_stream_kernel<FMT_FP6>), grid, block, 0, st, a);
    else if (fmt == FMT_FP6_E3M2) hipLaunchKernelGGL((split_stream_kernel<FMT_FP6_E3M2>), grid, block, 0, st, a);
    else if (fmt == FMT_INT8) hipLaunchKernelGGL((split_stream_kernel<FMT_INT8>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((split_stream_kernel<FMT_FP8>), grid, block, 0, st, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_transpose(const double* A, int64_t lda, int64_t m, int64_t k, double* At, hipStream_t st) {
    if (m == 0 || k == 0) return hipSuccess;
    dim3 grid((unsigned)((m + 31) / 32), (unsigned)((k + 31) / 32));
    hipLaunchKernelGGL(transpose_kernel, grid, dim3(256), 0, st, A, lda, m, k, At);
    return hipGetLastError();
}

namespace {
SplitVectors split_vectors(const double* X, int64_t ldv, int64_t es, const Operand* op) {
    SplitVectors v;
    memset(&v, 0, sizeof(v));
    if (op == nullptr || op->rows == 0) return v;                                 // no vectors: no workgroups
    v.X = X; v.ldv = ldv; v.es = es; v.rows = op->rows; v.rows_pad = op->rows_pad; v.slices = op->slices; v.exps = op->exps; v.l1 = op->l1;
    return v;
}
}  // namespace

hipError_t launch_split(const double* X0, int64_t ldv0, int64_t es0, const Operand* op0, const double* X1, int64_t ldv1, const Operand* op1,
                        const Plan& pl, int* flags, hipStream_t st) {
    SplitArgs a;
    a.v[0] = split_vectors(X0, ldv0, es0, op0);
    a.v[1] = split_vectors(X1, ldv1, 1, op1);
    a.wg_first = 0;
    a.k = pl.k; a.kb = pl.kb; a.chunks = pl.chunks; a.s = pl.s; a.b = pl.b; a.flags = flags;
    if (a.v[0].rows_pad + a.v[1].rows_pad == 0 || pl.T == 0) return hipSuccess;
    const int64_t vectors = (a.v[0].rows_pad + a.v[1].rows_pad) * pl.T;
    const int fmt = pl.fmt;
    if (pl.kb > MAX_K_BLOCK_IN_REGISTERS && es0 != 1) return hipErrorInvalidValue;
    if (pl.kb > MAX_K_BLOCK_IN_REGISTERS) return launch_split_long(a, fmt, pl.T, st);
    const int64_t octets = pl.chunks * pl.epc / 8;                              // per vector and block, padded
    // sixteen elements per thread (U = 2) is the measured optimum: more elements per thread cost registers and with
    // them the occupancy that hides the latency of the dependent integer chains (64 per thread: one wave per SIMD)
    if (octets <= 32 && fmt != FMT_FP16 && (a.v[0].slices != nullptr || a.v[1].slices != nullptr)) return launch_split_short(a, fmt, pl.T, st);
    if (octets <= 64) return launch_split_cfg<1, 64>(a, fmt, pl.T, st);
    // a small problem (few vectors) is bound by the length of a thread's dependent chain, not by throughput: eight
    // elements per thread there (1024 x 1024: 0.080 -> 0.065 ms for both operands; no gain from 2048 vectors on)
    if (vectors <= 2048) {
        if (octets <= 128) return launch_split_cfg<1, 128>(a, fmt, pl.T, st);
        if (octets <= 256) return launch_split_cfg<1, 256>(a, fmt, pl.T, st);
    }
    if (octets <= 128) return launch_split_cfg<2, 64>(a, fmt, pl.T, st);
    if (octets <= 256) return launch_split_cfg<2, 128>(a, fmt, pl.T, st);
    if (octets <= 512) return launch_split_cfg<2, 256>(a, fmt, pl.T, st);
    if (octets <= 1024) return launch_split_cfg<2, 512>(a, fmt, pl.T, st);
    if (octets <= 2048) return launch_split_cfg<2, 1024>(a, fmt, pl.T, st);
    // 32 elements per thread would cover blocks of up to 32768 elements, but at the 128 registers a thread of a
    // 1024-thread workgroup has, that variant lives on more than a hundred spilled registers; such blocks are streamed
    return hipErrorInvalidValue;
}

hipError_t launch_count_slices(const double* X, int64_t ldv, const Plan& pl, int64_t rows, int* flags, hipStream_t st) {
    Plan cp = pl;
    cp.s = MAX_SLICES + 1;                       // one more than the library can use: "not exhausted" is reported as 33
    Operand op;
    op.rows = rows;
    op.rows_pad = (rows + TILE - 1) / TILE * TILE;
    op.slices = nullptr; op.exps = nullptr; op.deltas = nullptr; op.l1 = nullptr; op.bounds = nullptr;
    return launch_split(X, ldv, 1, &op, nullptr, 0, nullptr, cp, flags, st);
}

hipError_t launch_deltas(const Plan& pl, const Operand* op0, const Operand* op1, hipStream_t st) {
    DeltaOperand o[2];
    memset(o, 0, sizeof(o));
    const Operand* ops[2] = {op0, op1};
    for (int i = 0; i < 2; ++i)
        if (ops[i] != nullptr && ops[i]->rows > 0) o[i] = DeltaOperand{ops[i]->exps, ops[i]->deltas, ops[i]->l1, ops[i]->bounds, ops[i]->rows, ops[i]->rows_pad};
    const unsigned t0 = (unsigned)(o[0].rows_pad / TILE), t1 = (unsigned)(o[1].rows_pad / TILE);
    if (t0 + t1 == 0 || pl.T == 0 || pl.s == 0) return hipSuccess;
    hipLaunchKernelGGL(delta_kernel, dim3(t0 + t1, (unsigned)pl.T), dim3(256), 0, st, o[0], o[1], t0, pl.s, pl.b);
    return hipGetLastError();
}

hipError_t launch_export_slices(const Plan& pl, const Operand& op, void* out, hipStream_t st) {
    if (op.rows == 0 || pl.k == 0) return hipSuccess;
    dim3 grid(1024, (unsigned)pl.s, (unsigned)pl.T);
    if (pl.fmt == FMT_FP16)
        hipLaunchKernelGGL((export_slices_kernel<FMT_FP16>), grid, dim3(256), 0, st, op.slices, op.rows, op.rows_pad, pl.k, pl.kb, pl.chunks, pl.s, out);
    else if (fmt_is_fp6(pl.fmt))
        hipLaunchKernelGGL((export_slices_kernel<FMT_FP6>), grid, dim3(256), 0, st, op.slices, op.rows, op.rows_pad, pl.k, pl.kb, pl.chunks, pl.s, out);
    else
        hipLaunchKernelGGL((export_slices_kernel<FMT_FP8>), grid, dim3(256), 0, st, op.slices, op.rows, op.rows_pad, pl.k, pl.kb, pl.chunks, pl.s, out);
    return hipGetLastError();
}

}  // namespace ozaki
