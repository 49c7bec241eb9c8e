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
// subtraction of sigma is exact.  The kernels compute the same q with integers; no FP64 instruction is executed.
//   * Blocks of up to 16384 elements: the slices of an element are read off one 96-bit fixed-point number, and the exponents of all of
//     them off one OR over the vector (slice_digits.hpp, slice_vectors).
//   * Longer blocks in two kernels (long_exponents_kernel, split_stream_kernel), the second of which carries the remainders from
//     slice to slice where the units do not follow the regular ladder (slice_element.hpp).
// HBM sees each input element once (long blocks: two or three times; a vector whose slices reach below 96 bits once more per 96) and
// each slice code once.
#include <string.h>

#include "deltas.hpp"
#include "layout.hpp"
#include "slice_digits.hpp"
#include "slice_element.hpp"

#include <type_traits>

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
    uint8_t* off_ladder;   // is a slice's exponent more than b + 1 below that of the slice before? (null: not wanted)
};

// A launch splits the vectors of up to two operands (same k, block length, format and slice count): the first wg_first
// workgroups of the grid belong to v[0], the rest to v[1].
struct SplitArgs {
    SplitVectors v[2];
    unsigned wg_first;     // a multiple of 64
    int64_t k, kb;
    int64_t chunks;        // chunks per block
    int s, b;
    DigitLadder ladder;    // of b
    int* flags;            // [0]: non-finite input seen; [1]: slice count (count-only mode); OffLadder's counts, cleared here
};

// (not in slice_short_kernel: such blocks are below ladder_pays' line)
__device__ __forceinline__ void clear_off_ladder(const SplitArgs& a) {
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < 2) a.flags[OFF_LADDER_FLAG + threadIdx.x] = 0;
}

// FP8 codes of the eight values qs[e] / scale (integers times a power of two, scale a power of two): the
// scaled FP32 -> FP8 pair conversion of gfx950 divides by the scale, so the slice integer is converted from where it
// sits in the slicer's upper word, without a shift or a separate scaling.  Exact: q 2^-b with |q| <= 2^b is a number of the format.
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

// Where the 6-bit codes of one octet of a vector go inside a slice matrix.  Four octets are the 24 bytes of a k-group: 16 in
// one plane, 8 in another.  Octets 0, 1 and 3 of the group store eight of them each, with the neighbours' share; stored octet by octet, as
// 4 and 2 bytes, they are twice the accesses to lines of the cache, and these are what the slicing of FP6 spends its time on.
struct Fp6Slot {
    size_t at;             // byte offset from the slice matrix
    uint32_t low, high;    // byte selections of the two words
    bool last, stores;     // octet 3, octets 0, 1 and 3
};
__device__ __forceinline__ Fp6Slot fp6_slot(int64_t ke, int64_t v_rows_pad, int64_t row) {
    const int64_t kc = ke / CHUNK_BYTES;
    const int o = (int)((ke % CHUNK_BYTES) / 8), g = o >> 2, j = o & 3;
    const size_t chunk = (size_t)kc * v_rows_pad * CHUNK_BYTES_FP6;
    const size_t p16 = chunk + ((size_t)g * v_rows_pad + row) * 16;
    const size_t p8 = chunk + (size_t)v_rows_pad * 32 + ((size_t)g * v_rows_pad + row) * 8;
    return Fp6Slot{j == 0 ? p16 : j == 1 ? p16 + 8 : p8, j == 0 ? 0x03020100u : j == 1 ? 0x05040302u : 0x01000504u,
                   j == 0 ? 0x01000504u : j == 1 ? 0x03020100u : 0x05040302u, j == 3, j != 2};
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

// Maximum and bitwise OR over the 64 lanes of a wave, returned to all of them: data-parallel-primitive steps inside rows of 16 lanes
// (swap inside pairs, pairs inside quads, mirror the half rows, mirror the rows), then the last lane of a row is passed on to the next
// row(s), and lane 63 holds the result.  A row that a step leaves out takes part with 0, which lets the compiler make one instruction of
// the move and the operation.
template <typename F>
__device__ __forceinline__ uint32_t wave_combine(uint32_t v, F f) {
    v = f(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true));       // quad_perm [1,0,3,2]
    v = f(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true));       // quad_perm [2,3,0,1]
    v = f(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true));      // row_half_mirror
    v = f(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, true));      // row_mirror
    v = f(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false));     // row_bcast15 into rows 1 and 3
    v = f(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false));     // row_bcast31 into rows 2 and 3
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
    return wave_combine(v, [](uint32_t x, uint32_t y) { return x > y ? x : y; });
}
__device__ __forceinline__ uint32_t wave_or(uint32_t v) {
    return wave_combine(v, [](uint32_t x, uint32_t y) { return x | y; });
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

// Type2 codes of G consecutive slice integers (G = 8, or 4 in blocks of at most 256 elements), stored where the layout wants them.
// scale: 2^b, code_unit: 2^-b.  at: byte offset of the codes inside a slice matrix, slot the same for FP6 (with G = 4 the even lane of a
// pair has the octet).  Called by all lanes of a k-group, whether they store or not.
template <int FMT, int G>
__device__ __forceinline__ void store_slice_codes(const int (&q)[G], bool stores, int b, float scale, float code_unit, uint8_t* dst_slice, size_t at,
                                                  const Fp6Slot& slot) {
    if constexpr (fmt_is_fp6(FMT)) {
        constexpr int K = FMT == FMT_FP6_E3M2 ? 3 : 4;
        uint32_t c[G];
#pragma unroll
        for (int e = 0; e < G; ++e) {
            // The magnitude in eighths is at most 16 (8); as unsigned numbers the smaller of v and 32 - v is v, or 32 (the sign) + |v|.
            // For E2M3 that is the code (magnitudes 0 .. 7 are subnormal, 8 .. 16 follow without a gap); for E3M2 (0, 2, 4, 6, 8, 9, .. 12)
            // magnitudes up to 4 count twice, others are 4 more.
            const int v = q[e] << (K - b);
            c[e] = digit_min((uint32_t)v, 32u - (uint32_t)v);
            if constexpr (FMT == FMT_FP6_E3M2) c[e] += digit_min(c[e] & 31u, 4u);
        }
        // the octet's 48 bits; with G = 4 in the even lane of a pair
        uint32_t lo32, hi16;
        if constexpr (G == 8) {
            lo32 = c[0] | (c[1] << 6) | (c[2] << 12) | (c[3] << 18) | (c[4] << 24) | (c[5] << 30);
            hi16 = (c[5] >> 2) | (c[6] << 4) | (c[7] << 10);
        } else {
            const uint32_t w = c[0] | (c[1] << 6) | (c[2] << 12) | (c[3] << 18);
            const uint32_t next = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0xB1, 0xF, 0xF, true);      // the other lane of the pair
            lo32 = w | (next << 24);
            hi16 = next >> 8;
        }
        // the neighbouring octets' share of the eight bytes (row shifts to the left and right, by one octet)
        const uint32_t next_lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)lo32, G == 8 ? 0x101 : 0x102, 0xF, 0xF, true);
        const uint32_t prev_hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)hi16, G == 8 ? 0x111 : 0x112, 0xF, 0xF, true);
        uint2 w;                                                     // octet 0: lo32 | hi16, next_lo; 1: the upper 32 bits | next_lo; 3: prev_hi, lo32 | hi16
        w.x = __builtin_amdgcn_perm(slot.last ? prev_hi : hi16, lo32, slot.low);
        w.y = __builtin_amdgcn_perm(hi16, slot.last ? lo32 : next_lo, slot.high);
        if (stores && slot.stores) *reinterpret_cast<uint2*>(dst_slice + slot.at) = w;
    } else if constexpr (FMT == FMT_FP16) {
        uint32_t w[G / 2];
#pragma unroll
        for (int h = 0; h < G / 2; ++h)
            w[h] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz((float)q[2 * h] * code_unit, (float)q[2 * h + 1] * code_unit));
        if (stores) {
#pragma unroll
            for (int h = 0; h < G / 8; ++h) *reinterpret_cast<uint4*>(dst_slice + at + 16 * h) = uint4{w[4 * h], w[4 * h + 1], w[4 * h + 2], w[4 * h + 3]};
        }
    } else {
        uint32_t w[G / 4];
#pragma unroll
        for (int h = 0; h < G / 4; ++h) {
            const int* const v = q + 4 * h;
            if constexpr (FMT == FMT_FP8) {
                typedef short short2v __attribute__((ext_vector_type(2)));
                short2v r = {0, 0};
                r = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(r, (float)v[0], (float)v[1], scale, false);
                r = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(r, (float)v[2], (float)v[3], scale, true);
                w[h] = __builtin_bit_cast(uint32_t, r);
            } else {                                                 // the lowest byte of each
                w[h] = __builtin_amdgcn_perm((uint32_t)v[1], (uint32_t)v[0], 0x0C0C0400u) | __builtin_amdgcn_perm((uint32_t)v[3], (uint32_t)v[2], 0x04000C0Cu);
            }
        }
        if (stores) {
            if constexpr (G == 8) *reinterpret_cast<uint2*>(dst_slice + at) = uint2{w[0], w[1]};
            else *reinterpret_cast<uint32_t*>(dst_slice + at) = w[0];
        }
    }
}

// Blocks of up to 16384 elements (slice_digits.hpp): the largest element gives the first exponent, one OR over the vector those of the
// following slices, and the slices are read off each element's 96-bit number without any further exchange.  Where they reach below
// the number, the next exponent is found from the remainders, which are formed anew from the inputs, and another number starts there.
// What bounds it: memory, mostly.  About 65 integer instructions per element and 5 per element and slice, 3 more for each move of the
// numbers (every D = 31 / (b + 1) regular slices, or where a unit lies further down), against 22 per element and slice and a maximum
// over the vector for each slice when the remainders were carried from slice to slice.  4096 vectors of 4096, 13 FP8 slices, us, with
// the differences of the exponents: dense vectors 133 carrying remainders, 85 now; one non-zero element per vector 150 and 92 (388 when
// each irregular unit took another reading of the vector, another maximum and another number); 2 non-zeros 148, 88 (316), bands of 5
// 152, 84 (183).
// U groups of G consecutive elements per thread.  Several waves per vector: the workgroup is one vector and has only the waves that
// hold elements; one wave: four vectors per workgroup, no barrier.
template <int U, int TPR, int G, int FMT>
__device__ __forceinline__ void slice_vectors(const SplitArgs& a) {
    constexpr bool FP16 = FMT == FMT_FP16;
    constexpr int EPC = FP16 ? CHUNK_BYTES / 2 : CHUNK_BYTES;
    constexpr int ROWB = fmt_is_fp6(FMT) ? CHUNK_BYTES_FP6 : CHUNK_BYTES;
    constexpr bool WHOLE = TPR > 64;
    constexpr int RPB = WHOLE ? 1 : 4, WAVES = TPR / 64;
    __shared__ uint32_t red_key[2][WAVES], red_turns[3][WAVES];
    __shared__ int l1_share[FP16 && WHOLE ? MAX_SLICES : 1][WAVES];

    const int tr = WHOLE ? threadIdx.x : threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int threads = WHOLE ? blockDim.x : 64;
    // Workgroups are handed to the eight XCDs (each with an L2 of its own) round-robin by their index.  Neighbouring
    // vectors share the cache lines of the slice layout (a line holds the 16-byte pieces of eight vectors in the
    // FP6 planes, the 64-byte chunks of two vectors otherwise), so eight consecutive workgroups' worth of vectors go to the
    // SAME XCD, where the partial lines meet in one L2 before they are written back; the next eight go to the next XCD, so that
    // also an operand of few vectors is spread over all of them.  Each operand's share of the grid is a multiple of 64.
    const bool second = blockIdx.x >= a.wg_first;
    const SplitVectors& v = second ? a.v[1] : a.v[0];
    const unsigned li = blockIdx.x - (second ? a.wg_first : 0u);
    const int64_t row = (int64_t)((li & ~63u) + (li & 7) * 8 + ((li >> 3) & 7)) * RPB + (WHOLE ? 0 : wave);
    const int64_t t = blockIdx.y, k0 = t * a.kb, padded = a.chunks * EPC;
    int64_t klen = a.k - k0;
    if (klen > a.kb) klen = a.kb;
    if (row >= v.rows) klen = 0;                                     // a padding vector: zero codes, c = 0
    const DigitLadder l = a.ladder;
    const float scale = ldexpf(1.0f, a.b), code_unit = ldexpf(1.0f, -a.b);
    const size_t slice_bytes = (size_t)a.chunks * v.rows_pad * ROWB;
    uint8_t* dst_slice = v.slices + (size_t)(t * a.s) * slice_bytes;
    const double* const src = v.X + row * v.ldv + k0 * v.es;
    struct Group {
        uint64_t bits[G];
        uint32_t x[3][G];                                            // the numbers, word by word
    };
    Group first_group, second_group;                                 // (two variables: an array of them does not stay in single registers)
    auto each_group = [&](auto f) {
        f(0, first_group);
        if constexpr (U > 1) f(1, second_group);
    };
    static_assert(U <= 2, "groups per thread");
    auto first_of = [&](int u) -> int64_t { return G * ((int64_t)tr + (int64_t)threads * u); };
    // does this wave hold elements of the block in group u?  (wave-uniform)
    auto wave_has = [&](int u) -> bool { return u == 0 || G * ((int64_t)__builtin_amdgcn_readfirstlane(tr & ~63) + (int64_t)threads * u) < padded; };
    auto load_group = [&](int u, uint64_t (&bits)[G]) {
        int64_t ke = first_of(u);
        asm volatile("" : "+v"(ke));                                 // (a second reading works its addresses out again: they would spill)
        if (v.es == 1 && ke + G <= klen) {
#pragma unroll
            for (int h = 0; h < G / 2; ++h) {
                const two_doubles w = *reinterpret_cast<const two_doubles*>(src + ke + 2 * h);
                bits[2 * h] = w.x;
                bits[2 * h + 1] = w.y;
            }
        } else {
            const double* at_e = src + ke * v.es;
            const int rest = (int)(klen - ke < G ? klen - ke : G);
#pragma unroll
            for (int e = 0; e < G; ++e) {
                bits[e] = e < rest ? (uint64_t)__double_as_longlong(*at_e) : 0ull;
                at_e += v.es;
                asm volatile("" : "+v"(at_e));                       // one address at a time
            }
        }
    };
    auto vector_max = [&](uint32_t key, int slot) -> uint32_t {
        key = wave_max(key);
        if constexpr (WHOLE) {
            if ((tr & 63) == 0) red_key[slot][wave] = key;
            __syncthreads();
            for (int w = 0; w < threads / 64; ++w) key = red_key[slot][w] > key ? red_key[slot][w] : key;
        }
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)key);
    };
    // where the codes of the first group go inside a slice matrix; the second one's lie a whole number of chunks further on
    const size_t at_codes = ((size_t)(first_of(0) / EPC) * v.rows_pad + row) * CHUNK_BYTES + (size_t)(first_of(0) % EPC) * (FP16 ? 2 : 1);
    const Fp6Slot slot = fp6_slot(first_of(0) & ~(int64_t)7, v.rows_pad, row);
    const size_t second_at = (size_t)(G * threads / EPC) * v.rows_pad * ROWB;
    static_assert(U == 1 || G * 64 % EPC == 0, "a wave's group is a whole number of chunks");

    uint32_t key = 0;
    each_group([&](int u, Group& g) {
        load_group(u, g.bits);
#pragma unroll
        for (int e = 0; e < G; ++e) {
            const uint32_t k = magnitude_key(g.bits[e]);
            key = k > key ? k : key;
        }
    });
    if (key >= 0x7FF00000u) atomicOr(a.flags, 1);                    // infinity or NaN
    key = vector_max(key, 0);
    bool left = key != 0;                                            // is there a remainder?
    int c = 0;
    if (left && key >= 0x100000u) {
        c = magnitude_exponent(key);
    } else if (left) {                                               // subnormal numbers only
        uint32_t sub = 0;
        each_group([&](int, Group& g) {
#pragma unroll
            for (int e = 0; e < G; ++e) {
                uint64_t bit = g.bits[e];
                asm volatile("" : "+v"(bit));
                const uint32_t k = exponent_key(bit & 0x000FFFFFFFFFFFFFull, -1074);
                sub = k > sub ? k : sub;
            }
        });
        c = (int)vector_max(sub, 1) - CD_BIAS;
    }

    auto clear = [&](Group& g) {
#pragma unroll
        for (int e = 0; e < G; ++e) g.x[0][e] = g.x[1][e] = g.x[2][e] = 0;
    };
    int my_exp = 0;                                                  // lane p of the first wave: c of slice p
    int filled = left ? a.s : 0;                                     // slices before there is nothing left
    for (int p = 0; p < a.s;) {
        uint32_t turns[3] = {0, 0, 0};
        if (left) {
            auto form = [&](auto beyond) {
                each_group([&](int u, Group& g) {
                    if (!wave_has(u)) {
                        clear(g);
                        return;
                    }
#pragma unroll
                    for (int e = 0; e < G; ++e) {
                        uint32_t x[3];
                        uint64_t bit = g.bits[e];
                        asm volatile("" : "+v"(bit));                // keeps what the two forms share from being worked out for all elements at once
                        digit_number<decltype(beyond)::value>(bit, c, x, turns);
#pragma unroll
                        for (int i = 0; i < 3; ++i) g.x[i][e] = x[i];
                        // two elements at a time (sixteen per thread: one): with all of them in flight the compiler runs out of registers
                        if (U == 2 || (e & 1)) __builtin_amdgcn_sched_barrier(0);
                    }
                });
            };
            if (p > 0 || c < -1021) form(std::true_type{});
            else form(std::false_type{});
#pragma unroll
            for (int i = 0; i < 3; ++i) turns[i] = wave_or(turns[i]);
            if constexpr (WHOLE) {
                if ((tr & 63) == 0) {
#pragma unroll
                    for (int i = 0; i < 3; ++i) red_turns[i][wave] = turns[i];
                }
                __syncthreads();
                for (int w = 0; w < threads / 64; ++w) {
#pragma unroll
                    for (int i = 0; i < 3; ++i) turns[i] |= red_turns[i][w];
                }
#pragma unroll
                for (int i = 0; i < 3; ++i) turns[i] = (uint32_t)__builtin_amdgcn_readfirstlane((int)turns[i]);
            }
        } else {                                                     // nothing left: zero codes, c := 0
            each_group([&](int, Group& g) { clear(g); });
            c = 0;
        }
        // the slices that can be read off these numbers, in runs of regular ones
        auto move_up = [&](int places) {
            for (; places > 0; places -= 31) {
                const int up = places < 31 ? places : 31;
                each_group([&](int, Group& g) {
#pragma unroll
                    for (int e = 0; e < G; ++e) digit_shift(g.x[2][e], g.x[1][e], g.x[0][e], up);
                });
            }
        };
        int at = 0, last = 0;                                        // places below 2^c of the run's first slice, of its last
        bool more = true;                                            // is there a remainder after the last one?
        while (true) {
            int run = left ? digit_run(turns, at, l) : a.s - p;
            run = run < a.s - p ? run : a.s - p;
            last = at + (run - 1) * l.step;
            int moved = 0;                                           // places, within the run
            if (v.slices != nullptr) {
                if (tr >= p && tr < p + run) my_exp = left ? c - at - (tr - p) * l.step : 0;
                for (int done = 0;;) {
                    const int fields = run - done < l.fields ? run - done : l.fields;
                    for (int d = 0; d < fields; ++d, dst_slice += slice_bytes) {
                        int l1 = 0;
                        each_group([&](int u, Group& g) {
                            if (!wave_has(u)) return;
                            int q[G];
#pragma unroll
                            for (int e = 0; e < G; ++e) {
                                q[e] = digit_of(g.x[2][e], d, l.step);
                                if constexpr (FP16) l1 += q[e] < 0 ? -q[e] : q[e];
                            }
                            const bool stores = first_of(u) < padded && (G == 8 || !fmt_is_fp6(FMT) || (tr & 1) == 0);
                            store_slice_codes<FMT, G>(q, stores, a.b, scale, code_unit, dst_slice + u * second_at, at_codes, slot);
                        });
                        if constexpr (FP16) {
                            if (v.l1 != nullptr) {                   // sum |q| of the slice
                                const int at_slice = p + done + d;
                                l1 = wave_sum(l1);
                                if constexpr (WHOLE) {
                                    if ((tr & 63) == 0) l1_share[at_slice][wave] = l1;
                                } else {
                                    if (tr == 0) v.l1[(t * a.s + at_slice) * v.rows_pad + row] = l1;
                                }
                            }
                        }
                    }
                    done += fields;
                    if (done == run) break;
                    move_up(l.fields * l.step);
                    moved += l.fields * l.step;
                }
            }
            p += run;
            if (p == a.s) break;
            const int next = digit_next(turns, run, l.step);
            more = next != NUMBER_BITS;
            if (!digit_in_number(at + next, l.step)) break;
            at += next;
            move_up(next - moved);
            for (int rest = next; rest > 0; rest -= 31) digit_shift(turns[2], turns[1], turns[0], rest < 31 ? rest : 31);
        }
        // count-only mode (slicing until the remainder is zero, paragraph before Eq. 4): something was left before the last of these slices
        if (v.slices == nullptr) {
            if (left && tr == 0) atomicMax(a.flags + 1, p);
        }
        if (p < a.s) {                                               // beyond the numbers, or nothing left
            uint32_t key = 0;
            if (more) {
                const int unit = c - last - a.b;
                each_group([&](int u, Group& g) {
                    load_group(u, g.bits);
#pragma unroll
                    for (int e = 0; e < G; ++e) {
                        uint64_t bit = g.bits[e];
                        asm volatile("" : "+v"(bit));
                        const uint32_t k = remainder_key(bit, unit);
                        key = k > key ? k : key;
                        if (e & 1) __builtin_amdgcn_sched_barrier(0);
                    }
                });
                key = vector_max(key, 1);
            }
            left = key != 0;
            if (!left && filled > p) filled = p;
            c = (int)key - CD_BIAS;
        }
    }
    if (!FP16 && v.off_ladder != nullptr && tr < 64) {               // (the wave that has the exponents)
        const int before = __shfl_up(my_exp, 1, 64);
        const uint64_t gaps = __ballot(tr > 0 && tr < filled && before - my_exp != l.step);
        if (tr == 0) v.off_ladder[t * v.rows_pad + row] = gaps != 0 ? 1 : 0;
    }
    if (v.slices != nullptr && tr < a.s) v.exps[(t * a.s + tr) * v.rows_pad + row] = my_exp;
    if constexpr (FP16 && WHOLE) {
        if (v.l1 != nullptr) {
            __syncthreads();
            if (tr < a.s) {
                int sum = 0;
                for (int w = 0; w < threads / 64; ++w) sum += l1_share[tr][w];
                v.l1[(t * a.s + tr) * v.rows_pad + row] = sum;
            }
        }
    }
}

// Waves per SIMD.  The registers would let six or seven share one, but the lines of the slice layout are put together in the L2s from
// several vectors, and more vectors in flight push them out half written.  4096 vectors, us: 13 FP6 slices of 4096 112 with five, 122
// with four, 143 with six; 8 FP16 slices in blocks of 2048 355 with four, 376 with five, 388 with six; 13 FP8 slices of 4096 82 with
// six, 88 with five; 6000 vectors of 4097 170 and 202 (five leave one workgroup of up to 1024 threads per CU).
constexpr int most_waves(int U, int TPR, int fmt) { return U == 2 || fmt == FMT_FP16 ? 4 : fmt_is_fp6(fmt) && TPR < 1024 ? 5 : 6; }
template <int U, int TPR, int FMT>
__global__ void __launch_bounds__((TPR < 128 ? 256 : TPR)) __attribute__((amdgpu_waves_per_eu(4, most_waves(U, TPR, FMT)))) split_kernel(SplitArgs a) {
    clear_off_ladder(a);
    slice_vectors<U, TPR, 8, FMT>(a);
}
// Blocks of at most 256 elements: four elements per lane (with eight, half the lanes are idle and a thread's chain is twice as long)
template <int FMT>
__global__ void __launch_bounds__(256) slice_short_kernel(SplitArgs a) {
    slice_vectors<1, 64, 4, FMT>(a);
}

// ---- Blocks too long for the registers of one workgroup --------------------------------------------------------
// x^(p) differs from x by a multiple of the previous unit, which is an even multiple of this one (every remainder is at most half a
// unit, so the units 2^u_p shrink by b+1 bits or more), hence  x^(p+1) = x - (x rounded to a multiple of 2^u_p, ties to even)
// directly from x.  So the exponents come first, from the elements alone (long_exponents_kernel), and with them known every element
// is sliced on its own (split_stream_kernel), with no exchange between threads and no state in memory.  256 + 320 vectors of 65536
// elements, 11 FP8 slices: exponents 212 us when every slice's key was formed from the whole block, 71 us now (302 MB read once at
// 4.7 TB/s: 64 us); slices 247 us carrying remainders, 228 us now (855 MB with the padding vectors: 182 us).

// Eq. 4 for all slices of one vector and block: the largest element in one reading, then the exponents of all slices from the turns of
// the elements' bits (slice_digits.hpp).  Those of part of the block are enough where they give regular units throughout, as a rule
// after the first 8192 elements.  1024 vectors of 65536, 11 FP8 slices, us with the slices themselves: dense 450 (752 when the exponents
// were found slice by slice); one non-zero element 617 (4134, and 2238 with two readings for each irregular unit).
__global__ void __launch_bounds__(1024) long_exponents_kernel(SplitArgs a) {
    __shared__ uint32_t red_key[16], red_turns[2][3][16];
    clear_off_ladder(a);
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
        if (v.off_ladder != nullptr && tid == 0) v.off_ladder[t * v.rows_pad + row] = 0;
        return;
    }
    const double* const src = v.X + row * v.ldv + t * a.kb;
    const DigitLadder l = a.ladder;
    // f(bits) for the elements i .. i + 8191, four 16-byte loads in flight per thread
    auto for_chunk = [&](int64_t i, auto f) {
        if (i + 8192 <= klen) {
            two_doubles w[4];
#pragma unroll
            for (int h = 0; h < 4; ++h) w[h] = *reinterpret_cast<const two_doubles*>(src + i + h * 2048 + 2 * tid);
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                f(w[h].x);
                f(w[h].y);
            }
        } else {
            for (i += tid; i < klen; i += 1024) f((uint64_t)__double_as_longlong(src[i]));
        }
    };
    auto block_max = [&](uint32_t key) -> uint32_t {
        __syncthreads();                                             // the previous maximum has been read
        key = wave_max(key);
        if ((tid & 63) == 0) red_key[wave] = key;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < 16; ++w) key = red_key[w] > key ? red_key[w] : key;
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)key);
    };
    auto largest_remainder = [&](int unit) -> uint32_t {
        uint32_t key = 0;
        for (int64_t i = 0; i < klen; i += 8192)
            for_chunk(i, [&](uint64_t w) {
                const uint32_t k = remainder_key(w, unit);
                key = k > key ? k : key;
            });
        return block_max(key);
    };

    uint32_t top = 0;
    for (int64_t i = 0; i < klen; i += 8192)
        for_chunk(i, [&](uint64_t w) {
            const uint32_t k = magnitude_key(w);
            top = k > top ? k : top;
        });
    if (top >= 0x7FF00000u) atomicOr(a.flags, 1);                    // infinity or NaN
    top = block_max(top);
    bool left = top != 0;                                            // is there a remainder before slice p?
    int c = 0, p = 0;
    if (left) c = top >= 0x100000u ? magnitude_exponent(top) : (int)largest_remainder(2000) - CD_BIAS;      // 2^2000: x itself
    while (left && p < a.s) {
        uint32_t turns[3] = {0, 0, 0}, all[3];
        int levels, at, last, my_exp = 0;                            // slices off these numbers, places of the last run's first and last
        bool more = true;                                            // is there a remainder after them?
        for (int64_t i = 0, turn = 0;; turn ^= 1) {
            for_chunk(i, [&](uint64_t w) {
                uint32_t x[3];
                digit_number<true>(w, c, x, turns);
            });
            i += 8192;
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const uint32_t m = wave_or(turns[j]);
                if ((tid & 63) == 0) red_turns[turn][j][wave] = m;
            }
            __syncthreads();                                         // (the other buffer's readers are behind the previous one)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                all[j] = 0;
#pragma unroll
                for (int w = 0; w < 16; ++w) all[j] |= red_turns[turn][j][w];
                all[j] = (uint32_t)__builtin_amdgcn_readfirstlane((int)all[j]);
            }
            // more elements can only bring the units closer, to `step` places at the least
            bool regular = true;
            for (at = 0, levels = 0;;) {
                int run = digit_run(all, at, l);
                run = run < a.s - p - levels ? run : a.s - p - levels;
                if (tid >= levels && tid < levels + run) my_exp = c - at - (tid - levels) * l.step;
                levels += run;
                last = at + (run - 1) * l.step;
                if (p + levels == a.s) break;
                const int next = digit_next(all, run, l.step);
                regular = regular && next == run * l.step;
                more = next != NUMBER_BITS;
                if (!digit_in_number(at + next, l.step)) break;
                at += next;
                for (int rest = next; rest > 0; rest -= 31) digit_shift(all[2], all[1], all[0], rest < 31 ? rest : 31);
            }
            if (i >= klen || regular) break;
        }
        if (exps != nullptr && tid < levels) exps[(int64_t)(p + tid) * v.rows_pad] = my_exp;
        p += levels;
        if (p >= a.s) break;
        const uint32_t key = more ? largest_remainder(c - last - a.b) : 0u;
        left = key != 0;
        c = (int)key - CD_BIAS;
    }
    if (v.off_ladder != nullptr) {                                   // off the exponents of the slices that are there (noted on the way it took 3 us of 65)
        __syncthreads();
        const bool gap = tid > 0 && tid < p && exps[(int64_t)(tid - 1) * v.rows_pad] - exps[(int64_t)tid * v.rows_pad] != l.step;
        const uint64_t gaps = __ballot(gap);                         // (of the first wave: 32 slices at most)
        if (tid == 0) v.off_ladder[t * v.rows_pad + row] = gaps != 0 ? 1 : 0;
    }
    // nothing left: the remaining slices are zero (c := 0); without slices to write, report how many there are
    if (exps != nullptr)
        for (int i = p + tid; i < a.s; i += 1024) exps[(int64_t)i * v.rows_pad] = 0;
    if (v.slices == nullptr && tid == 0 && p > 0) atomicMax(a.flags + 1, p);
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
    const Fp6Slot slot = fp6_slot(ke, v.rows_pad, row);
    // Where the units of all slices follow one ladder (the usual case), the slices are read off one number per element.
    {
        const DigitLadder l = a.ladder;
        const int c0 = exps[0];
        bool on_ladder = digit_in_number((a.s - 1) * l.step, l.step) && c0 >= -1021;
        for (int p = 1; p < a.s; ++p) on_ladder = on_ladder && exps[(int64_t)p * v.rows_pad] == c0 - p * l.step;
        if (__all(on_ladder || row >= v.rows)) {
            uint32_t x[3][8], turns[3];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                uint32_t y[3];
                digit_number<false>(bits[e], c0, y, turns);
#pragma unroll
                for (int i = 0; i < 3; ++i) x[i][e] = y[i];
                if (e & 1) __builtin_amdgcn_sched_barrier(0);
            }
            const float scale = ldexpf(1.0f, a.b), unit_value = ldexpf(1.0f, -a.b);
            const size_t at = ((size_t)kc * v.rows_pad + row) * CHUNK_BYTES + (size_t)(threadIdx.x % OCTETS) * (FP16 ? 16 : 8);
            for (int p = 0; p < a.s; p += l.fields) {
                if (p > 0) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) digit_shift(x[2][e], x[1][e], x[0][e], l.fields * l.step);
                }
                for (int d = 0; d < l.fields && p + d < a.s; ++d, dst_slice += slice_bytes) {
                    int q[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) q[e] = digit_of(x[2][e], d, l.step);
                    store_slice_codes<FMT, 8>(q, true, a.b, scale, unit_value, dst_slice, at, slot);
                }
            }
            return;
        }
    }
    // Blocks this long leave FP16 slices 4 bits at most, so the 32-bit element step serves every format.
    const int pos = F - 32, bias = (1 << (pos - 1)) - 1;
    const uint32_t keep = ~((1u << pos) - 1u);
    const float code_scale = ldexpf(1.0f, pos + a.b), code_unit = ldexpf(1.0f, -(pos + a.b));
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
            int q[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) q[e] = qs[e] >> pos;
            store_slice_codes<FMT, 8>(q, true, a.b, 0.0f, 0.0f, dst_slice, 0, slot);
        }
    };
    uint64_t T[8];
    int wait[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) decode_narrow(bits[e], F, T[e], wait[e]);
    int unit_prev = 0, p = 0;
    // while some element of the wave waits for its unit, then one shift for all
    for (bool settled = false; p < a.s && !settled; ++p, dst_slice += slice_bytes) {
        const int unit = exps[(int64_t)p * v.rows_pad] - a.b;
        const int step = unit_prev - unit;
        unit_prev = unit;
        int qs[8], longest = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            qs[e] = slice_narrow(T[e], wait[e], step, pos, bias, keep);
            longest = wait[e] < longest ? wait[e] : longest;
        }
        store(qs);
        settled = __ballot(longest < 0) == 0ull;
    }
    for (; p < a.s; ++p, dst_slice += slice_bytes) {
        const int unit = exps[(int64_t)p * v.rows_pad] - a.b, step = unit_prev - unit;
        unit_prev = unit;
        int qs[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) qs[e] = slice_narrow_active(T[e], step, pos, bias, keep);
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

// One workgroup per 256 vectors and block: the deltas, which vectors are off the ladder, the bounds.
__global__ void __launch_bounds__(256) delta_kernel(DeltaArgs a, OffLadder off_ladder) {
    const bool second = blockIdx.x >= a.tiles_first;
    const DeltaOperand& o = a.o[second ? 1 : 0];
    const int64_t tile = blockIdx.x - (second ? a.tiles_first : 0u), groups = o.rows_pad / LINK_ROWS, t = blockIdx.y;
    const int64_t row = tile * TILE + threadIdx.x;
    const int lane = threadIdx.x & 63;
    const bool off = off_ladder.counts != nullptr && o.off_ladder[(size_t)t * o.rows_pad + row] != 0;
    for (int p = 0; p < a.s; ++p) fill_delta(a, blockIdx.x, t, p);
    if (off_ladder.counts != nullptr) {
        const uint64_t bits = __ballot(off);
        if (bits != 0) {                                             // (they are few, or their list is of no use)
            int place = 0;
            if (lane == 0) place = atomicAdd(off_ladder.counts + (second ? 1 : 0), __popcll(bits));
            place = __shfl(place, 0, 64) + __popcll(bits & ((1ull << lane) - 1ull));
            if (off && place < off_ladder.limit) off_ladder.list[(second ? off_ladder.limit : 0) + place] = (int)row;
        }
    }
    if (o.l1 == nullptr) return;
    // Operand::bounds: 2^b times the largest sum |q| of the group
    int32_t* const bounds = o.bounds + (size_t)t * a.s * groups + row / LINK_ROWS;
    for (int p = 0; p < a.s; ++p) {
        int most = o.l1[(size_t)(t * a.s + p) * o.rows_pad + row];
#pragma unroll
        for (int off = 1; off < 32; off <<= 1) {
            const int other = __shfl_xor(most, off, 64);
            most = other > most ? other : most;
        }
        if ((lane & 31) == 0) bounds[(size_t)p * groups] = most << a.b;
    }
}

template <int U, int TPR>
hipError_t launch_split_cfg(const SplitArgs& a_in, int fmt, int64_t T, hipStream_t st) {
    constexpr int RPB = TPR == 64 ? 4 : 1;
    SplitArgs a = a_in;
    a.wg_first = (unsigned)(a.v[0].rows_pad / RPB);                     // rows_pad is a multiple of 256
    dim3 grid(a.wg_first + (unsigned)(a.v[1].rows_pad / RPB), (unsigned)T);
    const int64_t octets = a.chunks * (fmt == FMT_FP16 ? CHUNK_BYTES / 2 : CHUNK_BYTES) / 8;
    const dim3 block(RPB == 4 ? 256u : (unsigned)((octets + 64 * U - 1) / (64 * U)) * 64u);
    if (fmt == FMT_FP16) hipLaunchKernelGGL((split_kernel<U, TPR, FMT_FP16>), grid, block, 0, st, a);
    else if (fmt == FMT_FP6) hipLaunchKernelGGL((split_kernel<U, TPR, FMT_FP6>), grid, block, 0, st, a);
    else if (fmt == FMT_FP6_E3M2) hipLaunchKernelGGL((split_kernel<U, TPR, FMT_FP6_E3M2>), grid, block, 0, st, a);
    else if (fmt == FMT_INT8) hipLaunchKernelGGL((split_kernel<U, TPR, FMT_INT8>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((split_kernel<U, TPR, FMT_FP8>), grid, block, 0, st, a);
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
    v.X = X; v.ldv = ldv; v.es = es; v.rows = op->rows; v.rows_pad = op->rows_pad; v.slices = op->slices; v.exps = op->exps; v.l1 = op->l1; v.off_ladder = op->off_ladder;
    return v;
}
}  // namespace

hipError_t launch_split(const double* X0, int64_t ldv0, int64_t es0, const Operand* op0, const double* X1, int64_t ldv1, const Operand* op1,
                        const Plan& pl, int* flags, hipStream_t st) {
    SplitArgs a;
    a.v[0] = split_vectors(X0, ldv0, es0, op0);
    a.v[1] = split_vectors(X1, ldv1, 1, op1);
    a.wg_first = 0;
    a.k = pl.k; a.kb = pl.kb; a.chunks = pl.chunks; a.s = pl.s; a.b = pl.b; a.ladder = digit_ladder(pl.b); a.flags = flags;
    if (a.v[0].rows_pad + a.v[1].rows_pad == 0 || pl.T == 0) return hipSuccess;
    const int fmt = pl.fmt;
    if (pl.kb > MAX_K_BLOCK_IN_REGISTERS && es0 != 1) return hipErrorInvalidValue;
    if (pl.kb > MAX_K_BLOCK_IN_REGISTERS) return launch_split_long(a, fmt, pl.T, st);
    const int64_t octets = pl.chunks * pl.epc / 8;                              // per vector and block, padded
    // Eight elements per thread while a workgroup has threads for them, sixteen beyond: with two exchanges per vector the waves are
    // not held up by each other, and 65 to 80 registers let six of them share a SIMD (sixteen elements need 128: four).  FP16 in short
    // blocks keeps eight per lane, whose codes are one 16-byte store.
    if (octets <= 32 && fmt != FMT_FP16) return launch_split_short(a, fmt, pl.T, st);
    if (octets <= 64) return launch_split_cfg<1, 64>(a, fmt, pl.T, st);
    if (octets <= 128) return launch_split_cfg<1, 128>(a, fmt, pl.T, st);
    if (octets <= 256) return launch_split_cfg<1, 256>(a, fmt, pl.T, st);
    if (octets <= 512) return launch_split_cfg<1, 512>(a, fmt, pl.T, st);
    if (octets <= 768) return launch_split_cfg<1, 1024>(a, fmt, pl.T, st);
    if (octets <= 1024) return launch_split_cfg<2, 512>(a, fmt, pl.T, st);
    if (octets <= 1536) return launch_split_cfg<2, 768>(a, fmt, pl.T, st);
    if (octets <= 2048) return launch_split_cfg<2, 1024>(a, fmt, pl.T, st);
    // 32 elements per thread would cover blocks of up to 32768 elements, but not in the 128 registers a thread of a
    // 1024-thread workgroup has; such blocks are streamed
    return hipErrorInvalidValue;
}

hipError_t launch_count_slices(const double* X, int64_t ldv, const Plan& pl, int64_t rows, int* flags, hipStream_t st) {
    Plan cp = pl;
    cp.s = MAX_SLICES + 1;                       // one more than the library can use: "not exhausted" is reported as 33
    Operand op;
    op.rows = rows;
    op.rows_pad = (rows + TILE - 1) / TILE * TILE;
    op.slices = nullptr; op.exps = nullptr; op.deltas = nullptr; op.l1 = nullptr; op.bounds = nullptr; op.off_ladder = nullptr;
    return launch_split(X, ldv, 1, &op, nullptr, 0, nullptr, cp, flags, st);
}

hipError_t launch_deltas(const Plan& pl, const Operand* op0, const Operand* op1, const OffLadder& off, hipStream_t st) {
    const DeltaArgs a = delta_args(pl, op0, op1);
    if (a.tiles == 0 || pl.T == 0 || pl.s == 0) return hipSuccess;
    hipLaunchKernelGGL(delta_kernel, dim3(a.tiles, (unsigned)pl.T), dim3(256), 0, st, a, off);
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
