// All slice-pair products of a 64 x 64 tile of C and their sum in one kernel (launch_ladder_sums in layout.hpp), for vectors whose
// exponents are a regular ladder: c_p - c_(p+1) = b + 1 for every slice p, which is what a vector with entries enough gives.  All
// pairs of an anti-diagonal then have one scale for the whole tile and are summed in one accumulator, so that a wave keeps the S
// anti-diagonals p + q = g of its 32 x 32 tile in 16 S accumulator registers per lane and the products of all S (S + 1) / 2 pairs
// come from one pass over k.
//
// What bounded the other kernels is the stream of slices from the L2s to the compute units (16 TB/s over all of them, 256 flop per byte
// with a 256 x 256 tile of one pair).  Here 2 x 64 vectors x S slices are fetched per 64-byte stage for S (S + 1) / 2 products of
// 64 x 64 x 64: 448 flop per byte with 13 slices; and a wave reads 2 S fragments from LDS for S (S + 1) / 2 matrix instructions, 26 for
// 91 against 8 for 16.  That leaves the matrix unit as the bound: a stage of 13 slices takes 5960 cycles, its 91 matrix instructions
// 5824; of 11 slices 4400 and 4224; of 9 INT8 slices, 45 products, 3940 and 2880 (there the slices' stream again).  Every lane ends with all anti-diagonals of its sixteen elements
// of C and sums them itself, at scales that are the same for the whole launch: no product is stored or read again.
// One call by the GEMM kernels with the accumulation, and by this one: 4096^3 FP8, 13 slices, hardware sum 4.36 and 3.63 ms; 4096^3 FP6,
// 121 pairs, emulated 4.92 and 4.12 ms; 1000 x 777 x 1301 FP8, 12 slices, scaled, emulated 165 and 109 us; 600 x 600 x 1000 FP8, 11
// slices, emulated, in 64 MiB 108 and 73 us; 96 x 6000 x 4097 INT8, 9 slices 355 and 276 us; 1024^3 FP8, 121 pairs 148 and 104 us.
//
// A wave holds the S fragments of its A slices and walks the B slices from the last to the first: column j is B slice S - 1 - j (0-based) with
// the A slices 0 .. j, j + 1 products.  Every A slice meets B slice 0 in the last column, and its fragment of the next stage is read right
// behind that product.  LDS holds one stage of all slices, each part refilled as soon as all waves have read it; three barriers a
// stage say so (Ladder::A_FREE, MIDDLE and the last column), two of them also that the loads issued half a stage or more before
// have landed.
//
// Vectors of either operand may be off the ladder (few entries that count at some depth, or the end of the mantissas reached); the slicing
// kernels say which.  Where
// they are few, their rows and columns of C are left to off_ladder.hpp; where they are not, the kernel does nothing, and the GEMM
// kernels and the accumulation, which come behind it, do all (OffLadder in layout.hpp).  A vector whose remainder is zero from some slice on is regular as far as it goes: the slices behind add zeros, whatever their scale.
//
// LESSER_HALF: the same for the pairs p + q > s + 1 of the all-pairs set: with p' = s + 1 - p, q' = s + 1 - q they are the triangle
// p' + q' <= s of S = s - 1 slices, summed in the reverse order.
#pragma once
#include <type_traits>
#include <utility>

#include "deltas.hpp"
#include "fp64_emu.hpp"
#include "layout.hpp"

namespace ozaki {

struct LadderArgs {
    OffLadder off;
    DeltaArgs deltas;        // off.uncounted: filled for the kernels behind it where too many vectors are off the ladder
    unsigned deltas_of;      // so many pieces of work, a slice of 256 vectors and a block each
    const uint8_t* sa;       // A slices of the block: [s][chunks][rows_pad_a][row bytes]
    const uint8_t* sb;       // B slices of the block
    const int32_t* ea;       // exponents of the block: [s][rows_pad_a]
    const int32_t* eb;       // [s][rows_pad_b]
    int64_t rows_pad_a, rows_pad_b;
    int chunks, s;
    int blocks_m, blocks_n;  // 64 x 64 tiles of C
    WorkOrder work;
    int64_t m, n;
    int add_to_C;
    uint64_t* S;             // running block sum: [tile][wave][word][1024]
    double* C;
    int64_t ldc;
    const double* W;         // add_to_C: what the block is added to (C itself, or the product so far)
    int64_t ldw;
    int scaled, use_beta;    // the result is fl(fl(alpha * P) + fl(beta * C)), or fl(alpha * P) without reading C
    uint64_t alpha, beta;
};

// A workgroup per tile: one kernel per format, accumulation, slice count S and part.
template <int FMT, int MODE>
hipError_t launch_ladder_kernel(const LadderArgs& a, int S, int part, unsigned blocks, hipStream_t st);

namespace {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef int v16i __attribute__((ext_vector_type(16)));

#define OZAKI_LPTR(p) ((__attribute__((address_space(3))) void*)(p))

template <int I> using idx_t = std::integral_constant<int, I>;
template <int N, typename F, int... I>
__device__ __forceinline__ void static_for_(F&& f, std::integer_sequence<int, I...>) { (f(idx_t<I>{}), ...); }
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) { static_for_<N>(f, std::make_integer_sequence<int, N>{}); }

// At most N vector-memory operations of this wave outstanding, its LDS operations complete, then the barrier; no fence
// (it would wait for every load).
template <int N>
__device__ __forceinline__ void wait_and_barrier() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | 0x0070);   // vmcnt(N) expcnt(7) lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

template <int FMT, int S>
struct Ladder {
    static constexpr bool FP6 = fmt_is_fp6(FMT);
    static constexpr int PIECE = FP6 ? 3072 : 4096;                   // 64 vectors of a slice in one stage
    static constexpr int AHEAD = 3;                                   // columns that B fragments are read ahead
    static constexpr int A_FREE = 2;                                  // column before which the A slices in LDS are done with
    static constexpr int MIDDLE = (S + 1) / 2;                        // column before which the early B slices are
    static constexpr int EARLY = MIDDLE + AHEAD < S ? MIDDLE + AHEAD : S, LATE = S - EARLY;
    static constexpr int loads(int n) { return FP6 ? (3 * n + 3) / 4 : n; }      // per wave, for n slices
    static constexpr int LDS_BYTES = 2 * S * PIECE;
    static constexpr int start(int j) { return j * (j + 1) / 2; }
    static constexpr int PRODUCTS = S * (S + 1) / 2;
};

// The sum of an element in the three accumulations: terms of the integers v at the scales 2^(at * STEP), at = 0, 1, ... S - 1, in that
// order.  (On the ladder b is the format's largest: a window for S pairs at less would hold one at that.)  GO_ON: from the sum of terms below.
template <int FMT>
struct LadderScale {
    static constexpr int BITS = ladder_bits(FMT), STEP = BITS + 1;
    static constexpr int P_FRAC = FMT == FMT_INT8 ? 0 : FMT == FMT_FP6 ? 2 * BITS - 2 : 2 * BITS;      // v = product * 2^P_FRAC
    static constexpr int TERM_BITS = FMT == FMT_INT8 ? 31 : 24;
};
template <int FMT, int MODE, bool GO_ON, int S>
struct LadderSum;
template <int FMT, bool GO_ON, int S>
struct LadderSum<FMT, ACC_HW, GO_ON, S> {
    typedef LadderScale<FMT> Scale;
    double sum;
    __device__ __forceinline__ void zero() { sum = 0.0; }
    __device__ __forceinline__ void load(const uint64_t* at, int down) { sum = ldexp(__longlong_as_double((long long)at[0]), -down); }
    __device__ __forceinline__ void store(uint64_t* at) const { at[0] = (uint64_t)__double_as_longlong(sum); }
    template <int AT, typename T>
    __device__ __forceinline__ void add(T c) { sum = sum + ldexp((double)c, AT * Scale::STEP + Scale::P_FRAC); }
    __device__ __forceinline__ uint64_t result(int base) const { return (uint64_t)__double_as_longlong(ldexp(sum, base)); }
};
template <int FMT, typename T>
__device__ __forceinline__ int ladder_integer(T c) {
    if constexpr (FMT == FMT_INT8) return (int)c;
    else return (int)ldexpf((float)c, LadderScale<FMT>::P_FRAC);
}
// LadderAdd; the first additions of a new sum need no rounding: a term is STEP bits above the one before.
template <int FMT, bool GO_ON, int S>
struct LadderSum<FMT, ACC_EMU, GO_ON, S> {
    typedef LadderScale<FMT> Scale;
    static constexpr int SURE = GO_ON ? 0 : (52 - Scale::TERM_BITS) / Scale::STEP + 1;
    LadderAdd sum;
    __device__ __forceinline__ void zero() { sum = LadderAdd{0, 0}; }
    __device__ __forceinline__ void load(const uint64_t* at, int down) { sum = LadderAdd{(int64_t)at[0], (int)at[1024] - down}; }
    __device__ __forceinline__ void store(uint64_t* at) const {
        at[0] = (uint64_t)sum.x;
        at[1024] = (uint64_t)(int64_t)sum.ex;
    }
    template <int AT, typename T>
    __device__ __forceinline__ void add(T c) {
        const int v = ladder_integer<FMT>(c);
        if constexpr (AT < SURE) sum.x += (int64_t)((uint64_t)(int64_t)v << (AT * Scale::STEP));
        else sum.template add<(GO_ON ? 2 * S : S - 1) * Scale::STEP>(v, AT * Scale::STEP);
    }
    __device__ __forceinline__ uint64_t result(int base) const { return sum.value(base); }
};
// Exact: an integer of 128 bits in units of the first term's scale (ladder_exact_fits), rounded once as Fixed192 does.
template <int FMT, bool GO_ON, int S>
struct LadderSum<FMT, ACC_EXACT, GO_ON, S> {
    typedef LadderScale<FMT> Scale;
    unsigned __int128 sum;
    int above;                                                        // the unit of `sum` is 2^-above
    __device__ __forceinline__ void zero() { sum = 0, above = 0; }
    __device__ __forceinline__ void load(const uint64_t* at, int down) {
        sum = (unsigned __int128)at[1024] << 64 | at[0];
        above = down;
    }
    __device__ __forceinline__ void store(uint64_t* at) const {
        at[0] = (uint64_t)sum;
        at[1024] = (uint64_t)(sum >> 64);
    }
    template <int AT, typename T>
    __device__ __forceinline__ void add(T c) {
        const unsigned __int128 v = (unsigned __int128)(__int128)ladder_integer<FMT>(c);
        if constexpr (GO_ON) sum += v << (above + AT * Scale::STEP);
        else sum += v << (AT * Scale::STEP);
    }
    __device__ __forceinline__ uint64_t result(int base) const {
        const uint64_t hi = (uint64_t)(sum >> 64);
        return Fixed192{(uint64_t)sum, hi, (uint64_t)((int64_t)hi >> 63)}.round_to_fp64(base - above);
    }
};

// The sums of a launch: of a triangle of pairs, or of all pairs in two launches, the less significant triangle first.
constexpr int WHOLE = 0, LESSER_HALF = 1, GREATER_HALF = 2;

// Workgroups per compute unit: two up to 8 slices, whose registers (128 accumulators of 256) and LDS (66 KB) allow it, one beyond.  One
// of the two multiplies while the other waits at a barrier or sums.  The bound has to say so: left to themselves the sums took 296 registers
// with 6 INT8 slices in the emulated mode, and 8 slices 276 in any, so that one workgroup was left.  4096^3, us, with one and with two: INT8
// emulated, 6 slices 1661 and 1295, 7 of all pairs 3363 and 2698; hardware sum, 8 slices FP8 1895 and 1627, FP6 1580 and 1251, INT8 2071 and 1911.
constexpr int ladder_workgroups(int s) { return s <= 8 ? 2 : 1; }
template <int FMT, int S, int MODE, int PART>
__global__ void __launch_bounds__(256, ladder_workgroups(S)) ladder_sums_kernel(const LadderArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)                                   // buffer descriptors are not a type on the host
    typedef Ladder<FMT, S> L;
    typedef LadderScale<FMT> Scale;
    constexpr bool FLIP = PART == LESSER_HALF, GO_ON = PART == GREATER_HALF, LISTS = PART == WHOLE && !fmt_is_fp6(FMT);      // (OffLadder::limit: place_ladder)
    constexpr bool INT8 = FMT == FMT_INT8, FP6 = fmt_is_fp6(FMT);
    static_assert(L::LDS_BYTES >= 4 * 8192, "the waves' results");
    constexpr int FP6_CODE = FMT == FMT_FP6_E3M2 ? 3 : 2;
    constexpr int BK = FP6 ? CHUNK_BYTES_FP6 : CHUNK_BYTES;
    __shared__ __attribute__((aligned(16))) uint8_t lds[L::LDS_BYTES + 512];     // one array: with several, the compiler waits for all loads into LDS before every read
    int* const leading = reinterpret_cast<int*>(lds + L::LDS_BYTES);  // first-slice exponents of the 64 rows and 64 columns

    const int tid = threadIdx.x, lane = tid & 63;
    if (!GO_ON && a.off.uncounted != nullptr) {                       // (that one comes second)
        const v4i* const marks = reinterpret_cast<const v4i*>(a.off.uncounted);
        const int all = a.off.mark_bytes / 16;
        int found = 0;                                                // vectors of A off the ladder, and 2^16 times those of B; without a list: any?
#pragma unroll 4
        for (int i = lane; i < all; i += 64) {
            const v4i v = marks[i];
            if constexpr (LISTS) {
                const int c = __popc(v[0]) + __popc(v[1]) + __popc(v[2]) + __popc(v[3]);
                found += i < a.off.first_bytes / 16 ? c : c << 16;
            } else {
                found |= v[0] | v[1] | v[2] | v[3];
            }
        }
        if constexpr (LISTS) {
            if (__ballot(found != 0) != 0) {
#pragma unroll
                for (int by = 1; by < 64; by <<= 1) found += __shfl_xor(found, by, 64);
            }
            found = __builtin_amdgcn_readfirstlane(found);
        } else {
            found = __ballot(found != 0) != 0 ? 1 : 0;
        }
        const int rows_off = found & 0xFFFF, cols_off = found >> 16;
        if (blockIdx.x == 0 && tid == 0) {                            // for the launches behind this one
            a.off.counts[0] = rows_off;
            a.off.counts[1] = cols_off;
        }
        if (rows_off > a.off.limit || cols_off > a.off.limit) {
            for (unsigned i = blockIdx.x; i < a.deltas_of; i += gridDim.x) {
                const unsigned tile = i / (unsigned)a.s, p = i - tile * (unsigned)a.s, t = tile / a.deltas.tiles;
                fill_delta(a.deltas, tile - t * a.deltas.tiles, t, (int)p);
            }
            return;
        }
        if (LISTS && found != 0 && blockIdx.x == 0 && tid < 64) {      // the list, for off_ladder.hpp
            int of_a = 0, of_b = a.off.limit;
            for (int first = 0; first < all; first += 64) {
                const v4i v = first + lane < all ? marks[first + lane] : v4i{0, 0, 0, 0};
#pragma unroll
                for (int w = 0; w < 4; ++w)
                    for (uint64_t lanes = __ballot(v[w] != 0); lanes != 0; lanes &= lanes - 1) {
                        const int l = __ffsll((unsigned long long)lanes) - 1, word = __builtin_amdgcn_readlane(v[w], l);
                        for (int byte = 0; byte < 4; ++byte) {
                            if (((word >> (8 * byte)) & 1) == 0) continue;
                            const int vector = (first + l) * 16 + w * 4 + byte;
                            const bool of_first = vector < a.off.first_bytes;
                            if (lane == 0) a.off.list[of_first ? of_a : of_b] = of_first ? vector : vector - a.off.first_bytes;
                            of_a += of_first ? 1 : 0;
                            of_b += of_first ? 0 : 1;
                        }
                    }
            }
        }
    } else if (!on_ladder(a.off)) {
        return;
    }
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave >> 1, wm = wave & 1;
    const WorkItem item = work_item(blockIdx.x, gridDim.x, a.work, a.blocks_m, a.blocks_n);
    const int bm = item.bm, bn = item.bn;
    const int64_t row0 = (int64_t)bm * 64, col0 = (int64_t)bn * 64;

    const unsigned pad_a = (unsigned)a.rows_pad_a, pad_b = (unsigned)a.rows_pad_b;
    const unsigned cs_a = pad_a * BK, cs_b = pad_b * BK, slice_a = cs_a * (unsigned)a.chunks, slice_b = cs_b * (unsigned)a.chunks;
    const auto rsrc_a = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(a.sa), 0, slice_a * (unsigned)a.s, 0x00027000);
    const auto rsrc_b = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(a.sb), 0, slice_b * (unsigned)a.s, 0x00027000);
    const unsigned lrow = lane >> 2;
    const unsigned swizzled = (wave * 16 + lrow) * BK + (((lane & 3) ^ ((lrow >> 2) & 3)) << 4);
    const unsigned voff_a = FP6 ? ((unsigned)row0 + lane) * 16 : (unsigned)row0 * BK + swizzled;
    const unsigned voff_b = FP6 ? ((unsigned)col0 + lane) * 16 : (unsigned)col0 * BK + swizzled;
    const unsigned voff8_a = pad_a * 32 + ((lane >> 5) * pad_a + (unsigned)row0) * 8 + (lane & 31) * 16;
    const unsigned voff8_b = pad_b * 32 + ((lane >> 5) * pad_b + (unsigned)col0) * 8 + (lane & 31) * 16;
    uint8_t* const lds_a = lds;
    uint8_t* const lds_b = lds + S * L::PIECE;
    // Load `l` of this wave of the n slices from index `from` on of an operand; at: the first slice's part for the stage, by: from a slice
    // to the next one
    const unsigned first_a = FLIP ? S * slice_a : 0, first_b = FLIP ? S * slice_b : 0;
    const unsigned by_a = FLIP ? 0u - slice_a : slice_a, by_b = FLIP ? 0u - slice_b : slice_b;
    auto issue = [&](auto of_a, auto from, auto n, auto l, unsigned at, unsigned by) {
        constexpr bool A = decltype(of_a)::value;
        uint8_t* const buf = A ? lds_a : lds_b;
        auto slice_at = [&](int p) -> unsigned { return at + (unsigned)p * by; };
        if constexpr (FP6) {
            int idx = 4 * decltype(l)::value + wave;
            if (idx >= 3 * decltype(n)::value) idx = 3 * decltype(n)::value - 1;
            const int p = decltype(from)::value + idx / 3, part = idx % 3;
            const unsigned vo = part == 2 ? (A ? voff8_a : voff8_b) : (A ? voff_a : voff_b) + (part == 1 ? (A ? pad_a : pad_b) * 16 : 0);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(A ? rsrc_a : rsrc_b, OZAKI_LPTR(buf + p * L::PIECE + part * 1024), 16, vo, slice_at(p), 0, 0);
        } else {
            constexpr int p = decltype(from)::value + decltype(l)::value;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(A ? rsrc_a : rsrc_b, OZAKI_LPTR(buf + p * L::PIECE + wave * 1024), 16, A ? voff_a : voff_b,
                                                     slice_at(p), 0, 0);
        }
    };
    const std::true_type of_a;
    const std::false_type of_b;

    typedef typename std::conditional<INT8, v16i, v16f>::type acc_t;
    acc_t acc[S];
#pragma unroll
    for (int i = 0; i < S; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] = 0;

    struct Frag { typename std::conditional<INT8, v4i[2], v8i>::type v; };
    const int frow = lane & 31, fg = lane >> 5, fsw = (frow >> 2) & 3;
    const unsigned in_a = FP6 ? fg * 1024 + (wm * 32 + frow) * 16 : (wm * 32 + frow) * BK;
    const unsigned in_b = FP6 ? fg * 1024 + (wn * 32 + frow) * 16 : (wn * 32 + frow) * BK;
    const unsigned in8_a = 2048 + fg * 512 + (wm * 32 + frow) * 8, in8_b = 2048 + fg * 512 + (wn * 32 + frow) * 8;
    auto read_frag = [&](auto op_a, int p) -> Frag {
        constexpr bool A = decltype(op_a)::value;
        Frag f;
        const uint8_t* const base = (A ? lds_a : lds_b) + p * L::PIECE;
        const unsigned in = A ? in_a : in_b;
        if constexpr (INT8) {
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) f.v[ks] = *reinterpret_cast<const v4i*>(base + in + (((2 * ks + fg) ^ fsw) << 4));
        } else if constexpr (FP6) {
            const v4i lo = *reinterpret_cast<const v4i*>(base + in);
            unsigned at = (unsigned)(uintptr_t)OZAKI_LPTR(base + (A ? in8_a : in8_b));
            asm volatile("" : "+v"(at));                              // an address register of its own, see pair_gemm_body.hpp
            const v2i hi = *reinterpret_cast<const __attribute__((address_space(3))) v2i*>((uintptr_t)at);
            f.v = __builtin_shufflevector(lo, __builtin_shufflevector(hi, hi, 0, 1, -1, -1), 0, 1, 2, 3, 4, 5, -1, -1);
        } else {
            const v4i lo = *reinterpret_cast<const v4i*>(base + in + (((2 * fg) ^ fsw) << 4));
            const v4i hi = *reinterpret_cast<const v4i*>(base + in + (((2 * fg + 1) ^ fsw) << 4));
            f.v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        }
        return f;
    };
    constexpr int KS = INT8 ? 2 : 1;                                  // matrix instructions per product and stage
    auto multiply = [&](auto ks, const Frag& x, const Frag& y, acc_t& c) {
        constexpr int k = decltype(ks)::value;
        if constexpr (INT8) c = __builtin_amdgcn_mfma_i32_32x32x32_i8(x.v[k], y.v[k], c, 0, 0, 0);
        else if constexpr (FP6) c = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(x.v, y.v, c, FP6_CODE, FP6_CODE, 0, 0, 0, 0);
        else c = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(x.v, y.v, c, 0, 0, 0, 0, 0, 0);
    };

    static_for<L::loads(S)>([&](auto l) { issue(of_a, idx_t<0>{}, idx_t<S>{}, l, first_a, by_a); });
    static_for<L::loads(S)>([&](auto l) { issue(of_b, idx_t<0>{}, idx_t<S>{}, l, first_b, by_b); });
    if (tid < 128) leading[tid] = tid < 64 ? a.ea[row0 + tid] : a.eb[col0 + tid - 64];
    wait_and_barrier<0>();
    // Column j: the pairs of B slice S - 1 - j with the A slices 0 .. j (0-based); the product of (p, q) goes to accumulator p + q.
    Frag fa[S], fb[S];
    static_for<S>([&](auto p) { fa[p.value] = read_frag(of_a, p.value); });
    static_for<L::AHEAD>([&](auto j) { fb[j.value] = read_frag(of_b, S - 1 - j.value); });
#pragma unroll 1
    for (int stage = 0; stage < a.chunks; ++stage) {
        const unsigned next = (unsigned)(stage + 1 < a.chunks ? stage + 1 : stage);
        const unsigned next_a = first_a + next * cs_a, next_b = first_b + next * cs_b;
        unsigned step_a = by_a, step_b = by_b;
        asm volatile("" : "+s"(step_a), "+s"(step_b));                // multiplied where they are used: 2 S products would not fit the scalar registers
        static_for<S>([&](auto jc) {
            constexpr int J = decltype(jc)::value;
            constexpr bool last = J + 1 == S;
            if constexpr (J == L::A_FREE) wait_and_barrier<63>();     // every wave has read the A slices of this stage
            if constexpr (J == L::MIDDLE) wait_and_barrier<L::LATE == 0 ? 63 : L::loads(S)>();      // late B slices are here, early ones done with
            if constexpr (last) wait_and_barrier<0>();                // A and early B slices of the next stage are here, late B slices done with
            if constexpr (J + L::AHEAD < S) fb[J + L::AHEAD] = read_frag(of_b, S - 1 - J - L::AHEAD);
            __builtin_amdgcn_sched_barrier(0);
            Frag nb[L::AHEAD];
            if constexpr (KS == 2) static_for<J + 1>([&](auto p) { multiply(idx_t<0>{}, fb[J], fa[p.value], acc[S - 1 - J + decltype(p)::value]); });
            static_for<J + 1>([&](auto pc) {
                constexpr int P = decltype(pc)::value, AT = L::start(J) + P;
                multiply(idx_t<KS - 1>{}, fb[J], fa[P], acc[S - 1 - J + P]);
                // the loads, one or more per product from their barrier on
                auto batch = [&](auto op_a, auto from, auto n, auto first, auto end, unsigned at, unsigned by) {
                    constexpr int N = L::loads(decltype(n)::value), SPAN = decltype(end)::value - decltype(first)::value;
                    constexpr int PER = (N + SPAN - 1) / SPAN;
                    static_for<PER>([&](auto u) {
                        constexpr int l = (AT - decltype(first)::value) * PER + decltype(u)::value;
                        if constexpr (AT >= decltype(first)::value && l < N) issue(op_a, from, n, idx_t<l>{}, at, by);
                    });
                };
                batch(of_a, idx_t<0>{}, idx_t<S>{}, idx_t<L::start(L::A_FREE)>{}, idx_t<L::start(L::MIDDLE)>{}, next_a, step_a);
                batch(of_b, idx_t<S - L::EARLY>{}, idx_t<L::EARLY>{}, idx_t<L::start(L::MIDDLE)>{}, idx_t<L::start(S - 1)>{}, next_b, step_b);
                if constexpr (L::LATE > 0) batch(of_b, idx_t<0>{}, idx_t<L::LATE>{}, idx_t<L::start(S - 1)>{}, idx_t<L::PRODUCTS>{}, next_b, step_b);
                if constexpr (last) {
                    if constexpr (P < L::AHEAD) nb[P] = read_frag(of_b, S - 1 - P);
                    fa[P] = read_frag(of_a, P);
                }
                __builtin_amdgcn_sched_barrier(0);
            });
            if constexpr (last) static_for<L::AHEAD>([&](auto t) { fb[t.value] = nb[t.value]; });
        });
    }
    wait_and_barrier<0>();

    // The sums: lane l holds row l & 31 of its wave's 32 x 32 tile, columns 8 (r >> 2) + 4 (l >> 5) + (r & 3), r < 16; four elements
    // side by side, since there is no other wave to fill the gaps between dependent instructions.
    const int64_t mi = row0 + wm * 32 + (lane & 31), first_n = col0 + wn * 32 + (lane >> 5) * 4;
    const int* const lead_b = leading + 64 + wn * 32 + (lane >> 5) * 4;
    const int base_a = leading[wm * 32 + (lane & 31)] - 2 * Scale::BITS - (FLIP ? 2 * S : S - 1) * Scale::STEP;      // and the scale of the first term
    uint64_t* const sum_at = a.S + (((size_t)bn * a.blocks_m + bm) * 4 + wave) * 1024 * SUM_WORDS_MAX + lane;
    uint64_t* const c_at = reinterpret_cast<uint64_t*>(a.C) + mi + first_n * a.ldc;
    const bool combine = a.add_to_C || a.scaled;
    // the vectors off the ladder are not for this kernel to write
    bool row_here = mi < a.m;
    uint32_t cols_off = 0;                                            // of the wave's 32 columns
    if (LISTS && a.off.limit > 0) {
        row_here = row_here && a.off.marks[row0 + wm * 32 + (lane & 31)] == 0;
        cols_off = (uint32_t)__ballot(a.off.marks[a.rows_pad_a + col0 + wn * 32 + (lane & 31)] != 0) >> ((lane >> 5) * 4);
    }
    uint64_t* const mine = reinterpret_cast<uint64_t*>(lds + wave * 8192) + lane;
    static_for<4>([&](auto gc) {
        constexpr int G = decltype(gc)::value;
        LadderSum<FMT, MODE, GO_ON, S> sum[4];
        static_for<4>([&](auto r) {
            if constexpr (GO_ON) sum[r.value].load(sum_at + (4 * G + r.value) * 64, (S - 1) * Scale::STEP);
            else sum[r.value].zero();
        });
        static_for<S>([&](auto at) {
            static_for<4>([&](auto r) { sum[r.value].template add<decltype(at)::value>(acc[FLIP ? decltype(at)::value : S - 1 - decltype(at)::value][4 * G + decltype(r)::value]); });
        });
        static_for<4>([&](auto r) {
            const int n_in = 8 * G + decltype(r)::value;
            if constexpr (FLIP) {
                sum[r.value].store(sum_at + (4 * G + r.value) * 64);
            } else {
                const uint64_t v = sum[r.value].result(base_a + lead_b[n_in]);
                if (combine) mine[(4 * G + decltype(r)::value) * 64] = v;
                else if (row_here && first_n + n_in < a.n && ((cols_off >> n_in) & 1u) == 0) c_at[n_in * a.ldc] = v;
            }
        });
    });
    if (!FLIP && combine) {
        // the block's result meets C (or the product so far): once more by way of the wave's part of the LDS, their code is long
#pragma unroll 1
        for (int r0 = 0; r0 < 16; r0 += 4) {
            uint64_t w[4] = {0, 0, 0, 0}, c[4] = {0, 0, 0, 0};
            bool inside[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t nj = first_n + 2 * r0 + r;
                inside[r] = row_here && nj < a.n && ((cols_off >> (2 * r0 + r)) & 1u) == 0;
                if (inside[r] && a.add_to_C) w[r] = reinterpret_cast<const uint64_t*>(a.W)[mi + nj * a.ldw];
                if (inside[r] && a.use_beta) c[r] = c_at[(2 * r0 + r) * a.ldc];
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                uint64_t v = mine[(r0 + r) * 64];
                if (a.add_to_C) {
                    if constexpr (MODE == ACC_HW) v = (uint64_t)__double_as_longlong(__longlong_as_double((long long)w[r]) + __longlong_as_double((long long)v));
                    else v = fp64_add_emulated(w[r], v);
                }
                if (a.scaled) v = scaled_result<MODE != ACC_HW>(a.alpha, v, a.beta, a.use_beta, c[r]);
                if (inside[r]) c_at[(2 * r0 + r) * a.ldc] = v;
            }
        }
    }
#endif
}

template <int FMT, int MODE, int S>
hipError_t launch_ladder_slices(const LadderArgs& a, int slices, int part, unsigned blocks, hipStream_t st) {
    if constexpr (S > ladder_max_slices(FMT, false)) {
        return hipErrorInvalidValue;
    } else {
        if (slices != S) return launch_ladder_slices<FMT, MODE, S + 1>(a, slices, part, blocks, st);
        const dim3 grid(blocks), block(256);
        constexpr int FEWEST = ladder_min_slices(FMT, true), MOST = ladder_max_slices(FMT, true);
        constexpr bool WHOLE_FITS = MODE != ACC_EXACT || ladder_exact_fits(FMT, S, false), ALL_FIT = MODE != ACC_EXACT || ladder_exact_fits(FMT, S, true);
        if constexpr (S >= ladder_min_slices(FMT, false) && WHOLE_FITS) {
            if (part == WHOLE) {
                hipLaunchKernelGGL((ladder_sums_kernel<FMT, S, MODE, WHOLE>), grid, block, 0, st, a);
                return hipGetLastError();
            }
        }
        if constexpr (S + 1 >= FEWEST && S < MOST && WHOLE_FITS) {
            if (part == LESSER_HALF) {
                hipLaunchKernelGGL((ladder_sums_kernel<FMT, S, MODE, LESSER_HALF>), grid, block, 0, st, a);
                return hipGetLastError();
            }
        }
        if constexpr (S >= FEWEST && S <= MOST && ALL_FIT) {
            if (part == GREATER_HALF) {
                hipLaunchKernelGGL((ladder_sums_kernel<FMT, S, MODE, GREATER_HALF>), grid, block, 0, st, a);
                return hipGetLastError();
            }
        }
        return hipErrorInvalidValue;
    }
}

}  // namespace

template <int FMT, int MODE>
hipError_t launch_ladder_kernel(const LadderArgs& a, int S, int part, unsigned blocks, hipStream_t st) {
    return launch_ladder_slices<FMT, MODE, 6>(a, S, part, blocks, st);
}

}  // namespace ozaki
