// The products of the vectors off the ladder (OffLadder in layout.hpp) where they are few, behind ladder_sums.hpp: 32 such rows of A with 32
// columns of B per workgroup, or 32 such columns with 32 rows, all slice pairs and their sum.  Nothing is known of the exponents here:
// a workgroup of four waves keeps the product of every pair p + q <= s + 1 in accumulators of its own (16 per lane and pair, a quarter of
// the pairs per wave), and after the last stage the products go through LDS, as many at a time as the load ring holds, and every thread
// sums four elements of C in the order and with the rounding of accumulate.hip.
// 16384 x 8192 x 1024 FP8, 13 slices, a dozen vectors of 24576 off the ladder: 0.2 ms, and the call 8.25 ms, where one such vector would
// leave all of it to the GEMM kernels and the accumulation (10.9 ms).
#pragma once
#include <type_traits>
#include <utility>

#include "fp64_emu.hpp"
#include "layout.hpp"

namespace ozaki {

struct OffLadderArgs {
    OffLadder off;
    const uint8_t* sa;       // A slices: [s][chunks][rows_pad_a][row bytes]
    const uint8_t* sb;       // B slices
    const int32_t* ea;       // exponents: [s][rows_pad_a]
    const int32_t* eb;       // [s][rows_pad_b]
    int64_t rows_pad_a, rows_pad_b;
    int chunks;
    int blocks_m, blocks_n;  // 32 vectors each
    int64_t m, n;
    int two_b, p_frac, run_limit, exact;
    double* C;
    int64_t ldc;
    int scaled, use_beta;    // the result is fl(fl(alpha * P) + fl(beta * C)), or fl(alpha * P) without reading C
    uint64_t alpha, beta;
};

template <int FMT>
hipError_t launch_off_ladder_format(const OffLadderArgs& a, int s, bool integer_only, unsigned blocks, hipStream_t st);

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef int v16i __attribute__((ext_vector_type(16)));

#define OZAKI_LPTR(p) ((__attribute__((address_space(3))) void*)(p))

constexpr int MIN_S = OFF_LADDER_MIN_SLICES, MAX_S = OFF_LADDER_MAX_SLICES;
constexpr int AGPR_SLOTS = 16;

// Which wave forms the product of pair (p, q), 0-based, p + q < S: the pairs in the order (0,0) (0,1) ... (1,0) ...  At most
// ceil(pairs / 4) per wave; any such table will do that table_ok takes, these were found by moving pairs about at random and keep the number of different slices that a
// wave reads low.
constexpr const char* OWNERS[MAX_S + 1] = {
    "", "", "", "", "", "",
    "300033300032211221223",
    "1001011102101303303233222223",
    "001133110011331222333222330011222000",
    "111322333000322331113223000222000221113000111",
    "3333222223000022222000022221333111133311110010000333111",
    "003311110010033331100003333110222211112222111003333223332222222000",
    "000220022002000220022000002200220333223322333223321311133333113111111111111113",
    "3332333222323333233322232333233322231112111222111211122111211120000011000001000000000000113",
};

// Position of pair (p, q) in the accumulation order of the triangle: anti-diagonals from the least significant one, p ascending.
constexpr int pair_place(int S, int p, int q) {
    const int g = p + q;                              // 0 .. S - 1
    return S * (S + 1) / 2 - (g + 1) * (g + 2) / 2 + p;
}

template <int S, int W>
struct WaveShare {
    int count = 0, rows = 0, cols = 0;
    int row[S] = {}, col[S] = {};                     // slices of A and of B that the wave reads, ascending
    int slot[S][S] = {};                              // [index in col][index in row]: accumulator, -1: not this wave's pair
    int place[S * (S + 1) / 2] = {};                  // of each accumulator's pair
    constexpr WaveShare() {
        int owner[S][S] = {};
        int at = 0;
        for (int p = 0; p < S; ++p)
            for (int q = 0; q + p < S; ++q) owner[p][q] = OWNERS[S][at++] - '0';
        for (int p = 0; p < S; ++p) {
            bool any = false;
            for (int q = 0; q + p < S; ++q) any = any || owner[p][q] == W;
            if (any) row[rows++] = p;
        }
        for (int q = 0; q < S; ++q) {
            bool any = false;
            for (int p = 0; q + p < S; ++p) any = any || owner[p][q] == W;
            if (any) col[cols++] = q;
        }
        for (int j = 0; j < cols; ++j)
            for (int i = 0; i < rows; ++i) {
                const int p = row[i], q = col[j];
                slot[j][i] = -1;
                if (p + q < S && owner[p][q] == W) {
                    place[count] = pair_place(S, p, q);
                    slot[j][i] = count++;
                }
            }
    }
    // Products of column j before row i, of the columns before column j
    constexpr int in_row(int j, int i) const {
        int c = 0;
        for (int r = 0; r < i; ++r) c += slot[j][r] >= 0 ? 1 : 0;
        return c;
    }
    constexpr int before(int j) const {
        int c = 0;
        for (int i = 0; i < j; ++i) c += in_row(i, rows);
        return c;
    }
    // First column of the tail: the products that hide the first fragment reads of the next stage, a quarter of all or more
    constexpr int tail() const {
        int j = cols, c = 0;
        while (j > 1 && 4 * c < count) c += in_row(--j, rows);
        return j;
    }
};
template <int S, int W> constexpr WaveShare<S, W> SHARE{};
template <int S> constexpr int most_slots() {
    int c = SHARE<S, 0>.count;
    if (SHARE<S, 1>.count > c) c = SHARE<S, 1>.count;
    if (SHARE<S, 2>.count > c) c = SHARE<S, 2>.count;
    if (SHARE<S, 3>.count > c) c = SHARE<S, 3>.count;
    return c;
}
// Every pair has an owner, no wave more than its share, and each at least the two columns that its loop reads ahead.
template <int S> constexpr bool table_ok() {
    constexpr int PAIRS = S * (S + 1) / 2;
    for (int i = 0; i < PAIRS; ++i)
        if (OWNERS[S][i] < '0' || OWNERS[S][i] > '3') return false;
    return OWNERS[S][PAIRS] == 0 && SHARE<S, 0>.count + SHARE<S, 1>.count + SHARE<S, 2>.count + SHARE<S, 3>.count == PAIRS &&
           most_slots<S>() == (PAIRS + 3) / 4 && SHARE<S, 0>.cols >= 2 && SHARE<S, 1>.cols >= 2 && SHARE<S, 2>.cols >= 2 && SHARE<S, 3>.cols >= 2;
}
template <int S>
struct Places {
    int place[4][32] = {};
    constexpr Places() {
        for (int i = 0; i < 32; ++i) {
            place[0][i] = (i < SHARE<S, 0>.count ? SHARE<S, 0>.place[i] : -1);
            place[1][i] = (i < SHARE<S, 1>.count ? SHARE<S, 1>.place[i] : -1);
            place[2][i] = (i < SHARE<S, 2>.count ? SHARE<S, 2>.place[i] : -1);
            place[3][i] = (i < SHARE<S, 3>.count ? SHARE<S, 3>.place[i] : -1);
        }
    }
};

template <int I> using idx_t = std::integral_constant<int, I>;
template <int N, typename F, int... I>
__device__ __forceinline__ void static_for_(F&& f, std::integer_sequence<int, I...>) { (f(idx_t<I>{}), ...); }
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) { static_for_<N>(f, std::make_integer_sequence<int, N>{}); }

// At most N vector-memory operations of this wave outstanding, its LDS operations complete, then the barrier; no fence
// (it would drain the load ring).
template <int N>
__device__ __forceinline__ void wait_and_barrier() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | 0x0070);   // vmcnt(N) expcnt(7) lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

template <int S>
struct Ring {
    static constexpr int LPW = S;                     // loads per wave and stage: two waves per operand, 16 vectors of every slice each
    static constexpr int OPERAND_BYTES = S * 2048, STAGE_BYTES = 2 * OPERAND_BYTES;
    static constexpr int META_BYTES = 4096;
    static constexpr int FIT = (160 * 1024 - META_BYTES) / STAGE_BYTES, MOST = 63 / LPW;
    static constexpr int NSTAGE = FIT < MOST ? (FIT < 6 ? FIT : 6) : (MOST < 6 ? MOST : 6);
    static constexpr int RING_BYTES = NSTAGE * STAGE_BYTES;
    static_assert(NSTAGE >= 3, "the ring needs three stages");
    static_assert(META_BYTES >= 2 * MAX_S * 32 * 4 + MAX_S * (MAX_S + 1) / 2 * 4 + 2 * MAX_S * 4 + 256, "exponents, list of pairs, links and places");
};

// The sum of one thread's R elements of C in any of the three accumulations: accumulate.hip.
template <int MODE, bool PINT, int R>
struct ElementSums {
    static constexpr bool HW = MODE == ACC_HW, EMU = MODE == ACC_EMU, EXACT = MODE == ACC_EXACT;
    typedef typename std::conditional<PINT, int64_t, int>::type run_t;      // exact sum of a run

    double Sd[R];                                     // HW
    RoundedSum E[R];                                  // EMU: x * 2^ex with an integer significand of at most 53 bits
    Fixed192 X[R];                                    // EXACT
    run_t run_sum[R];
    int run_e[R];
    int two_b, p_frac;

    __device__ __forceinline__ void start(int two_b_, int p_frac_) {
        two_b = two_b_;
        p_frac = p_frac_;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            run_sum[r] = 0;
            run_e[r] = 0;
            if constexpr (HW) Sd[r] = 0.0;
            if constexpr (EMU) E[r].start_at_zero();
            if constexpr (EXACT) X[r].clear();
        }
    }
    __device__ __forceinline__ void add_run(int r) {
        if (run_sum[r] == 0) return;                                  // adding an exact zero changes nothing
        if constexpr (HW) Sd[r] = Sd[r] + ldexp((double)run_sum[r], run_e[r] - two_b);
        if constexpr (EMU) E[r].add(run_sum[r], run_e[r] - two_b);
        if constexpr (EXACT) X[r].add((int64_t)run_sum[r], EXACT_WINDOW_BITS + run_e[r]);      // unit: 2^(-2b - window) of the leading scale
    }
    // The stored sum of a run, element r, of scale 2^e: per element, consecutive ones of one anti-diagonal with the same scale
    // are merged further (integer, units of 2^-p_frac) before the FP64 addition.  Together with the tile-wide runs formed before
    // this is the element-wise rule "consecutive pairs of an anti-diagonal with equal scale are summed exactly".
    __device__ __forceinline__ void take(int r, uint32_t word, int e, bool first) {
        // the product as an integer in units of 2^-p_frac: exact in FP32 (|integer| <= 2^24), no FP64 involved
        const int iv = PINT ? (int)word : (int)ldexpf(__uint_as_float(word), p_frac);
        if (!first && e == run_e[r]) {
            run_sum[r] += iv;
        } else {
            add_run(r);
            run_sum[r] = iv;
            run_e[r] = e;
        }
    }
    __device__ __forceinline__ void finish() {
#pragma unroll
        for (int r = 0; r < R; ++r) add_run(r);
    }
    // FP64 bits of the sum of element r times 2^base
    __device__ __forceinline__ uint64_t result(int r, int base) const {
        if constexpr (HW) return (uint64_t)__double_as_longlong(ldexp(Sd[r], base));
        else if constexpr (EMU) return fp64_scale_pow2_emulated(E[r].value(), base);
        else return X[r].round_to_fp64(base - two_b - EXACT_WINDOW_BITS);
    }
};

// After the k loop: products through LDS in the order of the accumulation, four elements of C per thread.
template <int FMT, int S, int MODE, typename ACC>
__device__ __forceinline__ void sum_products(const OffLadderArgs& a, uint8_t* lds, const ACC (&acc)[most_slots<S>()], int wave, int lane, int tid, int place) {
    constexpr bool PINT = FMT == FMT_INT8;
    constexpr int NPAIRS = S * (S + 1) / 2, NSLOT = most_slots<S>();
    typedef typename std::conditional<PINT, v4i, v4f>::type acc4_t;
    constexpr int FIT = Ring<S>::RING_BYTES / 4096;              // products in LDS at a time
    constexpr int ROUNDS = (NPAIRS + FIT - 1) / FIT, PER_ROUND = (NPAIRS + ROUNDS - 1) / ROUNDS;
    int(*const relA)[32] = reinterpret_cast<int(*)[32]>(lds + Ring<S>::RING_BYTES);
    int(*const relB)[32] = relA + MAX_S;
    uint32_t* const entries = reinterpret_cast<uint32_t*>(relB + MAX_S);
    const int ml = lane & 31, nl = wave * 8 + (lane >> 5) * 4;
    const int* const row_at = reinterpret_cast<const int*>(entries + MAX_S * (MAX_S + 1) / 2) + 2 * MAX_S;
    const int* const col_at = row_at + 32;
    ElementSums<MODE, PINT, 4> sums;
    sums.start(a.two_b, a.p_frac);
#pragma unroll 1
    for (int lo = 0; lo < NPAIRS; lo += PER_ROUND) {
        const int hi = lo + PER_ROUND < NPAIRS ? lo + PER_ROUND : NPAIRS;
#pragma unroll
        for (int i = 0; i < NSLOT; ++i) {
            const int z = __builtin_amdgcn_readlane(place, i);
            if (z >= lo && z < hi) {
                uint8_t* const dst = lds + (z - lo) * 4096 + lane * 16;
#pragma unroll
                for (int g4 = 0; g4 < 4; ++g4)
                    *reinterpret_cast<acc4_t*>(dst + g4 * 1024) = acc4_t{acc[i][4 * g4], acc[i][4 * g4 + 1], acc[i][4 * g4 + 2], acc[i][4 * g4 + 3]};
            }
        }
        __syncthreads();
        for (int z = lo; z < hi;) {
            const uint32_t entry = __builtin_amdgcn_readfirstlane(entries[z]);
            const int p = entry & 31, q = (entry >> 5) & 31;
            const bool first = (entry >> 10) & 1;
            int len = entry >> 11;
            len = len < hi - z ? len : hi - z;
            const uint8_t* src = lds + (z - lo) * 4096 + tid * 16;
            z += len;
            // a run that the whole tile shares: exact in the format of the products, whatever the data (run_limit)
            v4i w = *reinterpret_cast<const v4i*>(src);
            auto plus = [](const v4i& x, const v4i& y) -> v4i {
                v4i t;
#pragma unroll
                for (int r = 0; r < 4; ++r) t[r] = PINT ? x[r] + y[r] : __float_as_int(__int_as_float(x[r]) + __int_as_float(y[r]));
                return t;
            };
            for (--len; len >= 3; len -= 3) {
                const v4i x0 = *reinterpret_cast<const v4i*>(src + 4096), x1 = *reinterpret_cast<const v4i*>(src + 8192),
                          x2 = *reinterpret_cast<const v4i*>(src + 12288);
                w = plus(plus(plus(w, x0), x1), x2);
                src += 12288;
            }
            for (; len > 0; --len) {
                src += 4096;
                w = plus(w, *reinterpret_cast<const v4i*>(src));
            }
            const int eA = p == 0 ? 0 : relA[p][ml];
#pragma unroll
            for (int r = 0; r < 4; ++r) sums.take(r, (uint32_t)w[r], eA + (q == 0 ? 0 : relB[q][nl + r]), first);
        }
        if (hi < NPAIRS) __syncthreads();
    }
    sums.finish();
    const int mi = row_at[ml];                                        // negative: not this workgroup's
    if (mi < 0) return;
    const int baseA = relA[0][ml];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int nj = col_at[nl + r];
        if (nj < 0) continue;
        uint64_t* const dst = reinterpret_cast<uint64_t*>(a.C) + mi + (int64_t)nj * a.ldc;
        uint64_t v = sums.result(r, baseA + relB[0][nl + r]);
        if (a.scaled) v = scaled_result<MODE != ACC_HW>(a.alpha, v, a.beta, a.use_beta, a.use_beta ? *dst : 0);
        *dst = v;
    }
}

template <int FMT, int S, bool INTEGER_ONLY>
__global__ void __launch_bounds__(256, 1) off_ladder_kernel(const OffLadderArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)                                   // buffer descriptors are not a type on the host
    typedef Ring<S> R;
    static_assert(table_ok<S>(), "OWNERS");
    constexpr bool INT8 = FMT == FMT_INT8;
    constexpr int BK = CHUNK_BYTES;
    constexpr int NSLOT = most_slots<S>();
    __shared__ __attribute__((aligned(16))) uint8_t lds[R::RING_BYTES + R::META_BYTES];      // one array: see ladder_sums.hpp
    static __constant__ const Places<S> places;

    if (!on_ladder(a.off)) return;
    const bool of_a = (int)blockIdx.x < a.off.limit / 32 * a.blocks_n;          // rows of A off the ladder, else columns of B
    const unsigned at = of_a ? blockIdx.x : blockIdx.x - a.off.limit / 32 * a.blocks_n;
    const unsigned across = of_a ? a.blocks_n : a.blocks_m, panel = at / across, other = at - panel * across;
    const int count = a.off.counts[of_a ? 0 : 1];
    if ((int)panel * 32 >= count) return;
    const int* const listed = a.off.list + (of_a ? 0 : a.off.limit);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Row r of the workgroup's rows of A or columns of B: one of the list (the last one again beyond its end) or one of 32 side by side
    auto vector_of = [&](bool a_rows, int r) -> int {
        const int i = (int)panel * 32 + r;
        return a_rows == of_a ? listed[i < count ? i : count - 1] : (int)other * 32 + r;
    };

    // Loader: waves 0 and 1 fetch the B slices of a stage, waves 2 and 3 the A slices, S kilobytes each.  A slice's place in the
    // operand is a scalar offset, the vector's and the stage's the lanes' (an operand's slices take less than 2 GiB: ladder_possible).
    const bool is_b = wave < 2;
    const int half = wave & 1;
    const unsigned rows_pad = (unsigned)(is_b ? a.rows_pad_b : a.rows_pad_a);
    const unsigned cs = rows_pad * BK, slice = cs * (unsigned)a.chunks;           // chunk stride, slice stride
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(is_b ? a.sb : a.sa), 0, slice * (unsigned)S, 0x00027000);
    const unsigned lrow = lane >> 2;                                  // a kilobyte is 16 vectors, swizzled on the global side
    unsigned voff = (unsigned)vector_of(!is_b, half * 16 + (int)lrow) * BK + (((lane & 3) ^ ((lrow >> 2) & 3)) << 4);
    const int lds_at = is_b ? 0 : R::OPERAND_BYTES;
    auto issue_one = [&](auto ic, uint8_t* stage_at) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, OZAKI_LPTR(stage_at + lds_at + ic.value * 2048 + half * 1024), 16, voff, (unsigned)ic.value * slice, 0, 0);
    };
    int issued = 0;
    auto next_stage = [&] {
        // after the last stage the offsets stay put: the (unused) reloads keep the outstanding-load count uniform
        const unsigned by = issued + 1 < a.chunks ? cs : 0;
        voff += by;
        ++issued;
    };

    // exponents of the tile's rows and columns, asked for before the slices
    int exp_a[2] = {}, exp_b[2] = {};
    const int my_row = vector_of(true, tid & 31), my_col = vector_of(false, tid & 31);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int p = (tid >> 5) + 8 * i;
        if (p < S) {
            exp_a[i] = a.ea[(int64_t)p * a.rows_pad_a + my_row];
            exp_b[i] = a.eb[(int64_t)p * a.rows_pad_b + my_col];
        }
    }
    // what the workgroup writes: of columns off the ladder the rows on it
    const bool listed_too = (int)panel * 32 + (tid & 31) < count;
    const bool row_here = of_a ? listed_too : my_row < a.m && a.off.marks[my_row] == 0;
    const bool col_here = of_a ? my_col < a.n : listed_too;
    static_assert(S <= 16, "two slices' exponents per thread");
    // lane i: where the product of the wave's slot i comes in the accumulation
    int place = places.place[wave][lane & 31];
    int(*const relA)[32] = reinterpret_cast<int(*)[32]>(lds + R::RING_BYTES);
    int(*const relB)[32] = relA + MAX_S;
    uint32_t* const entries = reinterpret_cast<uint32_t*>(relB + MAX_S);

    typedef typename std::conditional<INT8, v16i, v16f>::type acc_t;
    acc_t acc[NSLOT];
#pragma unroll
    for (int i = 0; i < NSLOT; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] = 0;

    static_for<R::NSTAGE - 1>([&](auto st) {
        static_for<R::LPW>([&](auto i) { issue_one(i, lds + st.value * R::STAGE_BYTES); });
        next_stage();
    });

    struct Frag { typename std::conditional<INT8, v4i[2], v8i>::type v; };
    const int frow = lane & 31, fg = lane >> 5, fsw = (frow >> 2) & 3;
    auto read_frag = [&](const uint8_t* stage, bool of_rows, int p) -> Frag {
        Frag f;
        const uint8_t* const base = stage + (of_rows ? R::OPERAND_BYTES : 0) + p * 2048 + frow * BK;
        if constexpr (INT8) {
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) f.v[ks] = *reinterpret_cast<const v4i*>(base + (((2 * ks + fg) ^ fsw) << 4));
        } else {
            const v4i lo = *reinterpret_cast<const v4i*>(base + (((2 * fg) ^ fsw) << 4));
            const v4i hi = *reinterpret_cast<const v4i*>(base + (((2 * fg + 1) ^ fsw) << 4));
            f.v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        }
        return f;
    };
    // The compiler keeps the results of the builtins in the 256 accumulator registers, 16 slots' worth; further slots go to ordinary
    // registers, of which this kernel has 256 too, by instructions of their own.  Their hazards are not the compiler's
    // business: the wait states after a write of a source register stand in front of them, and a result is only read by the next product of the
    // same slot, as the summand that it writes in place (which needs none but those; with INT8 the two steps of a product are a column
    // apart, three instructions for 11 slices), and after the wait states behind the k loop.  That nothing else touches those registers inside
    // the loop is checked on the built kernels (tests/test_off_ladder_listing.py).
    constexpr int KS = INT8 ? 2 : 1;                                  // matrix instructions per slot and stage
    auto multiply = [&](auto slot, auto ks, const Frag& x, const Frag& y, acc_t& c) {
        constexpr int k = decltype(ks)::value;
        if constexpr (decltype(slot)::value >= AGPR_SLOTS) {
            if constexpr (INT8) asm volatile("s_nop 1\n\tv_mfma_i32_32x32x32_i8 %0, %1, %2, %0" : "+v"(c) : "v"(x.v[k]), "v"(y.v[k]));
            else asm volatile("s_nop 1\n\tv_mfma_f32_32x32x64_f8f6f4 %0, %1, %2, %0" : "+v"(c) : "v"(x.v), "v"(y.v));
        } else if constexpr (INT8) {
            c = __builtin_amdgcn_mfma_i32_32x32x32_i8(x.v[k], y.v[k], c, 0, 0, 0);
        } else {
            c = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(x.v, y.v, c, 0, 0, 0, 0, 0, 0);
        }
    };

    // One stage: the wave's products column by column (a column: the pairs of one B slice), fragments read two columns ahead, the
    // loads of the stage NSTAGE - 1 ahead spread between the products.  The last TAIL columns come after the barrier: they hide the
    // reads of the next stage's first fragments.  The scheduling barriers keep this order.
    wait_and_barrier<(R::NSTAGE - 2) * R::LPW>();
    auto k_loop = [&](auto wc) {
        constexpr int W = decltype(wc)::value;
        constexpr int ROWS = SHARE<S, W>.rows, COLS = SHARE<S, W>.cols, TAIL = SHARE<S, W>.tail(), HEAD = SHARE<S, W>.before(TAIL);
        auto a_frag = [&](auto i, const uint8_t* at) { return read_frag(at, true, SHARE<S, W>.row[decltype(i)::value]); };
        auto b_frag = [&](auto j, const uint8_t* at) { return read_frag(at, false, SHARE<S, W>.col[decltype(j)::value]); };
        Frag fa[ROWS], fb[COLS];
        fb[0] = b_frag(idx_t<0>{}, lds);
        static_for<ROWS>([&](auto i) { fa[i.value] = a_frag(i, lds); });
        fb[1] = b_frag(idx_t<1>{}, lds);
        int buf = 0;
#pragma unroll 1
        for (int stage = 0; stage < a.chunks; ++stage) {
            const uint8_t* const base = lds + buf * R::STAGE_BYTES;
            uint8_t* const refill = lds + (buf == 0 ? R::NSTAGE - 1 : buf - 1) * R::STAGE_BYTES;
            buf = buf + 1 == R::NSTAGE ? 0 : buf + 1;
            const uint8_t* const nbase = lds + buf * R::STAGE_BYTES;
            static_for<TAIL>([&](auto j) {
                constexpr int J = decltype(j)::value;
                static_for<COLS>([&](auto t) {
                    if constexpr (t.value == J + 2 || (J + 1 == TAIL && t.value > J + 2)) fb[t.value] = b_frag(t, base);
                });
                __builtin_amdgcn_sched_barrier(0);
                static_for<KS>([&](auto ks) {
                    static_for<ROWS>([&](auto i) {
                        constexpr int slot = SHARE<S, W>.slot[J][decltype(i)::value];
                        if constexpr (slot >= 0) {
                            multiply(idx_t<slot>{}, ks, fb[J], fa[i.value], acc[slot]);
                            if constexpr (decltype(ks)::value == 0) {
                                constexpr int at = SHARE<S, W>.before(J) + SHARE<S, W>.in_row(J, decltype(i)::value);      // of HEAD products
                                static_for<R::LPW>([&](auto l) {
                                    if constexpr (decltype(l)::value * HEAD / R::LPW == at) issue_one(l, refill);
                                });
                            }
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    });
                });
            });
            next_stage();
            // this stage's fragments are all in registers: its part of the ring is free once every wave is here
            wait_and_barrier<(R::NSTAGE - 2) * R::LPW>();
            Frag na[ROWS];
            const Frag nb0 = b_frag(idx_t<0>{}, nbase);
            static_for<ROWS>([&](auto i) { na[i.value] = a_frag(i, nbase); });
            const Frag nb1 = b_frag(idx_t<1>{}, nbase);
            __builtin_amdgcn_sched_barrier(0);
            static_for<COLS - TAIL>([&](auto t) {
                constexpr int J = TAIL + decltype(t)::value;
                static_for<KS>([&](auto ks) {
                    static_for<ROWS>([&](auto i) {
                        constexpr int slot = SHARE<S, W>.slot[J][decltype(i)::value];
                        if constexpr (slot >= 0) multiply(idx_t<slot>{}, ks, fb[J], fa[i.value], acc[slot]);
                    });
                });
            });
            static_for<ROWS>([&](auto i) { fa[i.value] = na[i.value]; });
            fb[0] = nb0;
            fb[1] = nb1;
            __builtin_amdgcn_sched_barrier(0);
        }
        static_for<SHARE<S, W>.count>([&](auto i) {                   // the last products have left the pipeline
            acc_t& products = acc[i.value];
            if constexpr (decltype(i)::value >= AGPR_SLOTS) asm volatile("s_nop 15\n\ts_nop 15" : "+v"(products));
        });
    };
    if (wave == 0) k_loop(idx_t<0>{});
    else if (wave == 1) k_loop(idx_t<1>{});
    else if (wave == 2) k_loop(idx_t<2>{});
    else k_loop(idx_t<3>{});
    // every direct-to-LDS load (the tail's unused reloads too) must have landed before the ring is used for the products
    wait_and_barrier<0>();

#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int p = (tid >> 5) + 8 * i;
        if (p < S) {
            relA[p][tid & 31] = exp_a[i];
            relB[p][tid & 31] = exp_b[i];
        }
    }
    int* const linkA = reinterpret_cast<int*>(entries + MAX_S * (MAX_S + 1) / 2);
    int* const linkB = linkA + MAX_S;
    int* const row_at = linkB + MAX_S;
    int* const col_at = row_at + 32;
    if (tid < 32) {
        row_at[tid] = row_here ? my_row : -1;
        col_at[tid] = col_here ? my_col : -1;
    }
    __syncthreads();
    // Slot 0 keeps the first-slice exponent, slots p >= 1 the difference to it.  Half a wave per slice: is c_p - c_(p+1) the same for
    // all rows / columns of the tile?
    int rel_a[2], rel_b[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int p = (tid >> 5) + 8 * i, r = tid & 31, half_at = lane & 32;
        if (p < S) {
            rel_a[i] = p == 0 ? exp_a[i] : exp_a[i] - relA[0][r];
            rel_b[i] = p == 0 ? exp_b[i] : exp_b[i] - relB[0][r];
            const bool last = p + 1 == S;
            const int dA = last ? 0 : exp_a[i] - relA[p + 1][r], dB = last ? 0 : exp_b[i] - relB[p + 1][r];
            const int refA = __shfl(dA, half_at, 64), refB = __shfl(dB, half_at, 64);
            const uint64_t okA = __ballot(dA == refA), okB = __ballot(dB == refB);
            if (r == 0) {
                linkA[p] = !last && (uint32_t)(okA >> half_at) == 0xFFFFFFFFu ? refA : DELTA_IRREGULAR;
                linkB[p] = !last && (uint32_t)(okB >> half_at) == 0xFFFFFFFFu ? refB : DELTA_IRREGULAR;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int p = (tid >> 5) + 8 * i;
        if (p < S) {
            relA[p][tid & 31] = rel_a[i];
            relB[p][tid & 31] = rel_b[i];
        }
    }
    // entries[z]: the z-th pair in accumulation order, 0-based slices p | q << 5 | first of its anti-diagonal << 10 | length of the run from here << 11
    constexpr int NPAIRS = S * (S + 1) / 2;
    if (tid < NPAIRS) {
        int g = S - 1, z = tid;                                       // p + q, 0-based; g + 1 pairs
        while (z >= g + 1) z -= 1 + g--;
        const int p = z, q = g - z;
        int run = 1;
        while (z + run < g + 1 && run < a.run_limit && deltas_link(linkA[p + run - 1], linkB[q - run])) ++run;
        entries[tid] = (uint32_t)p | (uint32_t)q << 5 | (uint32_t)(z == 0) << 10 | (uint32_t)run << 11;
    }
    // (the first barrier of sum_products stands between these writes and their readers)
    if constexpr (INTEGER_ONLY) {
        if (a.exact) sum_products<FMT, S, ACC_EXACT>(a, lds, acc, wave, lane, tid, place);
        else sum_products<FMT, S, ACC_EMU>(a, lds, acc, wave, lane, tid, place);
    } else {
        sum_products<FMT, S, ACC_HW>(a, lds, acc, wave, lane, tid, place);
    }
#endif
}

template <int FMT, bool INTEGER_ONLY, int S>
hipError_t launch_off_ladder_slices(const OffLadderArgs& a, int slices, unsigned blocks, hipStream_t st) {
    if constexpr (S > MAX_S || S > ladder_max_slices(FMT, false)) {
        return hipErrorInvalidValue;
    } else {
        if (slices != S) return launch_off_ladder_slices<FMT, INTEGER_ONLY, S + 1>(a, slices, blocks, st);
        hipLaunchKernelGGL((off_ladder_kernel<FMT, S, INTEGER_ONLY>), dim3(blocks), dim3(256), 0, st, a);
        return hipGetLastError();
    }
}

}  // namespace

template <int FMT>
hipError_t launch_off_ladder_format(const OffLadderArgs& a, int s, bool integer_only, unsigned blocks, hipStream_t st) {
    return integer_only ? launch_off_ladder_slices<FMT, true, MIN_S>(a, s, blocks, st) : launch_off_ladder_slices<FMT, false, MIN_S>(a, s, blocks, st);
}

}  // namespace ozaki
