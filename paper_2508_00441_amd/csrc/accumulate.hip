// Accumulation of the slice-pair products into FP64 and the final rescale (paper Section 3, Eq. 10 and the
// paragraph after Eq. 11; Section 4.2 for the integer-only variants; Section 4.3 for the block sum).
//
// For one k-block, element (i, j), the pairs (p, q) are visited least significant anti-diagonal first, p
// ascending inside one.  The term of a pair is P_pq(i,j) * 2^e with e = (cA_p(i) - cA_1(i)) + (cB_q(j) - cB_1(j)).
// Rule "runs": inside an anti-diagonal, consecutive pairs with the same e form a run.  A run is summed exactly (an
// integer in units of 2^-2b: at most 32 products of at most 2^24, or 2^31 for INT8 slices, units each) and added to
// the block sum S with ONE rounded FP64 addition.  The GEMM kernel has already formed part of these sums in the
// matrix unit's accumulators, as far as the exact window of Eq. 11 reaches (in the worst case, or measured: RunCheck in
// layout.hpp) and where a whole 32 x 32 tile shares the scale; the rest is merged here, element by element.  Rule "plain": every
// product is added with its own rounded addition (the GEMM kernel then stores every pair on its own).  Then
//     C   = S * 2^(cA_1(i) + cB_1(j))            first block
//     C  += S * 2^(cA_1(i) + cB_1(j))            later blocks (one more FP64 addition)
// Scaling by a power of two commutes with rounding (inside the normal range), so summing with exponents
// relative to the first slice and rescaling once gives the same bits as scaling every term by
// 2^(cA_p + cB_q) as Eq. 10 writes it.  P_pq is the FP32 value left by the matrix unit; it already
// contains the factor 2^-2b of the two slice entries and is an exact integer multiple of 2^-2b.  (FP6 codes
// hold twice the slice value: the stored product is four times too large, an integer multiple of 2^-(2b-2); it
// is read as that integer and still weighted 2^-2b.  INT8 slices leave the INT32 integer itself.)
//
// Three instantiations of the sum: hardware FP64 (int->double convert, ldexp, add -- no multiply); integer-emulated
// FP64 (fp64_emu.hpp), which executes no FP64 instruction at all and returns the same bits; and the exact mode, a
// 192-bit fixed-point integer per element that takes every run without rounding and is rounded once at the end
// (integer-only as well).
//
// One workgroup handles one 32 x 32 MFMA tile position of a 256 x 256 tile (256 threads x 4 consecutive
// columns of C each), reading the products in the order the GEMM kernel stored them.
#include <string.h>

#include <type_traits>

#include "fp64_emu.hpp"
#include "layout.hpp"

namespace ozaki {

namespace {

struct AccArgs {
    OffLadder off;           // is there anything to do?
    const float* P;          // [nz][quads_n][quads_m][QUAD_ELEMS] FP32 (or INT32) words
    uint64_t* S;             // running block sum, word w of an element at S[w * plane + element] (may be null when unused)
    double* C;
    int64_t ldc;
    const int32_t* ea;       // exponents of the block: [s][rows_pad_a]
    const int32_t* eb;       // [s][rows_pad_b]
    int64_t rows_pad_a, rows_pad_b;
    int64_t m, n;
    int tiles_m, tiles_n;
    int quads_m, quads_n;
    int two_b;               // 2b: a term is (stored product) * 2^(p_frac - two_b) * 2^e
    int p_frac;              // the stored products are integer multiples of 2^-p_frac (2b; 2b - 2 for FP6 codes; 0 for INT32)
    int read_S, write_S, add_to_C;
    int allow_chain;         // the GEMM kernel summed tile-wide runs
    const uint8_t* starts;   // measured runs (RunCheck), or null
    int merge;               // rule "runs": merge equal-scale products of an anti-diagonal element by element
    const int32_t* da;       // deltas of the block: [s][rows_pad_a / 32]; null: formed here from the exponents
    const int32_t* db;       // [s][rows_pad_b / 32]
    PairOrder order;
    Pass pass;
    int early;               // the first products are asked for before the list of runs
    const double* W;         // add_to_C: what the block is added to (C itself, or the product so far)
    int64_t ldw;
    uint64_t alpha, beta;    // SCALED: the result is fl(fl(alpha * P) + fl(beta * C)), of fl(alpha * P) without reading C
    int use_beta;
};

// Verification export: is pair `pos` of anti-diagonal g (0-based position) stored on its own, i.e. does it start a run of
// the GEMM kernel?
// dA / dB: the block's deltas advanced to the group of the 32 rows / 32 columns concerned, ga / gb: groups per slice;
// p, q 0-based slice indices of the pair.
__device__ __forceinline__ bool starts_run(const PairOrder& o, int allow_chain, const int32_t* dA, int64_t ga, const int32_t* dB,
                                           int64_t gb, int pos, int p, int q) {
    return pos % o.group_len == 0 || !(allow_chain && pair_linked(dA, ga, dB, gb, p - 1, q + 1));
}

// R elements per thread: 4 (one workgroup per 32 x 32 position) or 1 (four workgroups per position, each eight of its
// columns).  DEPTH product loads are kept in flight per thread.
// SCALED: the last step of the last block of a product C = alpha * (A B) + beta * C.
// BEHIND: behind launch_ladder_sums.
template <int MODE, bool PINT, int R, int DEPTH, bool SCALED, bool BEHIND = false>
__device__ __forceinline__ void accumulate_body(const AccArgs& a) {
    static_assert(R == 4 || R == 1, "a thread reads 16 bytes or one word of a stored product");
    constexpr bool HW = MODE == ACC_HW, EMU = MODE == ACC_EMU, EXACT = MODE == ACC_EXACT;
    typedef typename std::conditional<PINT, int64_t, int>::type run_t;      // exact sum of a run
    __shared__ int relA[MAX_SLICES][32];
    __shared__ int relB[MAX_SLICES][32];
    __shared__ uint32_t entries[MAX_PAIRS];           // stored runs of this tile: slot | p << 12 | q << 18 | first-of-diagonal << 24
    __shared__ int32_t linkA[MAX_SLICES], linkB[MAX_SLICES];      // deltas of the 32 rows / 32 columns, per slice
    __shared__ uint8_t starts[MAX_PAIRS];
    __shared__ int n_entries;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const unsigned place = R == 4 ? blockIdx.x : blockIdx.x >> 2;
    const int g4 = R == 4 ? tid >> 6 : (int)(blockIdx.x & 3);         // the eight columns of the position the thread works on
    const int r0 = R == 4 ? 0 : tid >> 6;             // first of its R consecutive columns there
    const int pos = place & 63;                       // wave*16 + sub
    const int tile = place >> 6;
    const int tn = tile / a.tiles_m, tm = tile - tn * a.tiles_m;
    const int wave = pos >> 4, sub = pos & 15;
    const int wn = wave >> 1, wm = wave & 1, ti = sub >> 2, tj = sub & 3;
    const int64_t m0 = (int64_t)tm * TILE + wm * 128 + tj * 32;       // first row of C of this 32 x 32 position
    const int64_t n0 = (int64_t)tn * TILE + wn * 128 + ti * 32;       // first column
    if (m0 >= a.m || n0 >= a.n) return;               // padding only
    if (BEHIND && on_ladder(a.off)) return;

    const int ml = lane & 31;
    const int nl = g4 * 8 + (lane >> 5) * 4 + r0;
    const size_t tile_off = ((size_t)(tn * 2 + wn) * a.quads_m + tm * 2 + wm) * QUAD_ELEMS + (size_t)sub * 1024 + (size_t)(g4 * 64 + lane) * 4 + r0;
    const size_t pair_stride = (size_t)a.quads_m * a.quads_n * QUAD_ELEMS;
    struct Words { uint32_t w[R]; };
    auto load_slot = [&](unsigned slot) -> Words {
        const float* src = a.P + (size_t)slot * pair_stride + tile_off;
        if constexpr (R == 4) {
            const uint4 v = *reinterpret_cast<const uint4*>(src);
            return Words{{v.x, v.y, v.z, v.w}};
        } else {
            return Words{{*reinterpret_cast<const uint32_t*>(src)}};
        }
    };
    // The first pair of every group starts a run, whatever the exponents: where `early` says so, the first DEPTH of those products are
    // asked for now, and are the ones needed where the GEMM kernel stored nothing else (regular ladders).  See launch_accumulate.
    constexpr bool EARLY = R == 4 && (PINT || !EMU);
    Words v[DEPTH];
    if (EARLY && a.early && a.pass.npairs > 0) {
        int g = a.pass.g_hi, len = diag_len(a.order, g), at = 0, slot = 0;      // the group at position `at` of anti-diagonal g, whose first slot is `slot`
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            v[d] = load_slot((unsigned)(slot + at));                  // (past the last group: once more the last one)
            if (at + a.order.group_len < len) {
                at += a.order.group_len;
            } else if (g > a.pass.g_lo) {
                slot += len;
                len = diag_len(a.order, --g);
                at = 0;
            }
        }
    }

    // exponents of the 32 rows and 32 columns: slot 0 keeps the first-slice exponent, slots p >= 1 the difference to it
    for (int idx = tid; idx < a.order.s * 32; idx += 256) {
        const int p = idx >> 5, r = idx & 31;
        const int ca = a.ea[(int64_t)p * a.rows_pad_a + m0 + r], ca1 = a.ea[m0 + r];
        const int cb = a.eb[(int64_t)p * a.rows_pad_b + n0 + r], cb1 = a.eb[n0 + r];
        relA[p][r] = p == 0 ? ca1 : ca - ca1;
        relB[p][r] = p == 0 ? cb1 : cb - cb1;
    }
    if (a.starts != nullptr)
        for (int z = tid; z < a.pass.npairs; z += 256) starts[z] = a.starts[((size_t)z * a.tiles_m * a.tiles_n + tile) * 64 + pos];
    // the deltas that decide where the GEMM kernel ended its runs at this position: fetched once, all at the same time
    if (a.da == nullptr) {
        // (below, from the exponents in LDS)
    } else if (tid < a.order.s) linkA[tid] = a.da[(int64_t)tid * (a.rows_pad_a / LINK_ROWS) + m0 / LINK_ROWS];
    else if (tid >= 64 && tid - 64 < a.order.s) linkB[tid - 64] = a.db[(int64_t)(tid - 64) * (a.rows_pad_b / LINK_ROWS) + n0 / LINK_ROWS];
    __syncthreads();

    if (a.da == nullptr && a.starts == nullptr) {
        // half a wave per slice: is c_p - c_(p+1) the same for all real rows / columns of the position?
        for (int idx = tid; idx < a.order.s * 32; idx += 256) {
            const int p = idx >> 5, r = idx & 31, half = lane & 32;
            const bool last = p + 1 == a.order.s;
            const int dA = last ? 0 : (p == 0 ? 0 : relA[p][r]) - relA[p + 1][r], dB = last ? 0 : (p == 0 ? 0 : relB[p][r]) - relB[p + 1][r];
            const int refA = __shfl(dA, half, 64), refB = __shfl(dB, half, 64);
            const uint64_t okA = __ballot(m0 + r >= a.m || dA == refA), okB = __ballot(n0 + r >= a.n || dB == refB);
            if (r == 0) {
                linkA[p] = !last && (uint32_t)(okA >> half) == 0xFFFFFFFFu ? refA : DELTA_IRREGULAR;
                linkB[p] = !last && (uint32_t)(okB >> half) == 0xFFFFFFFFu ? refB : DELTA_IRREGULAR;
            }
        }
        __syncthreads();
    }

    // the block sum of this thread's elements, in the representation of the mode
    double Sd[R];                                     // HW
    RoundedSum E[R];                                  // EMU: x * 2^ex with an integer significand of at most 53 bits
    Fixed192 X[R];                                    // EXACT
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if constexpr (HW) Sd[r] = a.read_S ? __longlong_as_double((long long)a.S[tile_off + r]) : 0.0;
        if constexpr (EMU) {
            if (a.read_S) E[r].start_at(a.S[tile_off + r]);
            else E[r].start_at_zero();
        }
        if constexpr (EXACT) {
            if (a.read_S) {
                X[r].w0 = a.S[tile_off + r];
                X[r].w1 = a.S[pair_stride + tile_off + r];
                X[r].w2 = a.S[2 * pair_stride + tile_off + r];
            } else {
                X[r].clear();
            }
        }
    }

    // The stored runs of this 32 x 32 position, in accumulation order: a pair starts a run unless it is linked (for
    // the whole position) to the pair before it inside its group; for measured runs the GEMM kernel wrote it down.  Built by the first wave, one anti-diagonal at a time
    // (an anti-diagonal has at most 32 pairs).
    if (tid < 64) {
        int count = 0, slot0 = 0;
        const bool group_start = tid % a.order.group_len == 0;
        for (int g = a.pass.g_hi; g >= a.pass.g_lo; --g) {
            const int len = diag_len(a.order, g);
            bool start = false;
            uint32_t entry = 0;
            if (tid < len) {
                const int p = diag_first_p(a.order, g) + tid - 1, q = g - p - 2;     // 0-based slice indices
                const bool first = tid == 0;                                        // first pair of the anti-diagonal: ends every run
                start = a.starts != nullptr ? starts[slot0 + tid] != 0                          // stored on its own
                                            : group_start || !(a.allow_chain && pair_linked(linkA, 1, linkB, 1, p - 1, q + 1));
                entry = (uint32_t)(slot0 + tid) | ((uint32_t)p << 12) | ((uint32_t)q << 18) | ((uint32_t)first << 24);
            }
            const unsigned long long mask = __ballot(start);
            if (start) entries[count + __popcll(mask & ((1ull << tid) - 1ull))] = entry;
            count += __popcll(mask);
            slot0 += len;
        }
        if (tid == 0) n_entries = count;
    }
    __syncthreads();
    const int n_runs = n_entries;

    auto add_run = [&](int r, run_t run_sum, int run_e) {
        if (run_sum == 0) return;                                     // adding an exact zero changes nothing
        if constexpr (HW) Sd[r] = Sd[r] + ldexp((double)run_sum, run_e - a.two_b);
        if constexpr (EMU) E[r].add(run_sum, run_e - a.two_b);
        if constexpr (EXACT) X[r].add((int64_t)run_sum, EXACT_WINDOW_BITS + run_e);      // unit: 2^(-2b - window) of the leading scale
    };
    // Per element, consecutive stored runs of one anti-diagonal with the same scale are merged further (integer,
    // units of 2^-p_frac) before the FP64 addition: together with the tile-wide runs formed by the GEMM
    // kernel this is the element-wise rule "consecutive pairs of an anti-diagonal with equal scale are summed exactly".
    run_t run_sum[R] = {};
    int run_e[R] = {};
    auto process = [&](uint32_t entry, const Words& v) {
        const int p = (entry >> 12) & 63, q = (entry >> 18) & 63;
        const bool first = (entry >> 24) & 1;
        const int eA = p == 0 ? 0 : relA[p][ml];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int e = eA + (q == 0 ? 0 : relB[q][nl + r]);
            // the product as an integer in units of 2^-p_frac: exact in FP32 (|integer| <= 2^24), no FP64 involved
            const int iv = PINT ? (int)v.w[r] : (int)ldexpf(__uint_as_float(v.w[r]), a.p_frac);
            if (a.merge && !first && e == run_e[r]) {
                run_sum[r] += iv;
            } else {
                add_run(r, run_sum[r], run_e[r]);
                run_sum[r] = iv;
                run_e[r] = e;
            }
        }
    };
    auto load_run = [&](int i) -> Words { return load_slot(entries[i < n_runs ? i : n_runs - 1] & 0xFFFu); };
    // DEPTH loads in flight per thread; the loop is unrolled by DEPTH so that each load keeps its registers
    if (n_runs > 0) {
        if (!EARLY || !a.early || n_runs != a.pass.ngroups) {                             // not the products asked for above
#pragma unroll
            for (int d = 0; d < DEPTH; ++d) v[d] = load_run(d);
        }
        int i = 0;
        for (; i + DEPTH <= n_runs; i += DEPTH) {
#pragma unroll
            for (int d = 0; d < DEPTH; ++d) {
                const Words w = v[d];
                v[d] = load_run(i + DEPTH + d);
                process(entries[i + d], w);
            }
        }
#pragma unroll
        for (int d = 0; d < DEPTH - 1; ++d)
            if (i + d < n_runs) process(entries[i + d], v[d]);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) add_run(r, run_sum[r], run_e[r]);

    if (a.write_S) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if constexpr (HW) a.S[tile_off + r] = (uint64_t)__double_as_longlong(Sd[r]);
            if constexpr (EMU) a.S[tile_off + r] = E[r].value();
            if constexpr (EXACT) {
                a.S[tile_off + r] = X[r].w0;
                a.S[pair_stride + tile_off + r] = X[r].w1;
                a.S[2 * pair_stride + tile_off + r] = X[r].w2;
            }
        }
        return;
    }
    const int64_t mi = m0 + ml;
    if (mi >= a.m) return;
    const int baseA = relA[0][ml];
    uint64_t c_old[SCALED ? R : 1];                   // the C of a scaled product; see accumulate_scaled_kernel
    if constexpr (SCALED) {
#pragma unroll
        for (int r = 0; r < R; ++r) c_old[r] = a.use_beta && n0 + nl + r < a.n ? reinterpret_cast<const uint64_t*>(a.C)[mi + (n0 + nl + r) * a.ldc] : 0;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t nj = n0 + nl + r;
        if (nj >= a.n) continue;
        const int base = baseA + relB[0][nl + r];
        uint64_t* const dst = reinterpret_cast<uint64_t*>(a.C) + mi + nj * a.ldc;
        uint64_t v;
        if constexpr (HW) {
            double d = ldexp(Sd[r], base);
            if (a.add_to_C) d = a.W[mi + nj * a.ldw] + d;
            v = (uint64_t)__double_as_longlong(d);
        } else {
            if constexpr (EMU) v = fp64_scale_pow2_emulated(E[r].value(), base);
            else v = X[r].round_to_fp64(base - a.two_b - EXACT_WINDOW_BITS);
            if (a.add_to_C) v = fp64_add_emulated(reinterpret_cast<const uint64_t*>(a.W)[mi + nj * a.ldw], v);
        }
        if constexpr (SCALED) v = scaled_result<!HW>(a.alpha, v, a.beta, a.use_beta, c_old[r]);
        *dst = v;
    }
}

template <int MODE, bool PINT>
__global__ void __launch_bounds__(256) accumulate_kernel(const AccArgs a) { accumulate_body<MODE, PINT, 4, 4, false>(a); }

// Behind launch_ladder_sums (the question whether there is anything to do takes 0.3 us of the smallest calls)
template <int MODE, bool PINT>
__global__ void __launch_bounds__(256) accumulate_rest_kernel(const AccArgs a) { accumulate_body<MODE, PINT, 4, 4, false, true>(a); }
template <int MODE, bool PINT>
__global__ void __launch_bounds__(256) accumulate_scaled_rest_kernel(const AccArgs a) { accumulate_body<MODE, PINT, 4, 4, true, true>(a); }

// Few elements: a quarter of the work per thread
template <int MODE, bool PINT>
__global__ void __launch_bounds__(256) accumulate_fine_kernel(const AccArgs a) { accumulate_body<MODE, PINT, 1, 8, false>(a); }

// The last block of a scaled product: combined with C here, without a pass of its own over the product and C.  C is read after the last
// run: asked for before the first, it took 12 to 22 registers through the whole sum, which cost the launch all that the other pass
// had taken.  FP8, 12 slices, beta = 1, us, with a pass of its own / C read first / last: emulated 2048^2 107 / 105 / 93, 4096^2 372 / 363 /
// 309, 1537 x 1311 67 / 68 / 61; exact 4096^2 441 / 420 / 378; hardware 4096^2 288 / 200 / 191; 1000 x 777 emulated 41 / 40 / 39.
template <int MODE, bool PINT>
__global__ void __launch_bounds__(256) accumulate_scaled_kernel(const AccArgs a) { accumulate_body<MODE, PINT, 4, 4, true>(a); }
template <int MODE, bool PINT>
__global__ void __launch_bounds__(256) accumulate_scaled_fine_kernel(const AccArgs a) { accumulate_body<MODE, PINT, 1, 8, true>(a); }
// Both behind launch_ladder_sums, where small results have as few positions as anywhere.  Calls with vectors off the ladder, emulated, by the
// coarse forms and by these: 640 x 640 x 600, 9 INT8 slices 77.6 and 62.7 us, 600 x 600 x 1000, 11 FP8 slices in 64 MiB 135.5 and 117.7; with nothing to do
// the four times as many workgroups take 0.5 us of a launch.
template <int MODE, bool PINT>
__global__ void __launch_bounds__(256) accumulate_fine_rest_kernel(const AccArgs a) { accumulate_body<MODE, PINT, 1, 8, false, true>(a); }
template <int MODE, bool PINT>
__global__ void __launch_bounds__(256) accumulate_scaled_fine_rest_kernel(const AccArgs a) { accumulate_body<MODE, PINT, 1, 8, true, true>(a); }

// Verification export: one thread per stored word; grid.y = pair slot of the pass.  Writes the plain column-major
// matrices and, if asked, the number of pairs each slot sums for the element (see launch_export_products).
struct ExportArgs {
    const float* P;
    float* out;
    uint8_t* run_len;
    int64_t m, n;
    int quads_m, quads_n;
    float factor;            // FP32 products: the exact power of two that undoes the FP6 code scaling
    int p_is_int;
    int allow_chain;
    const int32_t* da;
    const int32_t* db;
    int64_t ga, gb;          // groups of 32 vectors per slice in da / db
    const uint8_t* starts;   // measured runs (RunCheck), or null: decided from the deltas
    int tiles_m, tiles_n;    // layout of starts
    PairOrder order;
    Pass pass;
};
__global__ void __launch_bounds__(256) export_products_kernel(const ExportArgs a) {
    const size_t pair_stride = (size_t)a.quads_m * a.quads_n * QUAD_ELEMS;
    const int z = blockIdx.y;
    // the pair of slot z: anti-diagonal g, position pos in it
    int g = a.pass.g_hi, pos = z;
    for (; g > a.pass.g_lo && pos >= diag_len(a.order, g); --g) pos -= diag_len(a.order, g);
    const int len = diag_len(a.order, g);
    const int p = diag_first_p(a.order, g) + pos - 1, q = g - p - 2;      // 0-based slice indices
    for (size_t gi = (size_t)blockIdx.x * 256 + threadIdx.x; gi < pair_stride; gi += (size_t)gridDim.x * 256) {
        const int block = (int)(gi / QUAD_ELEMS), idx = (int)(gi % QUAD_ELEMS);
        const int qn = block / a.quads_m, qm = block - qn * a.quads_m;
        int ml, nl;
        acc_order_to_mn(idx, ml, nl);
        const int64_t mi = (int64_t)qm * QUAD + ml, nj = (int64_t)qn * QUAD + nl;
        if (mi >= a.m || nj >= a.n) continue;
        const int32_t* dA = a.da + mi / LINK_ROWS;
        const int32_t* dB = a.db + nj / LINK_ROWS;
        const size_t tiles = (size_t)a.tiles_m * a.tiles_n;
        const size_t place = ((size_t)(qn >> 1) * a.tiles_m + (qm >> 1)) * 64 + ((qn & 1) * 2 + (qm & 1)) * 16 + (idx >> 10);
        auto starts_at = [&](int j) -> bool {                                   // pair j of the anti-diagonal behind this one
            if (a.starts != nullptr) return a.starts[(size_t)(z + j) * tiles * 64 + place] != 0;
            return starts_run(a.order, a.allow_chain, dA, a.ga, dB, a.gb, pos + j, p + j, q - j);
        };
        int run = 0;
        if (starts_at(0)) {
            run = 1;
            while (pos + run < len && !starts_at(run)) ++run;
        }
        const size_t o = ((size_t)z * a.n + nj) * a.m + mi;
        const uint32_t w = reinterpret_cast<const uint32_t*>(a.P)[(size_t)z * pair_stride + gi];
        uint32_t* const dst = reinterpret_cast<uint32_t*>(a.out) + o;
        if (run == 0) *dst = 0u;                                                // all-zero bits either way
        else if (a.p_is_int) *dst = w;                                          // the INT32 word, bit for bit
        else *dst = __float_as_uint(__uint_as_float(w) * a.factor);             // power of two: exact
        if (a.run_len) a.run_len[o] = (uint8_t)run;
    }
}

__global__ void __launch_bounds__(256) add_emulated_kernel(const uint64_t* a, const uint64_t* b, uint64_t* out, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        out[i] = fp64_add_emulated(a[i], b[i]);
}

// The same as a pass of its own: products without an inner dimension.
template <bool EMU>
__global__ void __launch_bounds__(256) axpby_kernel(uint64_t alpha, uint64_t beta, int use_beta, const uint64_t* __restrict__ W,
                                                    int64_t ldw, uint64_t* C, int64_t ldc, int64_t m, int64_t n) {
    const int64_t total = m * n;
    for (int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (int64_t)gridDim.x * 256) {
        const int64_t i = idx % m, j = idx / m;
        uint64_t* dst = C + i + j * ldc;
        *dst = scaled_result<EMU>(alpha, W[i + j * ldw], beta, use_beta, use_beta ? *dst : 0);
    }
}

__global__ void __launch_bounds__(256) fill_zero_kernel(uint64_t* C, int64_t ldc, int64_t m, int64_t n) {
    const int64_t total = m * n;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256)
        C[(i % m) + (i / m) * ldc] = 0;
}

unsigned grid_for(int64_t work_items) {
    int64_t blocks = (work_items + 255) / 256;
    if (blocks < 1) blocks = 1;
    if (blocks > 65536) blocks = 65536;
    return (unsigned)blocks;
}

}  // namespace

hipError_t launch_accumulate(const Plan& pl, const Operand& A, const Operand& B, const PairOrder& order, const Pass& ps,
                             bool first_pass, bool last_pass, int64_t t, const float* P, uint64_t* S_io,
                             double* C, int64_t ldc, const ScaledResult* scaled, int accum_mode, int sum_rule, bool chained, const uint8_t* starts,
                             const OffLadder& off, hipStream_t st) {
    if (pl.tiles_m == 0 || pl.tiles_n == 0) return hipSuccess;
    AccArgs a;
    a.P = P; a.S = S_io; a.C = C; a.ldc = ldc;
    a.ea = A.exps + (size_t)t * pl.s * A.rows_pad;
    a.eb = B.exps + (size_t)t * pl.s * B.rows_pad;
    a.rows_pad_a = A.rows_pad; a.rows_pad_b = B.rows_pad;
    a.m = pl.m; a.n = pl.n; a.tiles_m = (int)pl.tiles_m; a.tiles_n = (int)pl.tiles_n;
    a.quads_m = (int)pl.quads_m; a.quads_n = (int)pl.quads_n;
    a.two_b = 2 * pl.b;
    a.p_frac = pl.p_frac;
    a.allow_chain = chained ? 1 : 0;
    a.starts = starts;
    a.off = off;
    a.merge = (sum_rule == SUM_RUNS || accum_mode == ACC_EXACT) ? 1 : 0;
    a.da = A.deltas != nullptr ? A.deltas + (size_t)t * (A.rows_pad / LINK_ROWS) * pl.s : nullptr;
    a.db = B.deltas != nullptr ? B.deltas + (size_t)t * (B.rows_pad / LINK_ROWS) * pl.s : nullptr;
    a.order = order; a.pass = ps;
    a.read_S = !first_pass;
    a.write_S = !last_pass;
    a.add_to_C = t > 0;
    a.W = C; a.ldw = ldc;
    a.alpha = a.beta = 0; a.use_beta = 0;
    if (scaled != nullptr) {
        a.C = scaled->C; a.ldc = scaled->ldc;
        memcpy(&a.alpha, &scaled->alpha, 8);
        memcpy(&a.beta, &scaled->beta, 8);
        a.use_beta = scaled->beta != 0.0;
    }
    const int64_t blocks = pl.tiles_m * pl.tiles_n * 64;
    if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
    // With few positions a thread's serial chain (four elements per stored run, a round trip to memory per four runs) is the
    // kernel's length: 361 positions, 21 runs, emulated 28 -> 22 us; 64 positions 18.8 -> 12.7; at 800 the two are equal, and
    // beyond that four times the entry lists and word-wide loads lose (1024 positions 26 -> 37 us).
    const int64_t positions = ((pl.m + 31) / 32) * ((pl.n + 31) / 32);
    const bool fine = positions <= 512;
    // Products asked for before the list of runs is there, k = 256, us: FP8, hardware sum, 4096^2, 9 slices 157 -> 142, 4 slices 89 -> 78;
    // 2048^2 40.5 -> 36; exact 8192^2, 5 slices 637 -> 633; INT8, emulated 8192^2, 5 slices 546 -> 525, exact 706 -> 682.  Not worth it for
    // the emulated sum of FP32 products, which does not wait for its first products and loses the waves that their registers cost
    // (8192^2, 9 slices 728 -> 756, 4096^2 198 -> 204); nor with few positions and no more groups than are asked for at once (1024^2,
    // 4 slices 11.3 -> 11.9; 5 to 13 slices gain, 18.7 -> 17.9 with 9).  Where runs end off the ladder the early products are thrown away.
    a.early = positions > 1024 || (accum_mode == ACC_HW && ps.ngroups > 4);
    const dim3 grid((unsigned)(fine ? 4 * blocks : blocks)), block(256);
    auto launch = [&](auto coarse_kernel, auto fine_kernel, auto rest_kernel, auto fine_rest_kernel) {
        const bool rest = off.counts != nullptr;
        if (fine && rest) hipLaunchKernelGGL(fine_rest_kernel, grid, block, 0, st, a);
        else if (fine) hipLaunchKernelGGL(fine_kernel, grid, block, 0, st, a);
        else if (rest) hipLaunchKernelGGL(rest_kernel, grid, block, 0, st, a);
        else hipLaunchKernelGGL(coarse_kernel, grid, block, 0, st, a);
    };
    auto launch_mode = [&](auto mode, auto pint) {
        constexpr int M = decltype(mode)::value;
        constexpr bool I = decltype(pint)::value;
        if (scaled != nullptr)
            launch(accumulate_scaled_kernel<M, I>, accumulate_scaled_fine_kernel<M, I>, accumulate_scaled_rest_kernel<M, I>, accumulate_scaled_fine_rest_kernel<M, I>);
        else launch(accumulate_kernel<M, I>, accumulate_fine_kernel<M, I>, accumulate_rest_kernel<M, I>, accumulate_fine_rest_kernel<M, I>);
    };
    auto launch_words = [&](auto pint) {
        if (accum_mode == ACC_EXACT) launch_mode(std::integral_constant<int, ACC_EXACT>{}, pint);
        else if (accum_mode == ACC_EMU) launch_mode(std::integral_constant<int, ACC_EMU>{}, pint);
        else launch_mode(std::integral_constant<int, ACC_HW>{}, pint);
    };
    if (pl.p_is_int) launch_words(std::true_type{});
    else launch_words(std::false_type{});
    return hipGetLastError();
}

hipError_t launch_export_products(const Plan& pl, const Operand& A, const Operand& B, const PairOrder& order, const Pass& ps,
                                  bool chained, const uint8_t* starts, int64_t t, const float* P, float* out, uint8_t* run_len_out,
                                  hipStream_t st) {
    if (ps.npairs <= 0 || pl.m == 0 || pl.n == 0) return hipSuccess;
    ExportArgs a;
    a.P = P; a.out = out; a.run_len = run_len_out;
    a.m = pl.m; a.n = pl.n; a.quads_m = (int)pl.quads_m; a.quads_n = (int)pl.quads_n;
    a.factor = ldexpf(1.0f, pl.p_is_int ? 0 : pl.p_frac - 2 * pl.b);
    a.p_is_int = pl.p_is_int;
    a.allow_chain = chained ? 1 : 0;
    a.da = A.deltas + (size_t)t * (A.rows_pad / LINK_ROWS) * pl.s;
    a.db = B.deltas + (size_t)t * (B.rows_pad / LINK_ROWS) * pl.s;
    a.ga = A.rows_pad / LINK_ROWS; a.gb = B.rows_pad / LINK_ROWS;
    a.starts = starts; a.tiles_m = (int)pl.tiles_m; a.tiles_n = (int)pl.tiles_n;
    a.order = order; a.pass = ps;
    dim3 grid(grid_for(pl.quads_m * pl.quads_n * (int64_t)QUAD_ELEMS), (unsigned)ps.npairs);
    hipLaunchKernelGGL(export_products_kernel, grid, dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_add_emulated(const double* a, const double* b, double* out, int64_t n, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(add_emulated_kernel, dim3(grid_for(n)), dim3(256), 0, st, reinterpret_cast<const uint64_t*>(a),
                       reinterpret_cast<const uint64_t*>(b), reinterpret_cast<uint64_t*>(out), n);
    return hipGetLastError();
}

hipError_t launch_axpby(double alpha, double beta, const double* W, int64_t ldw, double* C, int64_t ldc, int64_t m, int64_t n,
                        int accum_mode, hipStream_t st) {
    if (m <= 0 || n <= 0) return hipSuccess;
    uint64_t ab, bb;
    memcpy(&ab, &alpha, 8);
    memcpy(&bb, &beta, 8);
    const int use_beta = beta != 0.0;
    if (accum_mode == 1)
        hipLaunchKernelGGL((axpby_kernel<true>), dim3(grid_for(m * n)), dim3(256), 0, st, ab, bb, use_beta,
                           reinterpret_cast<const uint64_t*>(W), ldw, reinterpret_cast<uint64_t*>(C), ldc, m, n);
    else
        hipLaunchKernelGGL((axpby_kernel<false>), dim3(grid_for(m * n)), dim3(256), 0, st, ab, bb, use_beta,
                           reinterpret_cast<const uint64_t*>(W), ldw, reinterpret_cast<uint64_t*>(C), ldc, m, n);
    return hipGetLastError();
}

hipError_t launch_fill_zero_f64(double* C, int64_t ldc, int64_t m, int64_t n, hipStream_t st) {
    if (m <= 0 || n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_zero_kernel, dim3(grid_for(m * n)), dim3(256), 0, st, reinterpret_cast<uint64_t*>(C), ldc, m, n);
    return hipGetLastError();
}

}  // namespace ozaki
