// Plan, internal data layouts and kernel-launcher prototypes shared by the libozaki translation units.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace ozaki {

constexpr int MAX_SLICES = 32;
constexpr int MAX_PAIRS = MAX_SLICES * MAX_SLICES;      // all s*s pairs in the full mode
constexpr int64_t MAX_K_BLOCK_IN_REGISTERS = 16384;     // longer blocks: split_stream_kernel, exponents first

// ---- tiling of the slice-pair GEMM: one workgroup computes one TILE x TILE block of one pair product ------
constexpr int TILE = 256;
constexpr int CHUNK_BYTES = 64;           // bytes of the inner dimension per row staged per pipeline step (FP8, FP16)
constexpr int CHUNK_BYTES_FP6 = 48;       // the same 64 inner indices as 6-bit codes
constexpr int QUAD = 128;                 // edge of a block of the product storage: a workgroup's share in the small-problem GEMM
                                          // kernel, a wave's in the other one
constexpr int QUAD_ELEMS = QUAD * QUAD;

// slice formats (values of ozaki_slice_format)
constexpr int FMT_FP8 = 0, FMT_FP16 = 1, FMT_FP6 = 2, FMT_FP6_E3M2 = 3, FMT_INT8 = 4;     // FMT_FP6 is E2M3
__host__ __device__ constexpr bool fmt_is_fp6(int fmt) { return fmt == FMT_FP6 || fmt == FMT_FP6_E3M2; }

// how the slice-pair products of a block are summed (values of the accum_mode / sum_rule arguments)
constexpr int ACC_HW = 0, ACC_EMU = 1, ACC_EXACT = 2;
constexpr int SUM_RUNS = 0, SUM_PLAIN = 1;

// "exact" accumulation: the block sum of an element is a 192-bit two's-complement integer in units of
// 2^(cA_1 + cB_1 - 2b - EXACT_WINDOW_BITS); at most 1024 terms of at most 2^36 units * 2^EXACT_WINDOW_BITS each.
constexpr int EXACT_WINDOW_BITS = 144;
constexpr int SUM_WORDS_MAX = 3;          // 64-bit words of a running block sum kept in work memory between passes

// ---- slice storage ---------------------------------------------------------------------------------------
// One slice matrix (block t, slice p) of an operand is stored as [chunk kc][vector r][CHUNK_BYTES]:
// the 256 vectors a workgroup stages for one pipeline step are 16 KiB of contiguous memory.  The number
// of vectors is padded to a multiple of TILE and every block to whole chunks; the padding holds zero
// codes, which contribute exact zeros to every product.
//
// FP6: a chunk holds 64 inner indices of every vector as 6-bit codes.  The matrix unit wants the 32 codes of a
// vector's k-group g (inner indices 32g .. 32g+31 of the chunk) as one 192-bit little-endian string (code i at
// bits 6i .. 6i+5).  A chunk stores the first 16 bytes and the last 8 bytes of these strings in four planes,
//     [g = 0: rows_pad x 16 B][g = 1: rows_pad x 16 B][g = 0: rows_pad x 8 B][g = 1: rows_pad x 8 B]
// (rows_pad x 48 bytes in all), so that the part of a plane that belongs to a 256-vector tile is contiguous and a
// wave's fragment reads from the staged copy are contiguous, bank-conflict-free 128- and 64-bit accesses.
struct Operand {
    int64_t rows;         // real vectors: m for A (its rows), n for B (its columns)
    int64_t rows_pad;     // multiple of TILE
    uint8_t* slices;      // [T][s][chunks][rows_pad][row_bytes]
    int32_t* exps;        // [T][s][rows_pad]   exponent c of Eq. 4 (0 for padding vectors)
    int32_t* l1;          // [T][s][rows_pad]   sum |q| of the slice (null: not wanted)
    int32_t* bounds;      // [T][s][rows_pad/LINK_ROWS]  2^b times the largest l1 of the group (see RunCheck)
    uint8_t* off_ladder;  // [T][rows_pad]   is the vector off the ladder (OffLadder)? (null: not wanted)
    int32_t* deltas;      // [T][s][rows_pad/LINK_ROWS]  per slice p and group of 32 vectors (one matrix-unit tile edge):
                          //                        c_p - c_(p+1) if that difference is the same for all real vectors of
                          //                        the group, else DELTA_IRREGULAR (always for the last slice); null:
                          //                        the kernels form them from the exponents (128 x 128 blocks only)
};

constexpr int LINK_ROWS = 32;             // granularity of the equal-scale decision: one 32 x 32 matrix-unit tile

constexpr int DELTA_IRREGULAR = -2147483647 - 1;

struct Plan {
    int64_t m, n, k;
    int fmt;              // FMT_FP8, FMT_FP16, FMT_FP6, FMT_FP6_E3M2
    int epc;              // inner indices per chunk: 64 (FP8, FP6) or 32 (FP16)
    int row_bytes;        // bytes of one vector in one chunk: 64 (FP8, FP16) or 48 (FP6)
    int p_frac;           // a stored pair product is an integer multiple of 2^-p_frac: 2b, for FP6 (whose codes hold
                          // twice the slice value) 2b - 2; the true product is the stored one times 2^(p_frac - 2b)
    int s;                // slices per operand
    int b;                // magnitude bits of a slice entry (53 - rho)
    int rho;
    int64_t kb;           // block length (elements)
    int64_t T;            // number of blocks
    int64_t chunks;       // chunks per block
    int full;             // 1: all s*s pairs, 0: the pairs with p + q <= s + 1
    int npairs;           // s(s+1)/2 or s*s
    int run_limit;        // floor(window / (kb * 4^b)): equal-scale pair products that may be summed exactly in the
                          // matrix unit's accumulators (window 2^24 for FP32, 2^31 - 1 for INT32)
    int pair_bound;       // kb * 4^b: no partial sum of a pair product is larger (FP32 formats: at most 2^24)
    int group_len;        // pairs per group of the GEMM kernel (choose_gemm): at most run_limit, with measured runs at most s
    int64_t tiles_m, tiles_n;
    int64_t quads_m, quads_n;    // 128 x 128 blocks that hold elements of C
    int64_t m_pad, n_pad;
    int small_tiles;      // 1: the GEMMs run in 128 x 128 blocks (launch_pair_gemm_small)
    int p_is_int;         // 1: the stored products are INT32 words (INT8 slices), 0: FP32
};

// The slice pairs (p, q), 1-based, and their accumulation order: anti-diagonals g = p + q from the least
// significant (largest g) down to g = 2, p ascending inside one.  Triangle mode uses the pairs with p + q <= s + 1,
// full mode all s * s.  Consecutive pairs of an anti-diagonal with equal scale are summed exactly before the FP64
// addition; the matrix unit can do that for as many pairs as surely fit the exact window (Plan::run_limit), or, with measured
// runs (RunCheck), for as many as its accumulators leave room for.  Every anti-diagonal is cut into groups of at most group_len
// consecutive pairs (Plan::group_len), the unit of work of the GEMM kernel; pairs are numbered z = 0, 1, ... in this order.
// Everything below is a closed form of (s, full, group_len), evaluated on the host and in the kernels.
struct PairOrder {
    int s;
    int full;
    int group_len;        // pairs per group
};
__host__ __device__ inline int order_top_diag(const PairOrder& o) { return o.full ? 2 * o.s : o.s + 1; }
__host__ __device__ inline int diag_first_p(const PairOrder& o, int g) { return g - o.s > 1 ? g - o.s : 1; }
__host__ __device__ inline int diag_len(const PairOrder& o, int g) {
    const int hi = g - 1 < o.s ? g - 1 : o.s;
    return hi - diag_first_p(o, g) + 1;
}
__host__ __device__ inline int diag_groups(const PairOrder& o, int g) { return (diag_len(o, g) + o.group_len - 1) / o.group_len; }
// First position of group i of an anti-diagonal of `len` pairs: whole groups, then the rest.  (Cuts of equal length would even
// out the workgroups, but groups of neighbouring anti-diagonals that start at the same slice read the same panels side by
// side: 1024 x 1024 x 8192 takes 0.51 ms with these cuts, 0.56 ms with equal ones.)
__host__ __device__ inline int group_first(const PairOrder& o, int len, int i) { return i * o.group_len < len ? i * o.group_len : len; }
__host__ __device__ inline int order_num_groups(const PairOrder& o) {
    int n = 0;
    for (int g = order_top_diag(o); g >= 2; --g) n += diag_groups(o, g);
    return n;
}
__host__ __device__ inline int order_num_pairs(const PairOrder& o) { return o.full ? o.s * o.s : o.s * (o.s + 1) / 2; }

// A pass of the accumulation: the anti-diagonals g_hi, g_hi - 1, ..., g_lo; its pair products occupy the slots
// 0 .. npairs-1 of the product buffer in pair order.
struct Pass {
    int g_hi, g_lo;
    int npairs, ngroups;
};

// The gi-th group of a pass, in accumulation order: slices (p0 + j, q0 - j), j < len (1-based), first product slot `slot`.
struct Group {
    int p0, q0, len, slot;
};
__host__ __device__ inline Group pass_group(const PairOrder& o, const Pass& ps, int gi) {
    int slot = 0;
    for (int g = ps.g_hi; g >= ps.g_lo; --g) {
        const int len = diag_len(o, g), ng = diag_groups(o, g);
        if (gi < ng) {
            const int pos = group_first(o, len, gi);
            Group r;
            r.p0 = diag_first_p(o, g) + pos;
            r.q0 = g - r.p0;
            r.len = group_first(o, len, gi + 1) - pos;
            r.slot = slot + pos;
            return r;
        }
        gi -= ng;
        slot += len;
    }
    return Group{1, 1, 0, 0};
}

inline int longest_group(const PairOrder& o, const Pass& ps) {
    int longest = 1;
    for (int g = ps.g_hi; g >= ps.g_lo; --g) longest = diag_len(o, g) > longest ? diag_len(o, g) : longest;
    return longest < o.group_len ? longest : o.group_len;
}

// The groups of a pass in the order in which workgroups take them, longest first (a long group that starts last would be
// the launch's tail), packed for the kernel arguments: p0 | q0 << 6 | len << 12 | slot << 18.  A pass of more groups than fit
// goes in accumulation order.
constexpr int MAX_LISTED_GROUPS = 512;
struct GroupList {
    int listed;
    uint32_t entry[MAX_LISTED_GROUPS];
};
inline void list_groups(const PairOrder& o, const Pass& ps, GroupList& list) {
    list.listed = ps.ngroups <= MAX_LISTED_GROUPS ? ps.ngroups : 0;
    if (list.listed == 0) return;
    int place[MAX_SLICES + 2] = {};                             // place[len]: groups longer than len, then their next place
    for (int pass = 0; pass < 2; ++pass) {
        int slot = 0;
        for (int g = ps.g_hi; g >= ps.g_lo; --g) {
            const int len = diag_len(o, g), ng = diag_groups(o, g);
            for (int i = 0; i < ng; ++i) {
                const int pos = group_first(o, len, i), glen = group_first(o, len, i + 1) - pos, p0 = diag_first_p(o, g) + pos;
                if (pass == 0) ++place[glen - 1];
                else list.entry[place[glen]++] = (uint32_t)p0 | (uint32_t)(g - p0) << 6 | (uint32_t)glen << 12 | (uint32_t)(slot + pos) << 18;
            }
            slot += len;
        }
        if (pass == 0)
            for (int len = MAX_SLICES; len >= 0; --len) place[len] += place[len + 1];
    }
}
__host__ __device__ inline Group listed_group(const GroupList& list, const PairOrder& o, const Pass& ps, int gi) {
    if (list.listed == 0) return pass_group(o, ps, gi);
    const uint32_t e = list.entry[gi];
    return Group{(int)(e & 63), (int)((e >> 6) & 63), (int)((e >> 12) & 63), (int)(e >> 18)};
}

// Which work item (group gi, block (bm, bn) of blocks_m x blocks_n) workgroup b of `total` takes.  Workgroups are handed to
// the eight XCDs, each with an L2 of its own, round-robin by their index.  unit == 0: plain order, block rows fastest.
// Otherwise the `unit` workgroups an XCD runs at the same time get consecutive items, and consecutive items of a group walk
// strips of `height` block rows column by column, so that they form a compact patch that shares its slice panels.
// Groups come longest first, so every second round deals the units in reverse order to keep the XCDs even.
struct WorkOrder {
    int unit, height;
};
struct WorkItem {
    unsigned gi, bm, bn;
};
__host__ __device__ inline WorkItem work_item(unsigned b, unsigned total, const WorkOrder& o, unsigned blocks_m, unsigned blocks_n) {
    unsigned w = b, strip_rows = blocks_m;
    if (o.unit != 0) {
        const unsigned unit = o.unit, round = 8 * unit, full = total / round * round, xcd = b & 7;
        strip_rows = o.height;
        if (b < full) {
            const unsigned r = b / round;
            w = r * round + ((r & 1) ? 7 - xcd : xcd) * unit + ((b - r * round) >> 3);
        } else {                                   // the last, incomplete round: one contiguous piece per XCD
            const unsigned rest = total - full, each = rest >> 3, more = rest & 7;
            w = full + xcd * each + (xcd < more ? xcd : more) + ((b - full) >> 3);
        }
    }
    WorkItem it;
    it.gi = w / (blocks_m * blocks_n);
    const unsigned r = w - it.gi * (blocks_m * blocks_n), strip = r / (strip_rows * blocks_n), in = r - strip * strip_rows * blocks_n;
    const unsigned left = blocks_m - strip_rows * strip, height = left < strip_rows ? left : strip_rows;
    it.bn = in / height;
    it.bm = strip_rows * strip + (in - it.bn * height);
    return it;
}
// Slice panels that an XCD fetches per workgroup and stage, of the two that a workgroup reads: rows + columns over the area of what it
// has in flight of one group, in strips and in the plain order (every eighth block, block rows fastest).
inline double strip_panels(int64_t blocks_m, int64_t blocks_n, const WorkOrder& o) {
    if (blocks_m * blocks_n < o.unit) return (double)(blocks_m + blocks_n) / (double)(blocks_m * blocks_n);
    const double rows = (double)(blocks_m < o.height ? blocks_m : o.height), cols = o.unit / rows < (double)blocks_n ? o.unit / rows : (double)blocks_n;
    return (rows + cols) / (rows * cols);
}
inline double plain_panels(int64_t blocks_m, int64_t blocks_n) {
    const int64_t blocks = blocks_m * blocks_n, stride = blocks_m % 8 == 0 ? 8 : blocks_m % 4 == 0 ? 4 : blocks_m % 2 == 0 ? 2 : 1;
    const double in_flight = blocks > 8 ? blocks / 8.0 : 1.0, rows = (double)(blocks_m / stride), cols = (double)blocks_n;
    return ((rows < in_flight ? rows : in_flight) + (cols < in_flight ? cols : in_flight)) / in_flight;
}

// The order for a launch of `groups` groups of `pairs` pairs together, none longer than `len`, over blocks_m x blocks_n blocks; `per_xcd`
// workgroups run at a time on an XCD.  Strips save traffic between the L2s and the memory behind them, a panel per workgroup
// and stage or more: 5 x 23 blocks of 128 x 128, 24 stages, 121 products in 2415 workgroups (4.7 rounds) 576 -> 290 us;
// 14 x 6 blocks of 256 x 256, 112 FP16 stages, 4.6 rounds 1.58 -> 1.31 ms; 4096^3 FP8 4.08 -> 4.01 ms.  In 700 random problems they
// take 0.7 to 0.9 of the plain time with 128 x 128 blocks and 0.92 to 0.97 with 256 x 256 blocks at two to four rounds of
// workgroups, 0.63 to 0.8 and 0.75 to 0.9 from eight rounds on, whatever the length of the groups.  What they cost: a unit's
// XCD waits for its longest group while others are idle, 1.0 to 1.2 of the plain time with few rounds.  Hence
//   - 128 x 128 blocks from 2 rounds on, 256 x 256 blocks from 2.5; where a group has a multiple of eight blocks, so that the plain
//     order keeps a block on its XCD from group to group, from 2.5 and 4 (8 x 8 blocks of 256 x 256, 32 FP16 stages, 3.25
//     rounds: strips 6 % slower);
//   - results of one row or column of blocks, where strips too fetch a panel and more: from 3 (128 x 128 blocks, pairs of 32 stages and more: 2), a multiple of eight blocks 6 (1.1 to 1.25
//     of the plain time before; 56 x 1 blocks of 128 x 128, groups of nine pairs, 2.6 rounds: 178 us plain, 226 in strips);
//   - pairs of fewer than eight stages, which are bound by their stores, from 4 (0.95 to 1.05 below);
//   - 128 x 128 blocks, pairs of 16 stages and more, where strips fetch less than a panel and the plain order 1.5 or more: from 0.6
//     in groups of equal length (0.85 of the longest on average), from 0.75 at 0.7 (0.76 to 0.89 of the plain time on average, 1.1
//     to 1.25 below; 5 x 5 blocks, groups of two to five: 72 -> 47, 62 -> 51, 60 -> 49, 54 -> 50 us; 12 x 3 blocks, 64 FP16
//     stages, groups of two: 679 -> 510); from 0.35 to 0.5, where no two workgroups share a compute unit and so none waits, if it
//     is 0.6 against 1.9 (passes of 21 to 24 pairs in groups of three, 5 x 5 blocks: the call 120 -> 116 us).
// The plain order also stays where it already gives every XCD a compact patch by itself: at 32 block rows, four of them per XCD
// (128 x 128 blocks: 1.0 to 1.1 of the plain time there; 16384^2 FP16: 2.5 % longer).  40, 44, 48, 52 and 56 block rows of 256:
// strips, equal to the plain order or up to 6 % faster.
inline WorkOrder work_order(int64_t pairs, int64_t groups, int len, int per_xcd, int64_t blocks_m, int64_t blocks_n, int64_t chunks) {
    const WorkOrder plain{0, 0}, strips{per_xcd, blocks_m > 8 ? 4 : 8};
    const int64_t blocks = blocks_m * blocks_n;
    const double rounds = (double)(groups * blocks) / (8 * per_xcd);
    const bool small = per_xcd == 64, keeps_xcd = blocks % 8 == 0;
    const double in_strips = strip_panels(blocks_m, blocks_n, strips), in_plain = plain_panels(blocks_m, blocks_n);
    double least = small ? (keeps_xcd ? 2.5 : 2.0) : (keeps_xcd ? 4.0 : 2.5);
    if (in_strips >= 1.0) least = keeps_xcd ? 6.0 : small && chunks >= 32 ? 2.0 : 3.0;
    if (chunks < 8 && least < 4.0) least = 4.0;
    if (small && !keeps_xcd && chunks >= 16 && 10 * pairs >= 7 * len * groups) {
        if (in_strips < 1.0 && in_plain >= 1.5) least = 20 * pairs >= 17 * len * groups ? 0.6 : 0.75;
        if (in_strips < 0.6 && in_plain >= 1.9 && rounds <= 0.5) least = 0.35;
    }
    return blocks_m % 32 == 0 || rounds < least ? plain : strips;
}

// Runs longer than run_limit pairs ("measured" runs).  run_limit assumes that every product of slice entries is as large as it
// can be; real slices stay far below that.  With measured runs a group may hold a whole anti-diagonal, and when a pair is
// complete the GEMM kernel looks at the accumulators of each 32 x 32 tile: the next pair may be added on top if their largest
// magnitude plus a bound on every partial sum of the next pair stays inside the exact window, so all sums are exact as
// before.  The bound is kb 4^b where run_limit >= 2; where a single pair may fill the window (FP16 with the widest slices) it
// is 2^b sum |q| over a vector, from the slicing, the smaller of the two operands' maxima over the tile's 32 vectors.  Which
// pairs start a run is then data; the GEMM kernel writes it down for the accumulation, a byte per product slot and tile:
// starts[slot][tile_n][tile_m][wave of the 256 x 256 kernel * 16 + sub], 1 if the slot holds a run's sum.
struct RunCheck {
    uint8_t* starts;          // null: runs of at most run_limit pairs, decided from the deltas alone
    const int32_t* bound_a;   // [T][s][rows_pad_a / LINK_ROWS] bounds of the slices' pair products, or null: pair_bound for all
    const int32_t* bound_b;
};

// True if, for every element of a 32 x 32 tile, pair (p+1, q-1) carries the same scale factor 2^(cA + cB) as pair
// (p, q) (0-based slice indices): then the two products can be summed in the accumulator of the matrix unit
// (that the sum stays inside the exact window is another matter: groups of at most run_limit pairs, or RunCheck).  a: the delta
// of slice p of the tile's 32 rows of A, b: the delta of slice q - 1 of its 32 columns of B.
__host__ __device__ inline bool deltas_link(int a, int b) { return a != DELTA_IRREGULAR && a == b; }
// dA / dB: Operand::deltas of the block, advanced to the tile's group of rows of A / columns of B; ga / gb: groups per
// slice (rows_pad / LINK_ROWS) of the two operands.
__host__ __device__ inline bool pair_linked(const int32_t* dA, int64_t ga, const int32_t* dB, int64_t gb, int p, int q) {
    return deltas_link(dA[p * ga], dB[(q - 1) * gb]);
}

// ---- pair-product storage ("accumulator order") ------------------------------------------------------------
// The FP32 product of one pair is stored in blocks of 128 x 128, [block_n][block_m][QUAD_ELEMS], only the blocks that hold
// elements of C, and inside a block in the order the matrix unit leaves it in the registers of a wave:
//     float index = ((sub*4 + a)*64 + lane)*4 + r
//     sub = ti*4 + tj (ti, tj in 0..3)
//     column of C (n) = block_n*128 + ti*32 + a*8 + (lane/32)*4 + r
//     row    of C (m) = block_m*128 + tj*32 + lane%32
// Every wave-wide store / load of this buffer is one contiguous kilobyte.
__host__ __device__ inline void acc_order_to_mn(int idx, int& m_in_block, int& n_in_block) {
    int r = idx & 3, lane = (idx >> 2) & 63, a = (idx >> 8) & 3, sub = idx >> 10;
    n_in_block = (sub >> 2) * 32 + a * 8 + (lane >> 5) * 4 + r;
    m_in_block = (sub & 3) * 32 + (lane & 31);
}

// ---- tiles done by ladder_sums.hpp ----------------------------------------------------------------------------
constexpr int LADDER_TILE = 64;
// Slice counts that have a kernel (each takes time to build): what the formats need for full accuracy and less, of all pairs the counts of
// the paper's Table 2 and their neighbours.  Accumulators for 16 anti-diagonals would fit, but not with what else a wave keeps (FP8, INT8; with
// FP6's smaller fragments it was not tried).
constexpr int ladder_min_slices(int fmt, bool full) { return fmt == FMT_FP6_E3M2 ? (full ? 13 : 10) : fmt == FMT_INT8 ? (full ? 7 : 6) : full ? 10 : 6; }
constexpr int ladder_max_slices(int fmt, bool full) { return fmt == FMT_FP6_E3M2 ? 15 : fmt == FMT_INT8 ? (full ? 9 : 11) : full ? 12 : 14; }
inline int64_t ladder_blocks(int64_t extent) { return (extent + LADDER_TILE - 1) / LADDER_TILE; }
// Magnitude bits of a slice entry where the window holds an anti-diagonal of four pairs or more: the format's own limit
constexpr int ladder_bits(int fmt) { return fmt == FMT_INT8 ? 6 : fmt == FMT_FP6_E3M2 ? 3 : 4; }
// The launch's limits: accumulators for the anti-diagonals, 32-bit offsets in an operand's slices, anti-diagonals whose sums are
// exact in the accumulators whatever the data.
inline bool ladder_possible(const Plan& pl) {
    const int64_t rows = pl.m_pad > pl.n_pad ? pl.m_pad : pl.n_pad, most = (int64_t)1 << 31;
    return pl.fmt != FMT_FP16 && pl.s >= ladder_min_slices(pl.fmt, pl.full != 0) && pl.s <= ladder_max_slices(pl.fmt, pl.full != 0) && pl.run_limit >= pl.s && pl.b == ladder_bits(pl.fmt) && pl.m > 0 && pl.n > 0 &&
           pl.chunks < most / (rows * pl.row_bytes * pl.s) && ladder_blocks(pl.m) * ladder_blocks(pl.n) < most;
}
// The exact mode keeps an element in 128 bits there: all terms fit, and none lies below the unit at which the 192 bits end.
constexpr bool ladder_exact_fits(int fmt, int s, bool full) {
    const int above = (ladder_bits(fmt) + 1) * (full ? 2 * s - 2 : s - 1);
    return 31 + above + 1 <= 127 && above <= EXACT_WINDOW_BITS;
}
// How many vectors of the two operands are off the ladder: those with a slice, other than zeros, whose exponent lies more than b + 1 below
// that of the slice before.  (The slicing kernels say so of every vector, Operand::off_ladder, and clear the counts; the exponents alone do not
// tell a slice that is left without a remainder, whose exponent is 0, from others.)  Up to `limit` of each: ladder_sums.hpp does the call's
// products but for theirs, which off_ladder.hpp does; beyond that the GEMM kernels and the accumulation, which come behind.
struct OffLadder {
    int* counts;             // null: no such distinction, the latter do all
    int limit;
    int* list;               // limit > 0: these vectors, up to `limit` of A, up to `limit` of B, in no order
    const uint8_t* marks;    // Operand::off_ladder of A, behind it that of B
    const uint8_t* uncounted;      // null, or the marks: there is no launch_deltas; the first launch of ladder_sums.hpp counts the vectors and lists
    int mark_bytes, first_bytes;   // them, or fills the deltas.  Then: all marks, and A's
};
constexpr OffLadder NO_LADDER{nullptr, 0, nullptr, nullptr, nullptr, 0, 0};
// Up to so many vectors and blocks every wave of that launch looks at all of them (128 bytes per lane, a round trip to memory as the counts
// are); a multiple of 4096, below 2^16.
constexpr int MOST_MARKS = 8192;
#if defined(__HIPCC__)
__device__ __forceinline__ bool on_ladder(const OffLadder& o) { return o.counts != nullptr && o.counts[0] <= o.limit && o.counts[1] <= o.limit; }
#endif
constexpr int OFF_LADDER_FLAG = 4;        // the counts' place in the flag words

// ---- launchers (each enqueues on `st` and returns the launch status) ----------------------------------------
hipError_t launch_transpose(const double* A, int64_t lda, int64_t m, int64_t k, double* At, hipStream_t st);

// Vector r of an operand starts at X + r*ldv and has k entries, contiguous ones in the second operand, `es0` apart in the
// first (1 for blocks beyond MAX_K_BLOCK_IN_REGISTERS).  Writes the internal layout of
// up to two operands in one launch (a null Operand, or one without vectors, is skipped).  Blocks longer than
// MAX_K_BLOCK_IN_REGISTERS take two launches: the exponents of all slices first, then the slices.  Clears OffLadder's counts (blocks beyond
// 256 elements).
hipError_t launch_split(const double* X0, int64_t ldv0, int64_t es0, const Operand* op0, const double* X1, int64_t ldv1, const Operand* op1,
                        const Plan& pl, int* flags, hipStream_t st);

// Slices until every remainder is zero (paragraph before Eq. 4): atomicMax of the per-vector count into flags[1]
// (which the caller has cleared); MAX_SLICES + 1 means that MAX_SLICES slices do not exhaust some vector.
hipError_t launch_count_slices(const double* X, int64_t ldv, const Plan& pl, int64_t rows, int* flags, hipStream_t st);

// Internal layout -> plain vector-major codes (verification export).
hipError_t launch_export_slices(const Plan& pl, const Operand& op, void* out, hipStream_t st);

// Fills Operand::deltas from Operand::exps (deltas.hpp), for up to two operands in one launch, and counts and lists the vectors off the ladder if
// off.counts is not null.
hipError_t launch_deltas(const Plan& pl, const Operand* op0, const Operand* op1, const OffLadder& off, hipStream_t st);

// Products of the pairs of pass `ps` of block t into P ([ps.npairs][quads_n][quads_m][QUAD_ELEMS] floats).  With
// allow_chain, consecutive pairs of a group that are linked for a tile (pair_linked) form a run whose exact sum is
// stored in the slot of the run's first pair; the slots of the other pairs of the run are left untouched.
hipError_t launch_pair_gemm(const Plan& pl, const Operand& A, const Operand& B, const PairOrder& order, const Pass& ps,
                            bool allow_chain, const RunCheck& check, const OffLadder& off, int64_t t, float* P, hipStream_t st);
// The same in 128 x 128 blocks (Plan::small_tiles; called by launch_pair_gemm).  Blocks without real elements are left out.
hipError_t launch_pair_gemm_small(const Plan& pl, const Operand& A, const Operand& B, const PairOrder& order, const Pass& ps,
                                  bool allow_chain, const RunCheck& check, const OffLadder& off, int64_t t, float* P, hipStream_t st);

// C = alpha * (A B) + beta * C, formed where the last block's sum is added (one rounding per operation, no fused multiply-add;
// beta == 0: C is not read).
struct ScaledResult {
    double alpha, beta;
    double* C;
    int64_t ldc;
};

// Accumulate the pairs of pass `ps` of block t.  S_io: running block sum in accumulator order (read unless the
// pass is the block's first, written unless it is the last): one 64-bit word per element (FP64 bits), three in the
// exact mode, word w of element e at S_io[w * quads * QUAD_ELEMS + e].  On the last pass the block sum is rescaled by
// the first-slice exponents and stored to C (t == 0) or added to C (t > 0); with `scaled` (last pass of the last block) that sum
// is the product of a scaled call, combined into scaled->C, and C is only read.  `chained`: the products were written
// with allow_chain; starts: RunCheck::starts of that launch.  sum_rule SUM_PLAIN: every product is added on its own.
hipError_t launch_accumulate(const Plan& pl, const Operand& A, const Operand& B, const PairOrder& order, const Pass& ps,
                             bool first_pass, bool last_pass, int64_t t, const float* P, uint64_t* S_io,
                             double* C, int64_t ldc, const ScaledResult* scaled, int accum_mode, int sum_rule, bool chained,
                             const uint8_t* starts, const OffLadder& off, hipStream_t st);

// The products of the vectors off the ladder if those are few (off_ladder.hpp); C, scaled as in launch_accumulate.  FP8 and INT8, the pairs
// of the triangle, one block.
constexpr int OFF_LADDER_MIN_SLICES = 6, OFF_LADDER_MAX_SLICES = 13;
hipError_t launch_off_ladder(const Plan& pl, const Operand& A, const Operand& B, const OffLadder& off, double* C, int64_t ldc,
                             const ScaledResult* scaled, int accum_mode, hipStream_t st);

// Products and sums of block t if the vectors are on the ladder, all but those of the list (ladder_sums.hpp).  S: with all pairs, work memory for the sum of the less significant half, SUM_WORDS_MAX words per
// element of the tiles.  The other arguments as in launch_accumulate.
hipError_t launch_ladder_sums(const Plan& pl, const Operand& A, const Operand& B, int64_t t, const OffLadder& off, uint64_t* S, double* C,
                              int64_t ldc, const ScaledResult* scaled, int accum_mode, hipStream_t st);

// P in accumulator order -> [nz][n][m] column-major matrices (verification export): FP32 values of Eq. 10-11, or INT32
// integers for INT8 slices.  run_len_out (may be null): for every element and pair slot of the pass, how many pairs'
// products the slot holds summed (1 without chaining; 0: the pair's product is part of an earlier slot's sum, and
// `out` gets 0 there).  chained, starts: as in launch_accumulate; without starts the operands' deltas are needed.
hipError_t launch_export_products(const Plan& pl, const Operand& A, const Operand& B, const PairOrder& order, const Pass& ps,
                                  bool chained, const uint8_t* starts, int64_t t, const float* P, float* out, uint8_t* run_len_out,
                                  hipStream_t st);

// C = alpha * W + beta * C element by element (one rounding per operation, no fused multiply-add; beta == 0: C is not
// read), W and C column-major m x n.
hipError_t launch_axpby(double alpha, double beta, const double* W, int64_t ldw, double* C, int64_t ldc, int64_t m, int64_t n,
                        int accum_mode, hipStream_t st);

hipError_t launch_add_emulated(const double* a, const double* b, double* out, int64_t n, hipStream_t st);
hipError_t launch_fill_zero_f64(double* C, int64_t ldc, int64_t m, int64_t n, hipStream_t st);

}  // namespace ozaki
