// The planner: Eq. 1-3, the work memory's carve-up and the route of a call (blocks, groups of pairs, runs, passes).  Host code
// without a call to the runtime, so that host programs can ask which route a call takes.
#pragma once
#include <math.h>
#include <string.h>

#include "../../include/ozaki_dgemm.h"
#include "layout.hpp"

namespace ozaki {

constexpr size_t ALIGN = 256;
constexpr size_t FLAG_BYTES = 256;
constexpr size_t P_BUDGET = (size_t)160 << 30;        // resident pair products: well inside the 288 GB of one GPU
inline size_t align_up(size_t v) { return (v + ALIGN - 1) / ALIGN * ALIGN; }

// Exact window of the matrix unit's accumulator, in units of the product of two slice units: |sum| <= window is exact.
inline int64_t exact_window(int fmt) { return fmt == OZAKI_SLICE_INT8 ? ((int64_t)1 << 31) - 1 : (int64_t)1 << 24; }

// Largest b <= m2 with kb * 4^b <= window (Eq. 1-3 with Type1 = FP64, Type3 = FP32 / INT32); -1 if none.
inline int slice_bits(int64_t kb, int fmt) {
    // significand bits with the hidden one: E4M3 and E2M3 have three fraction bits, E3M2 two; an INT8 byte holds |q| <= 2^6
    const int m2 = fmt == OZAKI_SLICE_FP16 ? 11 : fmt == OZAKI_SLICE_FP6_E3M2 ? 3 : fmt == OZAKI_SLICE_INT8 ? 6 : 4;
    const int64_t window = exact_window(fmt);
    for (int b = m2; b >= 0; --b)
        if (kb <= (window >> (2 * b))) return b;
    return -1;
}

inline bool format_ok(int fmt) { return fmt >= OZAKI_SLICE_FP8_E4M3 && fmt <= OZAKI_SLICE_INT8; }

// The pass that starts at anti-diagonal g_hi: as many whole anti-diagonals as fit into `capacity` products (at
// least one: the carve-up guarantees room for the longest anti-diagonal).
inline Pass next_pass(const PairOrder& o, int g_hi, int capacity) {
    Pass ps{g_hi, g_hi, 0, 0};
    for (int g = g_hi; g >= 2; --g) {
        const int len = diag_len(o, g);
        if (ps.npairs > 0 && ps.npairs + len > capacity) break;
        ps.g_lo = g;
        ps.npairs += len;
        ps.ngroups += diag_groups(o, g);
    }
    return ps;
}

// What a GEMM launch takes per 64-byte stage, in microseconds: a 128 x 128 block alone on its compute unit and one of two that
// share it, a 256 x 256 block.
struct StageTimes {
    double small_alone, small_shared, large;
};
inline StageTimes stage_times(int fmt) {
    if (fmt_is_fp6(fmt)) return {0.20, 0.35, 0.39};
    if (fmt == FMT_FP16) return {0.24, 0.41, 0.61};
    if (fmt == FMT_INT8) return {0.25, 0.45, 0.60};
    return {0.24, 0.44, 0.53};
}

// How the GEMMs run whose products are stored `pairs` at a time (several passes, each a launch of its own, if that is not all of
// them): 256 x 256 or 128 x 128 blocks, and the length of the groups.  Any choice gives the same bits (the accumulation kernel
// merges equal-scale products of an anti-diagonal element by element whatever the grouping).  Long groups store fewer products,
// shorter ones and smaller blocks give a problem of few tiles enough workgroups to keep 256 compute units evenly busy.  The
// estimate of GEMM + accumulation, in microseconds (pass_time), is the least that covers
//   - a workgroup's own stages (stage_times) and, added to the fourth power, the panels that the workgroups in flight fetch
//     beyond the L2s (strip_panels, plain_panels): 20 TB/s while the slices fit the memory-side cache, 17 TB/s beyond it (not
//     what the memory delivers: groups that start at the same slice share a panel);
//   - more workgroups than slots: the even share of all stages, but at least as many rounds of every length as the workgroups
//     of that length or more need, and up to two rounds the last ones behind the shortest of the first; then a sixth of a group
//     for the uneven end (not for 256 x 256 blocks in the plain order, longest first over all XCDs);
//   - filling the load ring and storing, per round; the products stored and read again.
// Measured on 720 random problems of fewer than 256 tiles, all formats, every block size and length, the constants fitted to two
// thirds of them: the choice takes 1.020 of the best one's time on average (1.029 on the other third), 1.27 at worst, on 70 more
// with inner dimensions of 8192 to 65536 1.05 and 1.39; the estimate before it (FP8's times for every format, no panels, group
// lengths of two and more and not all of them) 1.082 and 1.94.  From 256 tiles on long groups of the large blocks are always the choice.
inline double pass_time(const Plan& pl, const StageTimes& us, bool small, int len, const Pass& ps, bool chained) {
    const PairOrder order{pl.s, pl.full, len};
    int count[MAX_SLICES + 1] = {}, longest = 1;                 // groups of each length
    for (int g = ps.g_hi; g >= ps.g_lo; --g) {
        const int diag = diag_len(order, g), most = diag < len ? diag : len;
        count[len] += diag / len;
        if (diag % len != 0) ++count[diag % len];
        if (most > longest) longest = most;
    }
    const int64_t bm = small ? pl.quads_m : pl.tiles_m, bn = small ? pl.quads_n : pl.tiles_n;
    const int64_t blocks = bm * bn, slots = small ? 512 : 256;
    int64_t wgs = 0, line = 0;                                   // line: the longest line of groups on one slot, in pairs
    for (int l = longest; l >= 1; --l) {
        wgs += count[l] * blocks;
        const int64_t bound = (wgs + slots - 1) / slots * l;
        if (bound > line) line = bound;
    }
    if (wgs > slots && wgs <= 2 * slots) {                       // the last ones start where the shortest of the first ones end
        int64_t last = 0;
        for (int l = longest; l >= 1; --l) {
            last += count[l] * blocks;
            if (count[l] == 0 || last <= slots) continue;
            int64_t first = 0;
            int before = longest;
            for (int f = longest; f >= 1 && first < 2 * slots + 1 - last; --f) {
                first += count[f] * blocks;
                if (count[f] != 0) before = f;
            }
            if (l + before > line) line = l + before;
        }
    }
    const WorkOrder work = work_order(ps.npairs, wgs / blocks, longest, small ? 64 : 32, bm, bn, pl.chunks);
    const double fetched = work.unit == 0 ? plain_panels(bm, bn) : strip_panels(bm, bn, work), panels = fetched < 2.0 ? fetched : 2.0;
    const double slices_mb = 1e-6 * pl.s * (double)pl.chunks * pl.row_bytes * (double)(pl.m_pad + pl.n_pad);
    const double fetch = panels * 1e-6 * (small ? QUAD : TILE) * pl.row_bytes * (double)(wgs < slots ? wgs : slots) / (slices_mb < 160.0 ? 20.0 : 17.0);
    const double own = !small ? us.large : wgs <= 256 ? us.small_alone : us.small_shared;
    const double stage = sqrt(sqrt(own * own * own * own + fetch * fetch * fetch * fetch)), fixed = small ? 2.2 : 6.0;
    double pairs = longest;                                      // in line on the slot that ends last
    if (wgs > slots) {
        const double even = (double)ps.npairs * blocks / slots;
        pairs = (even > line ? even : (double)line) + (work.unit == 0 && !small ? 0.0 : 0.17 * longest);
    }
    const double rounds = (double)((wgs + slots - 1) / slots), stored = chained ? (double)(wgs / blocks) : (double)ps.npairs;
    return pairs * pl.chunks * stage + rounds * fixed + stored * (0.015 * blocks * (small ? 0.25 : 1.0) + 0.18 + 0.014 * (double)(pl.quads_m * pl.quads_n));
}

inline void choose_gemm(Plan& pl, int pairs, bool chained, bool measured_runs) {
    const int most = measured_runs || pl.run_limit > pl.s ? pl.s : pl.run_limit;
    pl.small_tiles = 0;
    pl.group_len = most;
    const int64_t tiles = pl.tiles_m * pl.tiles_n;
    if (tiles == 0 || tiles >= 256) return;
    const StageTimes us = stage_times(pl.fmt);
    double best = 1e300;
    for (int len = most; len >= 1; --len)
        for (int small = 0; small < 2; ++small) {
            const PairOrder order{pl.s, pl.full, len};
            double t = 0.0;
            for (int g_hi = order_top_diag(order); g_hi >= 2 && t < best;) {
                const Pass ps = next_pass(order, g_hi, pairs);
                t += pass_time(pl, us, small != 0, len, ps, chained);
                g_hi = ps.g_lo - 1;
            }
            if (t < best) {
                best = t;
                pl.small_tiles = small;
                pl.group_len = len;
            }
        }
}

// Builds the plan; returns 0 or a status / negative argument index in the numbering of ozaki_dgemm.
inline int make_plan(int64_t m, int64_t n, int64_t k, int fmt, int s, int64_t k_block, bool full, Plan& pl) {
    if (m < 0) return -1;
    if (n < 0) return -2;
    if (k < 0) return -3;
    if (!format_ok(fmt)) return -10;
    if (s < 0) return -11;
    if (k_block < 0) return -12;
    memset(&pl, 0, sizeof(pl));
    pl.m = m; pl.n = n; pl.k = k; pl.fmt = fmt;
    pl.epc = fmt == OZAKI_SLICE_FP16 ? CHUNK_BYTES / 2 : CHUNK_BYTES;
    pl.row_bytes = fmt_is_fp6(fmt) ? CHUNK_BYTES_FP6 : CHUNK_BYTES;
    pl.kb = (k_block == 0 || k_block > k) ? k : k_block;
    if (pl.kb < 1) pl.kb = 1;
    pl.b = slice_bits(pl.kb, fmt);
    if (pl.b < 0) return OZAKI_STATUS_INFEASIBLE;
    pl.rho = 53 - pl.b;
    pl.s = s == 0 ? (61 + pl.b) / (pl.b + 1) : s;
    if (pl.s > MAX_SLICES) return OZAKI_STATUS_SLICE_COUNT;
    pl.T = k == 0 ? 0 : (k + pl.kb - 1) / pl.kb;
    pl.p_frac = 2 * pl.b - (fmt == OZAKI_SLICE_FP6_E2M3 ? 2 : 0);
    pl.p_is_int = fmt == OZAKI_SLICE_INT8 ? 1 : 0;
    if (pl.p_is_int) pl.p_frac = 0;               // the stored words are the integers themselves
    pl.chunks = (pl.kb + pl.epc - 1) / pl.epc;
    pl.full = full ? 1 : 0;
    pl.npairs = full ? pl.s * pl.s : pl.s * (pl.s + 1) / 2;
    const int64_t rl = exact_window(fmt) / (pl.kb << (2 * pl.b));
    pl.pair_bound = (int)(pl.kb << (2 * pl.b));
    pl.run_limit = rl < 1 ? 1 : rl > MAX_SLICES ? MAX_SLICES : (int)rl;
    pl.tiles_m = (m + TILE - 1) / TILE;
    pl.tiles_n = (n + TILE - 1) / TILE;
    pl.quads_m = (m + QUAD - 1) / QUAD;
    pl.quads_n = (n + QUAD - 1) / QUAD;
    pl.m_pad = pl.tiles_m * TILE;
    pl.n_pad = pl.tiles_n * TILE;
    return 0;
}

// The memory a call may use
struct WorkMem {
    uint8_t* ptr;
    size_t bytes;
};

struct Carve {
    int* flags;
    double* At;
    Operand A, B;
    double* W;            // m x n product buffer of the scaled call (null otherwise)
    uint64_t* S;
    float* P;
    int chunk_pairs;
};

inline size_t slices_bytes(const Plan& pl, int64_t rows_pad) { return align_up((size_t)pl.T * pl.s * pl.chunks * rows_pad * pl.row_bytes); }
inline size_t exps_bytes(const Plan& pl, int64_t rows_pad) { return align_up((size_t)pl.T * pl.s * rows_pad * sizeof(int32_t)); }
inline size_t deltas_bytes(const Plan& pl, int64_t rows_pad) { return align_up((size_t)pl.T * (rows_pad / LINK_ROWS) * pl.s * sizeof(int32_t)); }
// Blocks beyond MAX_K_BLOCK_IN_REGISTERS: 12 bytes per (padded) element of the operands, part of the documented sizes.  No
// kernel needs them any more.
inline size_t long_block_reserve(const Plan& pl) {
    if (pl.kb <= MAX_K_BLOCK_IN_REGISTERS) return 0;
    return align_up((size_t)(pl.m + pl.n) * pl.T * pl.chunks * pl.epc * 12);
}
inline size_t fixed_bytes(const Plan& pl) {
    return FLAG_BYTES + align_up((size_t)pl.m * pl.k * sizeof(double)) + long_block_reserve(pl) + slices_bytes(pl, pl.m_pad) +
           slices_bytes(pl, pl.n_pad) + exps_bytes(pl, pl.m_pad) + exps_bytes(pl, pl.n_pad) + deltas_bytes(pl, pl.m_pad) +
           deltas_bytes(pl, pl.n_pad);
}
// The documented sizes count a product with whole 256 x 256 tiles, and the running block sum between passes with the three
// words of the exact mode whatever the mode; carve() packs closer (stored_bytes, sum_plane_bytes), so that more products of a
// small workspace stay resident and fewer passes are needed.
inline size_t pair_bytes(const Plan& pl) { return (size_t)pl.m_pad * pl.n_pad * sizeof(float); }
inline size_t stored_bytes(const Plan& pl) { return (size_t)pl.quads_m * pl.quads_n * QUAD_ELEMS * sizeof(float); }
inline size_t sum_plane_bytes(const Plan& pl) { return 2 * stored_bytes(pl); }
inline size_t sum_bytes(const Plan& pl) { return (size_t)pl.m_pad * pl.n_pad * sizeof(uint64_t) * SUM_WORDS_MAX; }

inline size_t recommended_bytes(const Plan& pl) {
    const size_t all = (size_t)pl.npairs * pair_bytes(pl);
    if (all <= P_BUDGET) return fixed_bytes(pl) + all;
    size_t fit = P_BUDGET / pair_bytes(pl);
    if (fit < (size_t)pl.s) fit = pl.s;
    return fixed_bytes(pl) + sum_bytes(pl) + fit * pair_bytes(pl);
}
// The pair list is processed in passes that end at anti-diagonal boundaries (a run of equal-scale products
// never spans two passes), so the smallest workspace holds the longest anti-diagonal: s products.
inline size_t minimum_bytes(const Plan& pl) {
    if (pl.npairs == 1) return fixed_bytes(pl) + pair_bytes(pl);
    return fixed_bytes(pl) + sum_bytes(pl) + (size_t)pl.s * pair_bytes(pl);
}

inline size_t product_bytes(const Plan& pl) { return align_up((size_t)pl.m * pl.n * sizeof(double)); }

// Places every buffer in the work memory; returns false if it does not fit.
// sum_words: 64-bit words per element of a running block sum in the call's mode.
inline bool carve(const Plan& pl, Carve& c, bool want_product, int sum_words, WorkMem wm) {
    uint8_t* const ws = wm.ptr;
    const size_t ws_bytes = wm.bytes;
    if (!ws) return false;
    size_t off = 0;
    c.flags = reinterpret_cast<int*>(ws);
    off += FLAG_BYTES;
    c.At = reinterpret_cast<double*>(ws + off);
    off += align_up((size_t)pl.m * pl.k * sizeof(double));
    off += long_block_reserve(pl);
    c.A.rows = pl.m; c.A.rows_pad = pl.m_pad;
    c.B.rows = pl.n; c.B.rows_pad = pl.n_pad;
    c.A.slices = ws + off; off += slices_bytes(pl, pl.m_pad);
    c.B.slices = ws + off; off += slices_bytes(pl, pl.n_pad);
    c.A.exps = reinterpret_cast<int32_t*>(ws + off); off += exps_bytes(pl, pl.m_pad);
    c.B.exps = reinterpret_cast<int32_t*>(ws + off); off += exps_bytes(pl, pl.n_pad);
    c.A.deltas = reinterpret_cast<int32_t*>(ws + off); off += deltas_bytes(pl, pl.m_pad);
    c.B.deltas = reinterpret_cast<int32_t*>(ws + off); off += deltas_bytes(pl, pl.n_pad);
    c.A.l1 = c.B.l1 = c.A.bounds = c.B.bounds = nullptr;
    c.A.off_ladder = c.B.off_ladder = nullptr;
    c.W = nullptr;
    if (want_product) { c.W = reinterpret_cast<double*>(ws + off); off += product_bytes(pl); }
    if (off > ws_bytes) return false;
    const size_t rest = ws_bytes - off, pb = pair_bytes(pl), stored = stored_bytes(pl);
    if (pb == 0) { c.S = nullptr; c.P = nullptr; c.chunk_pairs = pl.npairs; return true; }
    const bool all_documented = rest >= (size_t)pl.npairs * pb;
    if (!all_documented && rest < sum_bytes(pl) + (size_t)pl.s * pb) return false;      // below the documented minimum
    if (rest >= (size_t)pl.npairs * stored) {
        c.S = nullptr;
        c.P = reinterpret_cast<float*>(ws + off);
        c.chunk_pairs = pl.npairs;
        return true;
    }
    c.S = reinterpret_cast<uint64_t*>(ws + off);
    off += (size_t)sum_words * sum_plane_bytes(pl);
    c.P = reinterpret_cast<float*>(ws + off);
    const size_t fit = (ws_bytes - off) / stored;                                           // at least the documented s
    c.chunk_pairs = fit > (size_t)pl.npairs ? pl.npairs : (int)fit;
    return true;
}

// Measured runs (RunCheck) where run_limit cuts anti-diagonals, and the buffers they need.  These live in memory whose own
// contents are not needed at the time: the transposed A is dead once the operands are sliced (bounds, starts), the products
// are not there yet while they are (l1).  Without room the runs keep to run_limit.  Anti-diagonals cut in two at most are
// left so: looking at the accumulators then costs as much as the fewer products give (8192^3, 16 FP8 slices, run_limit 8:
// GEMMs 46.6 -> 47.0 ms, accumulation 1.97 -> 1.78 ms).  Where every pair was stored on its own: 8192^3 FP16 in blocks of 1024
// 57.8 -> 36.6 ms, in blocks of 4096 43.5 -> 37.9 ms, 2048^3 in blocks of 1024 1.36 -> 0.88 ms.
inline RunCheck place_run_check(const Plan& pl, Carve& c) {
    RunCheck none{nullptr, nullptr, nullptr};
    if (pl.p_is_int || 2 * pl.run_limit >= pl.s) return none;
    const bool from_slices = pl.run_limit == 1;            // a pair may fill the window: bounds from the slicing kernel
    if (from_slices && (pl.fmt != OZAKI_SLICE_FP16 || pl.kb > MAX_K_BLOCK_IN_REGISTERS)) return none;
    uint8_t* const at = reinterpret_cast<uint8_t*>(c.At);
    const size_t room = align_up((size_t)pl.m * pl.k * sizeof(double));
    const size_t ba = deltas_bytes(pl, pl.m_pad), bb = deltas_bytes(pl, pl.n_pad);
    const size_t starts = (size_t)c.chunk_pairs * pl.tiles_m * pl.tiles_n * 64;
    if ((from_slices ? ba + bb : 0) + starts > room) return none;
    if (!from_slices) return RunCheck{at, nullptr, nullptr};
    const size_t la = exps_bytes(pl, pl.m_pad), lb = exps_bytes(pl, pl.n_pad);
    if (la + lb > (size_t)c.chunk_pairs * stored_bytes(pl)) return none;
    c.A.l1 = reinterpret_cast<int32_t*>(c.P);
    c.B.l1 = reinterpret_cast<int32_t*>(reinterpret_cast<uint8_t*>(c.P) + la);
    c.A.bounds = reinterpret_cast<int32_t*>(at);
    c.B.bounds = reinterpret_cast<int32_t*>(at + ba);
    return RunCheck{at + ba + bb, c.A.bounds, c.B.bounds};
}

// How a call runs in its work memory.
struct Route {
    Plan pl;              // with the blocks and groups of the call's launches
    Carve c;              // c.A.deltas / c.B.deltas are null where the kernels form the links themselves
    RunCheck check;
    OffLadder off;        // counts null: launch_ladder_sums has no part in the call
    int32_t* deltas_a;    // where the deltas would go
    int32_t* deltas_b;
};
// chained: the matrix unit may sum pairs.  as_dgemm: as the DGEMM does, beyond the window's worst case where measured runs apply, in the
// groups that take the least time; otherwise in the longest groups of the worst case.  False if the memory does not hold it.
inline bool place_call(const Plan& plan, bool want_product, int sum_words, bool chained, bool as_dgemm, WorkMem wm, Route& r) {
    r.pl = plan;
    r.off = NO_LADDER;
    r.check = RunCheck{nullptr, nullptr, nullptr};
    if (!carve(plan, r.c, want_product, sum_words, wm)) return false;
    if (chained && as_dgemm) r.check = place_run_check(r.pl, r.c);
    choose_gemm(r.pl, r.c.chunk_pairs, chained, r.check.starts != nullptr);               // of one pass: each is a launch of its own
    if (chained && !as_dgemm) r.pl.group_len = r.pl.run_limit < r.pl.s ? r.pl.run_limit : r.pl.s;
    if (r.pl.group_len <= r.pl.run_limit) {                                               // no group passes the worst case: nothing to measure
        r.check = RunCheck{nullptr, nullptr, nullptr};
        r.c.A.l1 = r.c.B.l1 = r.c.A.bounds = r.c.B.bounds = nullptr;
    }
    r.deltas_a = r.c.A.deltas;
    r.deltas_b = r.c.B.deltas;
    if (r.pl.small_tiles && r.c.A.l1 == nullptr) r.c.A.deltas = r.c.B.deltas = nullptr;      // a launch less
    return true;
}

// Does the call start with launch_ladder_sums?  (The GEMM kernels and the accumulation come behind it.)
// Tiles: a workgroup does all pairs of its tile, so with few tiles most compute units have no part in the work, which the GEMM kernels deal
// out by groups of pairs as well.  Time of a call by those over its time by this one, 520, 1500 and 4500 inner indices:
//   tiles       64                 100                144                160                256                576                2209
//   FP8, 13     0.90 0.80 0.66     1.14 1.10 0.96     1.28 1.18 1.02     1.52 1.40 1.36     1.44 1.30 1.26     1.32 1.23 1.13     1.53 1.40 1.27
//   FP8, 7      1.02 0.80 0.72     1.03 1.07 0.90     1.16 1.16 0.95     1.28 1.26 1.11     1.40 1.26 1.16     1.25 1.29 1.06     1.80 1.31 1.18
//   INT8, 9     0.97 0.83 0.78     1.10 1.11 1.05     1.15 1.34 1.09     1.43 1.48 1.37     1.52 1.32 1.23     1.26 1.22 1.17     1.45 1.27 1.20
//   FP6, 13     1.18 0.96 0.81     1.06 1.26 1.09     1.39 1.36 1.16     1.59 1.53 1.51     1.51 1.36 1.31     1.39 1.34 1.21     1.65 1.49 1.36
// 94 tiles, 96 x 3000: 1.00 to 1.17, FP8 with 7 slices and 4500 inner indices 0.93.  Hence 90 tiles, for FP8 and more than 32 stages 160.
// Few slices gain least where these have tiles for every compute unit and the blocks are long: 2048 x 8192 x 6000, hardware sum, 6 to 9
// slices FP8 1.00, 1.05, 1.09, 1.05, FP6 1.10, 1.15, 1.18, 1.02, INT8 1.05, 1.14, 1.16 (6 to 8).
// Blocks: of short vectors some are off the ladder as a rule, and the call then takes the other route and the launch for nothing (3 to 5 us).  The share of vectors off it, entries (u - 1/2) exp(phi z), 13 FP8 slices (which reach the end of the mantissas): phi = 0.5,
// k = 256 2.3 %, k = 512 0.1 %, k = 1024 none of 2048; phi = 1, k = 64 5 %, k = 128 0.15 %, from k = 256 on none; phi = 2 0.05 to 0.2 % up
// to k = 1024; 9 INT8 slices none from k = 64 on (from 257 here: shorter blocks have a slicing kernel of their own).
inline bool ladder_pays(const Plan& pl) {
    const int64_t shortest = pl.k - (pl.T - 1) * pl.kb;          // the last block
    return ladder_possible(pl) && shortest >= (pl.fmt == FMT_INT8 ? 257 : 512) &&
           ladder_blocks(pl.m) * ladder_blocks(pl.n) >= (pl.fmt == FMT_FP8 && pl.chunks > 32 ? 160 : 90);
}
constexpr int OFF_LADDER_MOST = 64;
inline void place_ladder(Route& r) {
    if (!ladder_pays(r.pl)) return;
    // What the slicing kernels say of the vectors lies at the end of the products' memory, which the first launch that reads it leaves alone: with
    // all pairs the sums between its halves take 24 bytes per element of a 64 x 64 tile from the front.
    const size_t products = (size_t)r.c.chunk_pairs * stored_bytes(r.pl), marks = (size_t)r.pl.T * (size_t)(r.pl.m_pad + r.pl.n_pad);
    const size_t halves = r.pl.full ? (size_t)ladder_blocks(r.pl.m) * (size_t)ladder_blocks(r.pl.n) * LADDER_TILE * LADDER_TILE * sizeof(uint64_t) * SUM_WORDS_MAX : 0;
    if (halves + marks > products) return;
    r.c.A.off_ladder = reinterpret_cast<uint8_t*>(r.c.P) + (products - marks);
    r.c.B.off_ladder = r.c.A.off_ladder + (size_t)r.pl.T * (size_t)r.pl.m_pad;
    r.off.counts = r.c.flags + OFF_LADDER_FLAG;
    r.off.marks = r.c.A.off_ladder;
    // Some vectors off it: where the call is long against one more launch (3 to 5 us where there are none).  Their list lies in the
    // transposed A's memory, which is dead once the operands are sliced; the runs of such a call have no use for it (place_run_check:
    // run_limit covers an anti-diagonal).
    if ((r.pl.fmt == FMT_FP8 || r.pl.fmt == FMT_INT8) && r.pl.s <= OFF_LADDER_MAX_SLICES && !r.pl.full && r.pl.T == 1 && r.check.starts == nullptr &&
        ladder_blocks(r.pl.m) * ladder_blocks(r.pl.n) >= 1024 && 2 * OFF_LADDER_MOST * sizeof(int) <= (size_t)r.pl.m * r.pl.k * sizeof(double)) {
        r.off.limit = OFF_LADDER_MOST;
        r.off.list = reinterpret_cast<int*>(r.c.At);
    }
    // A launch in front of the pass that counts and lists the vectors off the ladder would also fill the deltas, which only the kernels behind the
    // pass use.  Up to MOST_MARKS the pass looks at the vectors itself, and fills the deltas if there are too many, so that the launch for nothing
    // takes that one's place (a slice of 256 vectors per workgroup: 1 us more than without; all slices of them by one workgroup 5).  us, with a vector
    // off the ladder in brackets, by the GEMM kernels and the accumulation alone, with a launch in front of the pass, now: 1000 x 777 x 1301, 12 FP8 slices,
    // scaled, emulated (174, 179) 110, 103.4 (172.7); 1024^3, 121 pairs (147, 153) 110, 103.2 (147.9); 2048 x 2048 x 1024, 13 FP8 slices (368, 300)
    // 263, 258 (296); 600 x 600 x 1000, 11 FP8 slices (71.4, 78.4) 64.2, 59.7 (74.7); 640 x 640 x 600, 13 FP6 slices (61.0, 68.7) 53.4, 48.2 (64.2);
    // 9 INT8 slices, emulated (55.5, 62.4) 50.0, 46.4 (59.3).  In the last three the other kernels form the links themselves if they have to
    // (place_call); without the deltas they take 0.5 us more.
    if (marks <= MOST_MARKS) {
        r.off.uncounted = r.off.marks;
        r.off.mark_bytes = (int)marks;
        r.off.first_bytes = (int)(r.pl.T * r.pl.m_pad);
    }
    r.c.A.deltas = r.deltas_a;
    r.c.B.deltas = r.deltas_b;
}

inline PairOrder order_of(const Plan& pl) { return PairOrder{pl.s, pl.full, pl.group_len}; }

}  // namespace ozaki
