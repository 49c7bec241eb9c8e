// Slice-pair GEMMs for problems with too few 256 x 256 tiles to fill the chip (see pair_gemm_body.hpp for the method).
//
// A workgroup of four waves computes a 128 x 128 block of the product for one group of pairs, each wave 64 x 64 (2 x 2
// MFMA tiles, 64 accumulator registers per lane).  Against the 256 x 256 kernel this costs twice the L2 -> LDS bytes per
// flop, but a problem has up to four times the workgroups, two of them share a compute unit (64 KiB of LDS each), a
// stage takes a quarter of the time, and rows and columns beyond the matrix are padded to 128 instead of 256.  Products
// are stored in the same layout: a 128 x 128 block is what one wave of the 256 x 256 kernel owns.
//
// The pipeline is the one of pair_gemm_body.hpp: direct-to-LDS loads through a ring of NSTAGE stages, fragments read one
// k-step ahead.  Two waves load the B slices (the matrix unit's "row" operand), two the A slices.
#pragma once
#include <math.h>

#include <type_traits>

#include "layout.hpp"

namespace ozaki {

struct SmallGemmArgs {
    const uint8_t* sa;       // A slices of the block: [s][chunks][rows_pad_a][row bytes]
    const uint8_t* sb;       // B slices of the block
    float* P;                // [nz][quads_n][quads_m][QUAD_ELEMS]
    int64_t rows_pad_a, rows_pad_b;
    int chunks;
    int tiles_m, tiles_n;    // 256 x 256 tiles: the layout of the run starts
    int quads_m, quads_n;    // 128 x 128 blocks that hold real elements
    int allow_chain;
    WorkOrder work;
    const int32_t* da;       // A deltas of the block: [s][rows_pad_a / 32]; null: formed here from the exponents
    const int32_t* db;       // B deltas of the block: [s][rows_pad_b / 32]
    const int32_t* ea;       // exponents of the block: [s][rows_pad_a]
    const int32_t* eb;       // [s][rows_pad_b]
    int64_t m, n;
    PairOrder order;
    Pass pass;
    GroupList groups;
    uint8_t* starts;         // measured runs (RunCheck): where runs start, or null
    const int32_t* ba;       // bounds of the block, as the deltas; null: pair_bound for every pair
    const int32_t* bb;
    int pair_bound;
    int sure;                // pairs of a group whose sum is inside the window whatever the data
    float unit;              // 2^-p_frac, the unit of the stored sums
    OffLadder off;           // is there anything to do?
};

// (a translation unit of their own: the two forms of the kernel)
hipError_t launch_pair_gemm_small_behind(const SmallGemmArgs& a, int fmt, const dim3& grid, hipStream_t st);

namespace {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));

#define OZAKI_GPTR(p) ((const __attribute__((address_space(1))) void*)(p))
#define OZAKI_LPTR(p) ((__attribute__((address_space(3))) void*)(p))

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

// BEHIND: behind launch_ladder_sums (the question whether there is anything to do takes 0.3 us of the smallest calls)
template <int FMT, bool BEHIND>
__global__ void __launch_bounds__(256, 2) pair_gemm_small_kernel(const SmallGemmArgs a) {
    if (BEHIND && on_ladder(a.off)) return;
    constexpr bool FP16 = FMT == FMT_FP16;
    constexpr bool INT8 = FMT == FMT_INT8;
    constexpr bool HALF = FP16 || INT8;               // 16-byte fragments, two k-steps per 64-byte stage
    constexpr bool FP6 = fmt_is_fp6(FMT);
    constexpr int FP6_CODE = FMT == FMT_FP6_E3M2 ? 3 : 2;
    constexpr int BK = FP6 ? CHUNK_BYTES_FP6 : CHUNK_BYTES;
    constexpr int ROWS = 128;
    constexpr int OPERAND_BYTES = ROWS * BK;
    constexpr int STAGE_BYTES = 2 * OPERAND_BYTES;
    constexpr int LPW = OPERAND_BYTES / 1024 / 2;     // direct-to-LDS loads per wave and stage: two waves per operand
    constexpr int NSTAGE = FP6 ? 5 : 4;               // 60 resp. 64 KiB: two workgroups per compute unit
    constexpr int KS = HALF ? 2 : 1;
    __shared__ __attribute__((aligned(16))) uint8_t lds[NSTAGE * STAGE_BYTES];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave >> 1, wm = wave & 1;          // the wave's 64 x 64 part of the block

    const WorkItem item = work_item(blockIdx.x, gridDim.x, a.work, a.quads_m, a.quads_n);
    const int qn = item.bn, qm = item.bm;
    const Group grp = listed_group(a.groups, a.order, a.pass, item.gi);
    const int glen = grp.len, p0 = grp.p0 - 1, q0 = grp.q0 - 1;       // 0-based slice indices from here on
    const int chunks = a.chunks;

    // Run continuation per 32 x 32 tile, as in pair_gemm_body.hpp; the wave's two row groups and two column groups are eight
    // contiguous bytes each per slice, read through the scalar cache.
    typedef int v2s __attribute__((ext_vector_type(2)));
    typedef const __attribute__((address_space(4))) v2s* delta2_ptr;
    const int64_t groups_a = a.rows_pad_a / LINK_ROWS, groups_b = a.rows_pad_b / LINK_ROWS;
    const int32_t* const dA = a.da + (qm * 4 + wm * 2);
    const int32_t* const dB = a.db + (qn * 4 + wn * 2);
    uint64_t links[2] = {0, 0};                        // without deltas: four bits per pair, formed below
    auto continue_mask = [&](int jp) -> unsigned {
        if (!a.allow_chain) return 0u;
        if (a.da == nullptr) return (unsigned)(links[jp >> 4] >> (4 * (jp & 15))) & 0xFu;
        const v2s dav = *(delta2_ptr)(dA + (size_t)(p0 + jp) * groups_a);
        const v2s dbv = *(delta2_ptr)(dB + (size_t)(q0 - jp - 1) * groups_b);
        unsigned cont = 0;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                cont |= deltas_link(__builtin_amdgcn_readfirstlane(dav[j]), __builtin_amdgcn_readfirstlane(dbv[i])) ? (1u << (i * 2 + j)) : 0u;
        return cont;
    };

    // Measured runs, as in pair_gemm_body.hpp
    auto drop_full_tiles = [&](unsigned cont, const v2s& bav, const v2s& bbv, const auto& acc) -> unsigned {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                if ((cont >> (i * 2 + j)) & 1u) {
                    const int next = bav[j] < bbv[i] ? bav[j] : bbv[i];
                    const float room = (float)((1 << 24) - next) * a.unit;
                    float most = 0.0f;
#pragma unroll
                    for (int r = 0; r < 16; ++r) most = fmaxf(most, fabsf((float)acc[i][j][r]));
                    if (__ballot(!(most <= room)) != 0ull) cont &= ~(1u << (i * 2 + j));
                }
        return cont;
    };
    auto write_starts = [&](int jp, unsigned first) {
        if (lane < 4)
            a.starts[((size_t)((grp.slot + jp) * a.tiles_n + (qn >> 1)) * a.tiles_m + (qm >> 1)) * 64 + ((qn & 1) * 2 + (qm & 1)) * 16 +
                     (wn * 2 + (lane >> 1)) * 4 + wm * 2 + (lane & 1)] = (uint8_t)((first >> lane) & 1u);
    };

    // Loader: waves 0 and 1 fetch the X (B slice) half of a stage, waves 2 and 3 the Y (A slice) half, LPW kilobytes each.
    // FP8 / FP16 / INT8: a kilobyte is 16 rows, swizzled on the global side.  FP6: kilobytes 0, 1 are the 16-byte plane of
    // k-group 0 (64 vectors each), 2, 3 that of k-group 1, 4 and 5 the two 8-byte planes (128 vectors each).
    const bool is_x = wave < 2;
    const int half = wave & 1;
    const int64_t rows_pad = is_x ? a.rows_pad_b : a.rows_pad_a;
    const size_t cs = (size_t)rows_pad * BK;                          // chunk stride
    const size_t first_row = (size_t)(is_x ? qn : qm) * ROWS;
    const uint8_t* ptr = (is_x ? a.sb : a.sa) + (size_t)(is_x ? q0 : p0) * chunks * cs;
    size_t piece[LPW];
    if constexpr (FP6) {
#pragma unroll
        for (int i = 0; i < LPW; ++i) {
            const int kb = half * LPW + i;
            piece[i] = kb < 4 ? ((size_t)(kb >> 1) * rows_pad + first_row + (kb & 1) * 64) * 16
                              : (size_t)rows_pad * 32 + ((size_t)(kb - 4) * rows_pad + first_row) * 8;
            piece[i] += (size_t)lane * 16;
        }
    } else {
        const unsigned lrow = lane >> 2, lpc = lane & 3;
        const unsigned goff = lrow * BK + ((lpc ^ ((lrow >> 2) & 3)) << 4);
#pragma unroll
        for (int i = 0; i < LPW; ++i) piece[i] = first_row * BK + (size_t)(half * LPW + i) * 1024 + goff;
    }
    // A slices of a group lie back to back; B slices are walked backwards (see pair_gemm_body.hpp)
    const int64_t d_wrap = is_x ? -(int64_t)((size_t)(2 * chunks - 1) * cs) : (int64_t)cs;
    const int lds_at = (is_x ? 0 : OPERAND_BYTES) + half * LPW * 1024;
    const int total = glen * chunks;
    int issued = 0, issue_kc = 0;
    auto issue_next = [&](int buf) {
        uint8_t* lb = lds + buf * STAGE_BYTES + lds_at;
#pragma unroll
        for (int i = 0; i < LPW; ++i)
            __builtin_amdgcn_global_load_lds(OZAKI_GPTR(ptr + piece[i]), OZAKI_LPTR(lb + i * 1024), 16, 0, 0);
        // after the last stage the pointer stays put: the (unused) reloads keep the outstanding-load count uniform
        const bool adv = issued + 1 < total;
        const bool wrap = issue_kc + 1 == chunks;
        ptr += adv ? (wrap ? d_wrap : (int64_t)cs) : 0;
        issued += adv ? 1 : 0;
        issue_kc = adv ? (wrap ? 0 : issue_kc + 1) : issue_kc;
    };

    const int frow = lane & 31, fg = lane >> 5;
    const int fsw = (frow >> 2) & 3;
    const int xrow = wn * 64 + frow, yrow = wm * 64 + frow;
    const int xbase = xrow * BK, ybase = OPERAND_BYTES + yrow * BK;

    typedef typename std::conditional<INT8, v16i, v16f>::type acc_t;
    typedef typename std::conditional<INT8, v4i, v4f>::type acc4_t;
    acc_t acc[2][2];
    auto zero_tile = [&](acc_t& t) {
#pragma unroll
        for (int r = 0; r < 16; ++r) t[r] = 0;
    };
    // 32 x 32 tile (i, j) of the wave is sub-tile (wn * 2 + i) * 4 + (wm * 2 + j) of the block
    const unsigned lane_bytes = (unsigned)lane * 16u;
    const size_t block_at = ((size_t)qn * a.quads_m + qm) * QUAD_ELEMS;
    const size_t pair_stride = (size_t)a.quads_n * a.quads_m * QUAD_ELEMS;
    auto store_tile = [&](int slot, int i, int j, const acc_t& t) {
        char* base = reinterpret_cast<char*>(a.P + (size_t)slot * pair_stride + block_at + (size_t)((wn * 2 + i) * 4 + wm * 2 + j) * 1024);
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
            acc4_t v = {t[4 * g4], t[4 * g4 + 1], t[4 * g4 + 2], t[4 * g4 + 3]};
            *reinterpret_cast<acc4_t*>(base + g4 * 1024 + lane_bytes) = v;
        }
    };

    typedef typename std::conditional<FP16, v8h, typename std::conditional<INT8, v4i, v8i>::type>::type frag_t;
    frag_t xf[2][2], yf[2][2];
    auto read_frags = [&](int stage, int ks, int fb) {
        const uint8_t* base = lds + ((unsigned)stage % NSTAGE) * STAGE_BYTES;
        if constexpr (HALF) {
            const int c0 = ((2 * ks + fg) ^ fsw) << 4;
#pragma unroll
            for (int i = 0; i < 2; ++i) xf[fb][i] = *reinterpret_cast<const frag_t*>(base + xbase + i * 32 * BK + c0);
#pragma unroll
            for (int j = 0; j < 2; ++j) yf[fb][j] = *reinterpret_cast<const frag_t*>(base + ybase + j * 32 * BK + c0);
        } else if constexpr (FP6) {
            // per operand: [k-group][128 vectors][16 B], then [k-group][128 vectors][8 B]
            const uint8_t* x16 = base + fg * 2048 + xrow * 16;
            const uint8_t* y16 = base + OPERAND_BYTES + fg * 2048 + yrow * 16;
            const unsigned x8 = (unsigned)(uintptr_t)OZAKI_LPTR(base + 4096 + fg * 1024 + xrow * 8);
            const unsigned y8 = (unsigned)(uintptr_t)OZAKI_LPTR(base + OPERAND_BYTES + 4096 + fg * 1024 + yrow * 8);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                unsigned ax = x8 + i * 32 * 8, ay = y8 + i * 32 * 8;      // an address register of its own each, see pair_gemm_body.hpp
                asm volatile("" : "+v"(ax), "+v"(ay));
                const v4i xlo = *reinterpret_cast<const v4i*>(x16 + i * 32 * 16);
                const v2i xhi = *reinterpret_cast<const __attribute__((address_space(3))) v2i*>((uintptr_t)ax);
                xf[fb][i] = __builtin_shufflevector(xlo, __builtin_shufflevector(xhi, xhi, 0, 1, -1, -1), 0, 1, 2, 3, 4, 5, -1, -1);
                const v4i ylo = *reinterpret_cast<const v4i*>(y16 + i * 32 * 16);
                const v2i yhi = *reinterpret_cast<const __attribute__((address_space(3))) v2i*>((uintptr_t)ay);
                yf[fb][i] = __builtin_shufflevector(ylo, __builtin_shufflevector(yhi, yhi, 0, 1, -1, -1), 0, 1, 2, 3, 4, 5, -1, -1);
            }
        } else {
            const int c0 = ((2 * fg) ^ fsw) << 4, c1 = ((2 * fg + 1) ^ fsw) << 4;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const v4i lo = *reinterpret_cast<const v4i*>(base + xbase + i * 32 * BK + c0);
                const v4i hi = *reinterpret_cast<const v4i*>(base + xbase + i * 32 * BK + c1);
                xf[fb][i] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const v4i lo = *reinterpret_cast<const v4i*>(base + ybase + j * 32 * BK + c0);
                const v4i hi = *reinterpret_cast<const v4i*>(base + ybase + j * 32 * BK + c1);
                yf[fb][j] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            }
        }
    };
    auto mfmas = [&](int fb) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) {
                const int j = (i & 1) ? 1 - jj : jj;
                if constexpr (FP16) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(xf[fb][i], yf[fb][j], acc[i][j], 0, 0, 0);
                else if constexpr (INT8) acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(xf[fb][i], yf[fb][j], acc[i][j], 0, 0, 0);
                else if constexpr (FP6) acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(xf[fb][i], yf[fb][j], acc[i][j], FP6_CODE, FP6_CODE, 0, 0, 0, 0);
                else acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(xf[fb][i], yf[fb][j], acc[i][j], 0, 0, 0, 0, 0, 0);
            }
    };

#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) zero_tile(acc[i][j]);
#pragma unroll
    for (int st = 0; st < NSTAGE; ++st) issue_next(st);
    if (a.da == nullptr && a.allow_chain) {
        // Lane l has row l of the wave's 64 rows of A and column l of its 64 columns of B; the first stages are on their way
        // meanwhile.  A launch of its own for the deltas (5 us) would be a tenth of the smallest calls.
        const int64_t row = (int64_t)qm * QUAD + wm * 64 + lane, col = (int64_t)qn * QUAD + wn * 64 + lane;
        const int32_t* const ea = a.ea + (size_t)p0 * a.rows_pad_a + row;
        const int32_t* const eb = a.eb + (size_t)q0 * a.rows_pad_b + col;
        int cA = ea[0], cB = eb[0];
        auto same = [&](int d, int ref, bool pad, bool (&ok)[2]) {
            const uint64_t mask = __ballot(pad || d == ref);
            ok[0] = (uint32_t)mask == 0xFFFFFFFFu;
            ok[1] = (uint32_t)(mask >> 32) == 0xFFFFFFFFu;
        };
        for (int j0 = 0; j0 + 1 < glen; j0 += 8) {
            int nA[8], nB[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int j = j0 + u + 1 < glen ? j0 + u + 1 : glen - 1;
                nA[u] = ea[(size_t)j * a.rows_pad_a];
                nB[u] = *(eb - (size_t)j * a.rows_pad_b);
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int jp = j0 + u;
                if (jp + 1 >= glen) break;
                const int d_a = cA - nA[u], d_b = nB[u] - cB;          // deltas of slices p0 + jp and q0 - jp - 1
                cA = nA[u];
                cB = nB[u];
                const int a0 = __builtin_amdgcn_readlane(d_a, 0), a1 = __builtin_amdgcn_readlane(d_a, 32);
                const int b0 = __builtin_amdgcn_readlane(d_b, 0), b1 = __builtin_amdgcn_readlane(d_b, 32);
                bool okA[2], okB[2];
                same(d_a, lane < 32 ? a0 : a1, row >= a.m, okA);
                same(d_b, lane < 32 ? b0 : b1, col >= a.n, okB);
                const unsigned bits = (okA[0] && okB[0] && a0 == b0 ? 1u : 0u) | (okA[1] && okB[0] && a1 == b0 ? 2u : 0u) |
                                      (okA[0] && okB[1] && a0 == b1 ? 4u : 0u) | (okA[1] && okB[1] && a1 == b1 ? 8u : 0u);
                if (jp < 16) links[0] |= (uint64_t)bits << (4 * jp);
                else links[1] |= (uint64_t)bits << (4 * (jp - 16));
            }
        }
    }
    wait_and_barrier<(NSTAGE - 1) * LPW>();
    read_frags(0, 0, 0);

    int stage = 0;
    auto kstep = [&](auto fbc, auto ksc) {
        constexpr int fb = decltype(fbc)::value;
        constexpr int ks = decltype(ksc)::value;
        constexpr bool last_of_stage = ks + 1 == KS;
        if constexpr (!last_of_stage) {
            read_frags(stage, ks + 1, fb ^ 1);
        } else {
            wait_and_barrier<(NSTAGE - 2) * LPW>();
            read_frags(stage + 1 < total ? stage + 1 : stage, 0, fb ^ 1);
            issue_next((unsigned)stage % NSTAGE);
        }
        mfmas(fb);
        if constexpr (last_of_stage) ++stage;
    };
    const std::integral_constant<int, 0> c0;
    const std::integral_constant<int, 1> c1;
    if constexpr (!INT8) {
        if (a.starts != nullptr) write_starts(0, 0xFu);
    }
    unsigned run_start = 0;                             // byte i*2+j: first pair of the run tile (i, j) is accumulating
    for (int jp = 0; jp < glen; ++jp) {
        const bool last_pair = jp + 1 == glen;
        unsigned cont = last_pair ? 0u : continue_mask(jp);
        v2s bav = {a.pair_bound, a.pair_bound}, bbv = bav;
        if constexpr (!INT8) {
            if (a.ba != nullptr && !last_pair) {
                bav = *(delta2_ptr)(a.ba + (qm * 4 + wm * 2) + (size_t)(p0 + jp + 1) * groups_a);
                bbv = *(delta2_ptr)(a.bb + (qn * 4 + wn * 2) + (size_t)(q0 - jp - 1) * groups_b);
            }
        }
        if constexpr (KS == 1) {
            int c = 0;
            for (; c + 1 < chunks; c += 2) {
                kstep(c0, c0);
                kstep(c1, c0);
            }
            if (c < chunks) {
                kstep(c0, c0);
                // odd number of stages: the fragments just fetched sit in buffer 1; the next k-step reads buffer 0
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    xf[0][i] = xf[1][i];
                    yf[0][i] = yf[1][i];
                }
            }
        } else {
            for (int c = 0; c < chunks; ++c) {
                kstep(c0, c0);
                kstep(c1, c1);
            }
        }
        if constexpr (!INT8) {
            if (a.starts != nullptr && !last_pair) {
                if (jp + 2 > a.sure && cont != 0u) cont = drop_full_tiles(cont, bav, bbv, acc);
                write_starts(jp + 1, ~cont);
            }
        }
        if (cont != 0xFu) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    if (!((cont >> (i * 2 + j)) & 1u)) {
                        store_tile(grp.slot + (int)((run_start >> (8 * (i * 2 + j))) & 0xFFu), i, j, acc[i][j]);
                        zero_tile(acc[i][j]);
                        run_start = (run_start & ~(0xFFu << (8 * (i * 2 + j)))) | ((unsigned)(jp + 1) << (8 * (i * 2 + j)));
                    }
        }
    }
    // every direct-to-LDS load (the tail's unused reloads too) must have landed before the LDS is released
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0) lgkmcnt(0)
    asm volatile("" ::: "memory");
}

template <bool BEHIND>
hipError_t launch_small_kernel(const SmallGemmArgs& a, int fmt, const dim3& grid, hipStream_t st) {
    const dim3 block(256);
    if (fmt == FMT_FP16) hipLaunchKernelGGL((pair_gemm_small_kernel<FMT_FP16, BEHIND>), grid, block, 0, st, a);
    else if (fmt == FMT_FP6) hipLaunchKernelGGL((pair_gemm_small_kernel<FMT_FP6, BEHIND>), grid, block, 0, st, a);
    else if (fmt == FMT_FP6_E3M2) hipLaunchKernelGGL((pair_gemm_small_kernel<FMT_FP6_E3M2, BEHIND>), grid, block, 0, st, a);
    else if (fmt == FMT_INT8) hipLaunchKernelGGL((pair_gemm_small_kernel<FMT_INT8, BEHIND>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((pair_gemm_small_kernel<FMT_FP8, BEHIND>), grid, block, 0, st, a);
    return hipGetLastError();
}

}  // namespace

}  // namespace ozaki
