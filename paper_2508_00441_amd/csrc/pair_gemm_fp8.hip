// The 256 x 256 slice-pair GEMM of pair_gemm_body.hpp for FP8 slices on v_mfma_f32_16x16x128_f8f6f4.
//
// What bounds the GEMM is the power the matrix unit draws (the clock falls to 1.8 - 1.95 GHz under it) together with the L2 -> LDS
// stream.  On slice codes the 16 x 16 x 128 form of the FP8 instruction does the same work for less: from registers alone 4.8 PFLOP/s
// against 4.0 - 4.4 of the 32 x 32 x 64 form (uniform codes), 4.9 against 4.57 (codes of normally distributed values); on constant
// data both reach 5.0.  (FP16 1.70 against 1.80, INT8 3.3 against 3.6, FP6 5.9 against 6.0 PFLOP/s: there the larger form is the better one.)
// With it the kernel runs at 2.0 - 2.1 GHz instead of 1.83 - 1.90; part of that is lost again to the ring, which holds two and a
// half of the longer k-steps instead of five of the shorter ones (matrix pipes busy 80 % of the cycles instead of 83 %).  Against
// pair_gemm_kernel<FMT_FP8>, ms: 8192 x 8192 x 8192, 16 slices 45.1 -> 43.5 (3.43 PFLOP/s); 4096 x 4096 x 4096, 13 slices 3.92 -> 3.85;
// 16384 x 8192 x 1024, 13 slices 8.87 -> 8.39, of which 0.44 are the non-temporal stores.  Problems of few
// tiles, which wait for their panels rather than for the matrix unit, lose (1000 x 777 x 1301 94 -> 100 us, 1024 x 1024 x 1024 101 -> 103,
// 256 x 320 x 65536 676 -> 685), and so do pairs of a single step and short odd numbers of stages: see fp8_long_steps in pair_gemm.hip.
//
// The work items, the stage ring, the LDS swizzle, the runs and the order of the stored words are those of pair_gemm_body.hpp.  What differs:
//   * A k-step takes two stages (128 bytes of the inner dimension): lanes 0 .. 31 hold the first, lanes 32 .. 63 the second.  A pair
//     with an odd number of stages is filled up with a stage of zeros (every lane loads the same sixteen).
//   * The fragments of a k-step are 128 registers, so two sets of both operands do not fit beside 256 accumulators.  The k-step runs
//     along rows of eight MFMAs that share a B fragment; that fragment's successor is read into its place once the row is done, and
//     only the A fragments, which every row needs, and the last two rows' B fragments (whose successors would come too late for the
//     barrier) have two sets.
//   * A wave's 32 x 32 tile is four accumulator tuples of 16 x 16, stored where the 32 x 32 tuple's lanes would store them.
#include "pair_gemm_body.hpp"

namespace ozaki {

namespace {

__device__ __attribute__((aligned(16))) uint8_t zero_piece[16];

template <bool MEASURED>
__device__ __forceinline__ void pair_gemm_fp8_body(const GemmArgs& a) {
    constexpr int BK = CHUNK_BYTES, OPERAND_BYTES = TILE * BK, STAGE_BYTES = 2 * OPERAND_BYTES;
    constexpr int LPW = OPERAND_BYTES / 1024 / 4;     // direct-to-LDS load instructions per wave, operand and stage
    constexpr int NSTAGE = 5;
    __shared__ __attribute__((aligned(16))) uint8_t lds[NSTAGE * STAGE_BYTES];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave >> 1, wm = wave & 1;
    const WorkItem item = work_item(blockIdx.x, gridDim.x, a.work, a.tiles_m, a.tiles_n);
    const int tn = item.bn, tm = item.bm;
    if (on_ladder(a.off)) return;
    const Group grp = listed_group(a.groups, a.order, a.pass, item.gi);
    const int glen = grp.len, p0 = grp.p0 - 1, q0 = grp.q0 - 1;
    const int chunks = (int)a.chunks, steps = (chunks + 1) >> 1;

    // runs: as in pair_gemm_body
    typedef int v4s __attribute__((ext_vector_type(4)));
    typedef const __attribute__((address_space(4))) v4s* delta4_ptr;
    const int64_t groups_a = a.rows_pad_a / LINK_ROWS, groups_b = a.rows_pad_b / LINK_ROWS;
    const int32_t* const dA = a.da + (tm * 8 + wm * 4);
    const int32_t* const dB = a.db + (tn * 8 + wn * 4);
    auto continue_mask = [&](int jp) -> unsigned {
        if (!a.allow_chain) return 0u;
        const v4s dav = *(delta4_ptr)(dA + (size_t)(p0 + jp) * groups_a);
        const v4s dbv = *(delta4_ptr)(dB + (size_t)(q0 - jp - 1) * groups_b);
        unsigned cont = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                cont |= deltas_link(__builtin_amdgcn_readfirstlane(dav[j]), __builtin_amdgcn_readfirstlane(dbv[i])) ? (1u << (i * 4 + j)) : 0u;
        return cont;
    };
    auto write_starts = [&](int jp, unsigned first) {
        if (lane < 16)
            a.starts[((size_t)((grp.slot + jp) * a.tiles_n + tn) * a.tiles_m + tm) * 64 + wave * 16 + lane] = (uint8_t)((first >> lane) & 1u);
    };

    // loader: as in pair_gemm_body for 64-byte rows
    const size_t cs_x = (size_t)a.rows_pad_b * BK, cs_y = (size_t)a.rows_pad_a * BK;
    const unsigned lrow = lane >> 2, lpc = lane & 3;
    const unsigned goff = wave * LPW * 1024 + lrow * BK + ((lpc ^ ((lrow >> 2) & 3)) << 4);
    const uint8_t* xptr = a.sb + (size_t)tn * TILE * BK + goff + (size_t)q0 * chunks * cs_x;
    const uint8_t* yptr = a.sa + (size_t)tm * TILE * BK + goff + (size_t)p0 * chunks * cs_y;
    const size_t x_wrap = (size_t)(2 * chunks - 1) * cs_x;           // from a slice's last chunk back to the first of the slice before it
    const int total = 2 * glen * steps;                               // stages
    int issued = 0, issue_kc = 0, issue_buf = 0;
    // instructions 2h and 2h+1 of the next stage's 2 * LPW, h < 4
    auto issue_two = [&](int h) {
        const bool none = issue_kc >= chunks;                         // the stage of zeros
#pragma unroll
        for (int i = 2 * h; i < 2 * h + 2; ++i) {
            const uint8_t* src = (i < LPW ? xptr : yptr) + (i % LPW) * 1024;
            src = none ? zero_piece : src;
            __builtin_amdgcn_global_load_lds(OZAKI_GPTR(src),
                                             OZAKI_LPTR(lds + issue_buf * STAGE_BYTES + (i < LPW ? 0 : OPERAND_BYTES) + (wave * LPW + i % LPW) * 1024), 16, 0, 0);
        }
    };
    // to the next stage; after the last one the pointers stay put (the unused reloads keep the outstanding-load count uniform)
    auto advance = [&]() {
        const bool adv = issued + 1 < total, wrap = issue_kc + 1 == 2 * steps, into_zeros = issue_kc + 1 == chunks && !wrap;
        const int64_t dx = adv && !into_zeros ? (wrap ? -(int64_t)x_wrap : (int64_t)cs_x) : 0;
        const int64_t dy = adv && !into_zeros ? (int64_t)cs_y : 0;
        xptr += dx;
        yptr += dy;
        issued += adv ? 1 : 0;
        issue_kc = adv ? (wrap ? 0 : issue_kc + 1) : issue_kc;
        issue_buf = issue_buf + 1 == NSTAGE ? 0 : issue_buf + 1;
    };

    // fragments: lane reads row lane % 16 of each 16-row tile, 32 bytes of k-group lane / 16; groups 0, 1 are the first stage of the
    // step, 2, 3 the second
    const int frow = lane & 15, fg = (lane >> 4) & 1, fsw = (frow >> 2) & 3;
    // (Group 0 takes pieces 0 and 1 of its row, group 1 pieces 3 and 2: the sixteen lanes that a 128-bit LDS read serves together are
    // 0-3, 12-15, 20-23, 24-27 and the like; with 2 and 3 in group 1 they meet in pairs on the banks, 18 % of the cycles.)
    const int piece0 = ((fg ? 3 : 0) ^ fsw) << 4, piece1 = ((fg ? 2 : 1) ^ fsw) << 4;
    const int xbase = (wn * 128 + frow) * BK, ybase = OPERAND_BYTES + (wm * 128 + frow) * BK;
    v8i xf[6], xl[2][2], yf[2][8];                    // B fragments of rows 0 .. 5, of rows 6 and 7 (two sets), A fragments (two sets)
    int read_buf = 0;
    unsigned read_at = 0;                             // this lane's stage buffer
    auto set_read = [&]() {
        const int other = read_buf + 1 == NSTAGE ? 0 : read_buf + 1;
        read_at = (unsigned)(lane < 32 ? read_buf : other) * STAGE_BYTES;
    };
    auto read_one = [&](int base, int f) -> v8i {
        const uint8_t* at = lds + read_at + base + f * 16 * BK;
        const v4i lo = *reinterpret_cast<const v4i*>(at + piece0), hi = *reinterpret_cast<const v4i*>(at + piece1);
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };

    v4f acc[8][8];                                    // tile (i, j) of 32 x 32: acc[2i .. 2i+1][2j .. 2j+1]
    auto zero_tile = [&](int i, int j) {
#pragma unroll
        for (int h = 0; h < 4; ++h) acc[2 * i + (h >> 1)][2 * j + (h & 1)] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    };
    // In a 32 x 32 tile of P the four words of rows n = 8g + 4h .. + 3 and column m are the 16 bytes at g * 1024 + (h * 32 + m) * 16.
    // A 16 x 16 tuple (ti, tj) holds in lane l rows 16 ti + 4 (l / 16) .. + 3 of column 16 tj + l % 16.
    const unsigned lane_bytes = (unsigned)(((lane >> 5) * 64 + ((lane >> 4) & 1) * 32 + (lane & 15)) * 16);
    const int qn = tn * 2 + wn, qm = tm * 2 + wm;
    const bool has_block = qn < a.quads_n && qm < a.quads_m;
    // Non-temporal whatever the size of the products: this kernel has 256 tiles and more, 64 MiB per group, and unlike with
    // pair_gemm_kernel (STREAMED_PRODUCT_BYTES) that is the faster form from there on.  GEMM and accumulation, us, with ordinary stores below
    // 512 MiB and without: 4096 x 4096 x 4096, 4 slices 579 and 572, 5 slices 738 and 728, 6 slices 957 and 950, 7 slices 1242 and 1220;
    // 5120 x 4096 x 2048, 4 slices 456 and 438; 8192 x 4096 x 512, 4 slices 341 and 337.
    auto store_tile = [&](int slot, int i, int j) {
        if (!has_block) return;
        char* base = reinterpret_cast<char*>(a.P + ((size_t)(slot * a.quads_n + qn) * a.quads_m + qm) * QUAD_ELEMS + (size_t)(i * 4 + j) * 1024);
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            v4f* const dst = reinterpret_cast<v4f*>(base + (h >> 1) * 2048 + (h & 1) * 256 + lane_bytes);
            __builtin_nontemporal_store(acc[2 * i + (h >> 1)][2 * j + (h & 1)], dst);
        }
    };
    // Measured runs: tile (i, j) may only go on if its accumulators leave room for every partial sum of the next pair.
    auto drop_full_tiles = [&](unsigned cont, const v4s& bav, const v4s& bbv) -> unsigned {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (!((cont >> (i * 4 + j)) & 1u)) continue;
                const int next = bav[j] < bbv[i] ? bav[j] : bbv[i];
                const float room = (float)((1 << 24) - next) * a.unit;          // exact: an integer below 2^24 times a power of two
                float most = 0.0f;
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    v4f c = acc[2 * i + (h >> 1)][2 * j + (h & 1)];
                    asm volatile("" : "+v"(c));       // one copy of the tuple (see largest)
#pragma unroll
                    for (int r = 0; r < 4; ++r) most = fmaxf(most, fabsf(c[r]));
                }
                if (__ballot(!(most <= room)) != 0ull) cont &= ~(1u << (i * 4 + j));
            }
        return cont;
    };

#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) zero_tile(i, j);
    // prologue: fill the ring, wait for stages 0 and 1, read the first step's fragments
#pragma unroll
    for (int st = 0; st < NSTAGE; ++st) {
#pragma unroll
        for (int h = 0; h < 4; ++h) issue_two(h);
        advance();
    }
    wait_and_barrier<(NSTAGE - 2) * 2 * LPW>();
    set_read();
#pragma unroll
    for (int f = 0; f < 8; ++f) {
        if (f < 6) xf[f] = read_one(xbase, f);
        else xl[0][f - 6] = read_one(xbase, f);
        yf[0][f] = read_one(ybase, f);
    }

    // LDS reads and loads are spread evenly over the step, two loads and about four reads per row, the loads four MFMAs apart: the
    // LDS port is busy three quarters of the time and bunched traffic stops the wave that issues it.  8192 x 8192 x 8192, ms: 43.8 as
    // here, 44.3 with all reads in the first five rows, 47.6 with all loads in the first four rows too; a second barrier in the middle
    // of the step, with which every stage is asked for a whole step before it is needed, 44.9.
    // One k-step.  At its head every wave waits for its own LDS reads (the fragments of this step: their two buffers are dead once
    // all waves have met) and for the stages of the next step, whose fragments are read while this step's MFMAs run; the dead
    // buffers are refilled.
    auto step = [&](auto set) {
        constexpr int S = decltype(set)::value;
        wait_and_barrier<2 * LPW>();
        read_buf = read_buf + 2 >= NSTAGE ? read_buf + 2 - NSTAGE : read_buf + 2;
        set_read();
        auto row = [&](auto rc) {
            constexpr int R = decltype(rc)::value;
            // LDS reads of the row, two per fragment
            if constexpr (R == 0) {
                xl[S ^ 1][0] = read_one(xbase, 6);
                xl[S ^ 1][1] = read_one(xbase, 7);
                yf[S ^ 1][0] = read_one(ybase, 0);
            } else {
                if constexpr (R <= 6) xf[R - 1] = read_one(xbase, R - 1);
                yf[S ^ 1][R] = read_one(ybase, R);
            }
            constexpr int READS = R == 0 ? 6 : R == 7 ? 2 : 4;
            issue_two(R & 3);
            if constexpr ((R & 3) == 3) advance();
#pragma unroll
            for (int jj = 0; jj < 8; ++jj) {
                const int j = (R & 1) ? 7 - jj : jj;  // boustrophedon: consecutive MFMAs differ in one operand only
                acc[R][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(R < 6 ? xf[R < 6 ? R : 0] : xl[S][R < 6 ? 0 : R - 6], yf[S][j], acc[R][j], 0, 0, 0, 0, 0, 0);
            }
#pragma unroll
            for (int jj = 0; jj < 8; ++jj) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                       // one MFMA
                if (jj < READS) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);       // an LDS read
                if (jj == 2 || jj == 6) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);          // a VMEM read
            }
            __builtin_amdgcn_sched_barrier(0);        // a fragment's successor is not read before its row is done
        };
        row(std::integral_constant<int, 0>{});
        row(std::integral_constant<int, 1>{});
        row(std::integral_constant<int, 2>{});
        row(std::integral_constant<int, 3>{});
        row(std::integral_constant<int, 4>{});
        row(std::integral_constant<int, 5>{});
        row(std::integral_constant<int, 6>{});
        row(std::integral_constant<int, 7>{});
    };
    const std::integral_constant<int, 0> s0;
    const std::integral_constant<int, 1> s1;
    if constexpr (MEASURED) write_starts(0, 0xFFFFu);
    unsigned run_start[4] = {0u, 0u, 0u, 0u};           // byte j of word i: first pair of the run tile (i, j) is accumulating
    for (int jp = 0; jp < glen; ++jp) {
        const bool last_pair = jp + 1 == glen;
        unsigned cont = last_pair ? 0u : continue_mask(jp);
        v4s bav = {a.pair_bound, a.pair_bound, a.pair_bound, a.pair_bound}, bbv = bav;
        if constexpr (MEASURED) {
            if (a.ba != nullptr && !last_pair) {
                bav = *(delta4_ptr)(a.ba + (tm * 8 + wm * 4) + (size_t)(p0 + jp + 1) * groups_a);
                bbv = *(delta4_ptr)(a.bb + (tn * 8 + wn * 4) + (size_t)(q0 - jp - 1) * groups_b);
            }
        }
        int c = 0;
        for (; c + 1 < steps; c += 2) {
            step(s0);
            step(s1);
        }
        if (c < steps) {
            step(s0);
            // odd number of steps: the next one's fragments sit in the second sets, the next step reads the first
#pragma unroll
            for (int f = 0; f < 8; ++f) yf[0][f] = yf[1][f];
            xl[0][0] = xl[1][0];
            xl[0][1] = xl[1][1];
        }
        if constexpr (MEASURED) {
            if (!last_pair) {
                if (jp + 2 > a.sure && cont != 0u) cont = drop_full_tiles(cont, bav, bbv);
                write_starts(jp + 1, ~cont);
            }
        }
        if (cont != 0xFFFFu) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (!((cont >> (i * 4 + j)) & 1u)) {
                        store_tile(grp.slot + (int)((run_start[i] >> (8 * j)) & 0xFFu), i, j);
                        zero_tile(i, j);
                        run_start[i] = (run_start[i] & ~(0xFFu << (8 * j))) | ((unsigned)(jp + 1) << (8 * j));
                    }
        }
    }

    // every direct-to-LDS load of this wave must have landed before the workgroup's LDS allocation is released
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0) lgkmcnt(0)
    asm volatile("" ::: "memory");
}

__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) pair_gemm_fp8_kernel(const GemmArgs a) { pair_gemm_fp8_body<false>(a); }
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) pair_gemm_fp8_measured_kernel(const GemmArgs a) { pair_gemm_fp8_body<true>(a); }

}  // namespace

hipError_t launch_pair_gemm_fp8(const GemmArgs& a, bool measured, unsigned blocks, hipStream_t st) {
    if (measured) hipLaunchKernelGGL(pair_gemm_fp8_measured_kernel, dim3(blocks), dim3(256), 0, st, a);
    else hipLaunchKernelGGL(pair_gemm_fp8_kernel, dim3(blocks), dim3(256), 0, st, a);
    return hipGetLastError();
}

}  // namespace ozaki
