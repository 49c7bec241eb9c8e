// C ABI of libozaki: contexts, argument checks and the kernel sequence (the planner is plan.hpp).
#include <stdio.h>
#include <string.h>

#include <new>
#include <vector>

#include "plan.hpp"

using namespace ozaki;

static_assert(OZAKI_MAX_SLICES == MAX_SLICES, "header and implementation disagree");
static_assert(OZAKI_SLICE_INT8 == FMT_INT8 && OZAKI_ACCUM_EXACT_FIXED == ACC_EXACT && OZAKI_SUM_PLAIN == SUM_PLAIN,
              "header and implementation disagree");

// A context: everything a call needs beyond its arguments.
struct ozaki_context_s {
    hipStream_t stream = nullptr;
    uint8_t* ws = nullptr;
    size_t ws_bytes = 0;
    int last_hip_error = 0;
    bool profiling = false;
    struct Span { hipEvent_t e0, e1; int phase; };
    std::vector<Span> spans;       // recorded since the last ozaki_profile_read
    std::vector<hipEvent_t> pool;  // idle events
};

namespace {

typedef ozaki_context_s Context;

Context default_context;
thread_local Context* current_context = nullptr;
Context& ctx() { return current_context ? *current_context : default_context; }

constexpr size_t MAX_SPANS = 4096;

// Work memory of ozaki_dgemm_static: one array per GPU the library runs on, part of the loaded code object (zero when
// the object is loaded), so that the entry point never allocates.  Host code must not use the array's name as an
// address: the per-device address comes from hipGetSymbolAddress, once per device, and is kept in static_scratch_ptr.
static __device__ __align__(256) unsigned char static_scratch[OZAKI_STATIC_SCRATCH_BYTES];
constexpr int MAX_DEVICES = 64;
uint8_t* static_scratch_ptr[MAX_DEVICES] = {};

int fail_hip(hipError_t e) {
    ctx().last_hip_error = (int)e;
    return OZAKI_STATUS_HIP_ERROR;
}
#define HIP_TRY(expr) do { hipError_t e_ = (expr); if (e_ != hipSuccess) return fail_hip(e_); } while (0)

// ---- profiling spans -------------------------------------------------------------------------------------------
hipEvent_t take_event(Context& c) {
    hipEvent_t e = nullptr;
    if (!c.pool.empty()) { e = c.pool.back(); c.pool.pop_back(); return e; }
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
}
// Brackets a phase with two events when profiling is on, the span list has room and the stream is not being
// captured into a graph (events recorded under capture cannot be timed).
struct Phase {
    Context& c;
    int phase; hipEvent_t e0 = nullptr, e1 = nullptr;
    explicit Phase(int ph) : c(ctx()), phase(ph) {
        if (!c.profiling || c.spans.size() >= MAX_SPANS) return;
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(c.stream, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone) return;
        e0 = take_event(c);
        e1 = e0 ? take_event(c) : nullptr;
        if (!e1) {                                       // no second event: give the first one back
            if (e0) c.pool.push_back(e0);
            e0 = nullptr;
            return;
        }
        (void)hipEventRecord(e0, c.stream);
    }
    ~Phase() {
        if (!e0 || !e1) return;
        (void)hipEventRecord(e1, c.stream);
        c.spans.push_back({e0, e1, phase});
    }
};

// Up to this many elements A is sliced from its columns as they are: the strided reads stay in the caches and cost less than a
// launch of their own (256 x 256: 5 us of 40; 64 x 16384: slicing 125 -> 117 us, 1000 x 777 x 1301: 48 -> 42, 7000 x 150: 58 -> 52).
constexpr int64_t MAX_ELEMS_WITHOUT_TRANSPOSE = 1 << 20;

// split both operands of the plan into the carved buffers
int run_split(const Plan& pl, const Carve& c, const double* A, int64_t lda, const double* B, int64_t ldb, bool do_a, bool do_b,
              const OffLadder& off = NO_LADDER) {
    Phase ph(0);
    hipStream_t st = ctx().stream;
    const bool a_on = do_a && pl.m > 0, b_on = do_b && pl.n > 0;
    const bool transpose = pl.kb > MAX_K_BLOCK_IN_REGISTERS || pl.m * pl.k > MAX_ELEMS_WITHOUT_TRANSPOSE;
    if (a_on && transpose) HIP_TRY(launch_transpose(A, lda, pl.m, pl.k, c.At, st));
    // both operands in one launch each: on a small problem neither fills the chip alone
    HIP_TRY(launch_split(transpose ? c.At : A, transpose ? pl.k : 1, transpose ? 1 : lda, a_on ? &c.A : nullptr, B, ldb, b_on ? &c.B : nullptr, pl,
                         c.flags, st));
    if (c.A.deltas != nullptr && off.uncounted == nullptr) HIP_TRY(launch_deltas(pl, a_on ? &c.A : nullptr, b_on ? &c.B : nullptr, off, st));
    return 0;
}

// zeros and normal numbers only: what the emulated multiplication covers (Section 4.2)
bool scalar_ok(double v) {
    uint64_t b;
    memcpy(&b, &v, 8);
    const int e = (int)((b >> 52) & 0x7FF);
    return (e != 0 && e != 0x7FF) || (b << 1) == 0;
}

struct Options {
    int slice_format, num_slices;
    int64_t k_block;
    int accum_mode, pair_set, sum_rule;
};

// Argument checks shared by the DGEMM entry points (positions of ozaki_dgemm / ozaki_dgemm_ex).
int check_dgemm_args(int64_t m, int64_t n, int64_t k, const double* A, int64_t lda, const double* B, int64_t ldb,
                     const double* C, int64_t ldc, const Options& o, Plan& pl) {
    if (o.pair_set != OZAKI_PAIRS_TRIANGLE && o.pair_set != OZAKI_PAIRS_ALL) return -14;
    const int st = make_plan(m, n, k, o.slice_format, o.num_slices, o.k_block, o.pair_set == OZAKI_PAIRS_ALL, pl);
    if (st != 0) return st;
    if (o.accum_mode < OZAKI_ACCUM_FP64_HW || o.accum_mode > OZAKI_ACCUM_EXACT_FIXED) return -13;
    if (o.sum_rule != OZAKI_SUM_RUNS && o.sum_rule != OZAKI_SUM_PLAIN) return -15;
    if (m == 0 || n == 0) return 0;
    if (!C) return -8;
    if (ldc < (m > 1 ? m : 1)) return -9;
    if (k > 0) {
        if (!A) return -4;
        if (lda < (m > 1 ? m : 1)) return -5;
        if (!B) return -6;
        if (ldb < (k > 1 ? k : 1)) return -7;
    }
    return 0;
}

// One Ozaki product on (a panel of) the operands: C = alpha * (A B) + beta * C.  (alpha, beta) = (1, 0): the product
// goes straight to C.  Otherwise the last accumulation combines it with C (earlier blocks of k go to the work memory).
// The arguments have been checked and the plan made (check_dgemm_args).
int dgemm_core(const Plan& plan, double alpha, const double* A, int64_t lda, const double* B, int64_t ldb, double beta, double* C,
               int64_t ldc, const Options& o, WorkMem wm) {
    const int64_t m = plan.m, n = plan.n, k = plan.k;
    if (m == 0 || n == 0) return 0;
    hipStream_t st = ctx().stream;
    const bool scaled = !(alpha == 1.0 && beta == 0.0);
    // the plain rule adds every product on its own, so the matrix unit must not sum across pairs
    const bool chained = o.sum_rule == OZAKI_SUM_RUNS || o.accum_mode == OZAKI_ACCUM_EXACT_FIXED;
    Route r;
    r.c.W = nullptr;
    if ((k > 0 || scaled) && !place_call(plan, scaled, o.accum_mode == OZAKI_ACCUM_EXACT_FIXED ? SUM_WORDS_MAX : 1, chained, true, wm, r))
        return OZAKI_STATUS_WORKSPACE;
    if (k > 0 && chained && (o.accum_mode != OZAKI_ACCUM_EXACT_FIXED || ladder_exact_fits(r.pl.fmt, r.pl.s, r.pl.full != 0))) place_ladder(r);
    const Plan& pl = r.pl;
    const Carve& c = r.c;
    const RunCheck& check = r.check;
    const OffLadder& off = r.off;
    double* const out = scaled ? c.W : C;
    const int64_t ldo = scaled ? (m > 1 ? m : 1) : ldc;
    const ScaledResult result = {alpha, beta, C, ldc};
    if (k == 0) {
        HIP_TRY(launch_fill_zero_f64(out, ldo, m, n, st));
        if (scaled) {
            Phase ph(2);
            HIP_TRY(launch_axpby(alpha, beta, c.W, ldo, C, ldc, m, n, o.accum_mode != OZAKI_ACCUM_FP64_HW, st));
        }
    } else {
        const PairOrder order = order_of(pl);
        int rc = run_split(pl, c, A, lda, B, ldb, true, true, off);
        if (rc) return rc;
        for (int64_t t = 0; t < pl.T; ++t) {
            for (int g_hi = order_top_diag(order); g_hi >= 2;) {
                const Pass ps = next_pass(order, g_hi, c.chunk_pairs);
                const bool first = g_hi == order_top_diag(order), last = ps.g_lo == 2 && t + 1 == pl.T;
                {
                    Phase ph(1);
                    // (between the halves of all pairs its sum lies where products will: an element's three words take less than s of them)
                    if (off.counts != nullptr && first) {
                        const ScaledResult* const combine = scaled && t + 1 == pl.T ? &result : nullptr;
                        HIP_TRY(launch_ladder_sums(pl, c.A, c.B, t, off, reinterpret_cast<uint64_t*>(c.P), out, ldo, combine, o.accum_mode, st));
                        if (off.limit > 0) HIP_TRY(launch_off_ladder(pl, c.A, c.B, off, out, ldo, combine, o.accum_mode, st));
                    }
                    HIP_TRY(launch_pair_gemm(pl, c.A, c.B, order, ps, chained, check, off, t, c.P, st));
                }
                {
                    Phase ph(2);
                    HIP_TRY(launch_accumulate(pl, c.A, c.B, order, ps, first, ps.g_lo == 2, t, c.P, c.S, out, ldo, scaled && last ? &result : nullptr,
                                              o.accum_mode, o.sum_rule, chained, check.starts, off, st));
                }
                g_hi = ps.g_lo - 1;
            }
        }
    }
    return 0;
}

// Outer-product-wise blocking (Section 4.3): panels of rows of A times panels of columns of B, each an Ozaki product
// of its own inside the capped work memory.  Rows of A and columns of B are sliced independently of the rest
// of their matrices, so every panel product carries the bits of the unblocked call.
int dgemm_panels(const Plan& whole, const double* A, int64_t lda, const double* B, int64_t ldb, double* C, int64_t ldc,
                 const Options& o, WorkMem wm) {
    int64_t mb = whole.m_pad, nb = whole.n_pad;
    Plan pl;
    for (;;) {
        const int st = make_plan(mb < whole.m ? mb : whole.m, nb < whole.n ? nb : whole.n, whole.k, o.slice_format, whole.s, o.k_block,
                                 whole.full != 0, pl);
        if (st != 0) return st;
        if (minimum_bytes(pl) <= wm.bytes) break;
        if (mb <= TILE && nb <= TILE) return OZAKI_STATUS_WORKSPACE;
        int64_t& big = mb >= nb ? mb : nb;                 // halve the longer side, in whole tiles
        big = ((big / TILE + 1) / 2) * TILE;
    }
    for (int64_t i0 = 0; i0 < whole.m; i0 += mb)
        for (int64_t j0 = 0; j0 < whole.n; j0 += nb) {
            const int64_t mi = whole.m - i0 < mb ? whole.m - i0 : mb, nj = whole.n - j0 < nb ? whole.n - j0 : nb;
            const int st = make_plan(mi, nj, whole.k, o.slice_format, whole.s, o.k_block, whole.full != 0, pl);
            if (st != 0) return st;
            const int rc = dgemm_core(pl, 1.0, A + i0, lda, B + j0 * ldb, ldb, 0.0, C + i0 + j0 * ldc, ldc, o, wm);
            if (rc != 0) return rc;
        }
    return 0;
}

WorkMem context_workspace() { return WorkMem{ctx().ws, ctx().ws_bytes}; }

int plan_for_query(int64_t m, int64_t n, int64_t k, int fmt, int s, int64_t k_block, int pair_set, Plan& pl) {
    if (pair_set != OZAKI_PAIRS_TRIANGLE && pair_set != OZAKI_PAIRS_ALL) return -14;
    return make_plan(m, n, k, fmt, s, k_block, pair_set == OZAKI_PAIRS_ALL, pl);
}

}  // namespace

extern "C" {

int ozaki_context_create(ozaki_context_t* ctx_out) {
    if (!ctx_out) return -1;
    *ctx_out = new (std::nothrow) ozaki_context_s();
    return *ctx_out ? 0 : OZAKI_STATUS_HIP_ERROR;
}

int ozaki_context_destroy(ozaki_context_t c) {
    if (!c || c == &default_context) return -1;
    if (current_context == c) current_context = nullptr;
    for (auto& sp : c->spans) { (void)hipEventDestroy(sp.e0); (void)hipEventDestroy(sp.e1); }
    for (auto e : c->pool) (void)hipEventDestroy(e);
    delete c;
    return 0;
}

int ozaki_context_use(ozaki_context_t c) {
    current_context = (c == &default_context) ? nullptr : c;
    return 0;
}

int ozaki_plan(int64_t k_block, int slice_format, int* rho_out, int* bits_out) {
    if (k_block < 1) return -1;
    if (!format_ok(slice_format)) return -2;
    const int b = slice_bits(k_block, slice_format);
    if (b < 0) return OZAKI_STATUS_INFEASIBLE;
    if (rho_out) *rho_out = 53 - b;
    if (bits_out) *bits_out = b;
    return 0;
}

int64_t ozaki_suggest_k_block(int64_t k, int slice_format) {
    if (k < 0) return -1;
    if (!format_ok(slice_format)) return -2;
    if (slice_format == OZAKI_SLICE_FP16) return k > 4096 ? 4096 : 0;
    if (slice_format == OZAKI_SLICE_INT8) return k > 524287 ? 262144 : 0;
    return k > 65536 ? MAX_K_BLOCK_IN_REGISTERS : 0;
}

int ozaki_set_stream(void* hip_stream) {
    ctx().stream = reinterpret_cast<hipStream_t>(hip_stream);
    return 0;
}

size_t ozaki_workspace_bytes_ex(int64_t m, int64_t n, int64_t k, int slice_format, int num_slices, int64_t k_block, int pair_set,
                                int minimum) {
    Plan pl;
    if (plan_for_query(m, n, k, slice_format, num_slices, k_block, pair_set, pl) != 0) return 0;
    return minimum ? minimum_bytes(pl) : recommended_bytes(pl);
}

size_t ozaki_workspace_bytes(int64_t m, int64_t n, int64_t k, int slice_format, int num_slices, int64_t k_block) {
    return ozaki_workspace_bytes_ex(m, n, k, slice_format, num_slices, k_block, OZAKI_PAIRS_TRIANGLE, 0);
}

size_t ozaki_workspace_min_bytes(int64_t m, int64_t n, int64_t k, int slice_format, int num_slices, int64_t k_block) {
    return ozaki_workspace_bytes_ex(m, n, k, slice_format, num_slices, k_block, OZAKI_PAIRS_TRIANGLE, 1);
}

int ozaki_set_workspace(void* dev_ptr, size_t bytes) {
    if ((dev_ptr == nullptr) != (bytes == 0)) return -1;
    if (reinterpret_cast<uintptr_t>(dev_ptr) % ALIGN != 0) return -1;
    if (dev_ptr && bytes < FLAG_BYTES) return -2;
    Context& c = ctx();
    c.ws = reinterpret_cast<uint8_t*>(dev_ptr);
    c.ws_bytes = bytes;
    if (c.ws) HIP_TRY(hipMemsetAsync(c.ws, 0, FLAG_BYTES, c.stream));
    return 0;
}

int ozaki_last_device_status(void) {
    // the flag words of the context's workspace and of this device's static scratch (if ozaki_dgemm_static has used it)
    Context& c = ctx();
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    uint8_t* places[2] = {c.ws, (dev >= 0 && dev < MAX_DEVICES) ? static_scratch_ptr[dev] : nullptr};
    int flags[2] = {0, 0};
    for (int i = 0; i < 2; ++i)
        if (places[i]) HIP_TRY(hipMemcpyAsync(&flags[i], places[i], sizeof(int), hipMemcpyDeviceToHost, c.stream));
    HIP_TRY(hipStreamSynchronize(c.stream));
    for (int i = 0; i < 2; ++i)
        if (flags[i]) HIP_TRY(hipMemsetAsync(places[i], 0, FLAG_BYTES, c.stream));
    return ((flags[0] | flags[1]) & 1) ? OZAKI_STATUS_NONFINITE : 0;
}

int ozaki_last_hip_error(void) { return ctx().last_hip_error; }

const char* ozaki_status_string(int status) {
    switch (status) {
        case OZAKI_STATUS_OK: return "success";
        case OZAKI_STATUS_INFEASIBLE: return "infeasible: no slice width keeps the matrix unit's accumulation exact for this block length";
        case OZAKI_STATUS_WORKSPACE: return "workspace missing or too small";
        case OZAKI_STATUS_HIP_ERROR: return "HIP runtime error";
        case OZAKI_STATUS_NONFINITE: return "non-finite input";
        case OZAKI_STATUS_STATIC_LIMIT: return "problem needs more work memory than the static scratch of ozaki_dgemm_static holds";
        case OZAKI_STATUS_SLICE_COUNT: return "num_slices exceeds OZAKI_MAX_SLICES";
        default: return status < 0 ? "invalid argument (the negated value is its 1-based position)" : "unknown status";
    }
}

int ozaki_profile_enable(int on) {
    ctx().profiling = on != 0;
    return 0;
}

int ozaki_profile_read(float* ms_out, int* launches_out) {
    if (!ms_out) return -1;
    Context& c = ctx();
    for (int i = 0; i < 3; ++i) { ms_out[i] = 0.0f; if (launches_out) launches_out[i] = 0; }
    // whatever happens below, every span leaves the list and its events return to the pool exactly once
    std::vector<Context::Span> spans;
    spans.swap(c.spans);
    hipError_t err = hipStreamSynchronize(c.stream);
    for (auto& sp : spans) {
        float ms = 0.0f;
        if (err == hipSuccess) err = hipEventElapsedTime(&ms, sp.e0, sp.e1);
        if (err == hipSuccess) {
            ms_out[sp.phase] += ms;
            if (launches_out) launches_out[sp.phase] += 1;
        }
        c.pool.push_back(sp.e0);
        c.pool.push_back(sp.e1);
    }
    return err == hipSuccess ? 0 : fail_hip(err);
}

int ozaki_dgemm_ex(int64_t m, int64_t n, int64_t k, const double* A, int64_t lda, const double* B, int64_t ldb, double* C,
                   int64_t ldc, int slice_format, int num_slices, int64_t k_block, int accum_mode, int pair_set, int sum_rule,
                   size_t mem_cap) {
    const Options o{slice_format, num_slices, k_block, accum_mode, pair_set, sum_rule};
    Plan pl;
    const int st = check_dgemm_args(m, n, k, A, lda, B, ldb, C, ldc, o, pl);
    if (st != 0) return st;
    WorkMem wm = context_workspace();
    if (mem_cap == 0 || m == 0 || n == 0 || k == 0) return dgemm_core(pl, 1.0, A, lda, B, ldb, 0.0, C, ldc, o, wm);
    if (wm.bytes > mem_cap) wm.bytes = mem_cap;
    return dgemm_panels(pl, A, lda, B, ldb, C, ldc, o, wm);
}

int ozaki_dgemm(int64_t m, int64_t n, int64_t k, const double* A, int64_t lda, const double* B, int64_t ldb,
                double* C, int64_t ldc, int slice_format, int num_slices, int64_t k_block, int accum_mode) {
    return ozaki_dgemm_ex(m, n, k, A, lda, B, ldb, C, ldc, slice_format, num_slices, k_block, accum_mode, OZAKI_PAIRS_TRIANGLE,
                          OZAKI_SUM_RUNS, 0);
}

int ozaki_dgemm_static(int64_t m, int64_t n, int64_t k, const double* A, int64_t lda, const double* B, int64_t ldb,
                       double* C, int64_t ldc, int slice_format, int num_slices, int64_t k_block, int accum_mode) {
    const Options o{slice_format, num_slices, k_block, accum_mode, OZAKI_PAIRS_TRIANGLE, OZAKI_SUM_RUNS};
    Plan pl;
    const int st = check_dgemm_args(m, n, k, A, lda, B, ldb, C, ldc, o, pl);
    if (st != 0) return st;
    if (m > 0 && n > 0 && k > 0 && minimum_bytes(pl) > (size_t)OZAKI_STATIC_SCRATCH_BYTES) return OZAKI_STATUS_STATIC_LIMIT;
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= MAX_DEVICES) return fail_hip(hipErrorInvalidDevice);
    if (!static_scratch_ptr[dev]) {
        void* p = nullptr;
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(static_scratch)));
        if (!p) return fail_hip(hipErrorInvalidSymbol);
        static_scratch_ptr[dev] = static_cast<uint8_t*>(p);
    }
    // Nothing in the scratch has to start at zero except the flag word, which is zero when the code object is loaded
    // and is cleared by ozaki_last_device_status after it has reported a flag: every other buffer of the carve-up is
    // written in full by the slicing and GEMM kernels before it is read.
    return dgemm_core(pl, 1.0, A, lda, B, ldb, 0.0, C, ldc, o, WorkMem{static_scratch_ptr[dev], (size_t)OZAKI_STATIC_SCRATCH_BYTES});
}

int ozaki_dgemm_scaled(int64_t m, int64_t n, int64_t k, double alpha, const double* A, int64_t lda, const double* B, int64_t ldb,
                       double beta, double* C, int64_t ldc, int slice_format, int num_slices, int64_t k_block, int accum_mode) {
    if (!scalar_ok(alpha)) return -4;
    if (!scalar_ok(beta)) return -9;
    const Options o{slice_format, num_slices, k_block, accum_mode, OZAKI_PAIRS_TRIANGLE, OZAKI_SUM_RUNS};
    Plan pl;
    int st = check_dgemm_args(m, n, k, A, lda, B, ldb, C, ldc, o, pl);
    if (st == 0) st = dgemm_core(pl, alpha, A, lda, B, ldb, beta, C, ldc, o, context_workspace());
    // argument positions of ozaki_dgemm -> positions in this signature (alpha and beta inserted)
    if (st < 0) return st >= -3 ? st : st >= -7 ? st - 1 : st - 2;
    return st;
}

size_t ozaki_workspace_bytes_scaled(int64_t m, int64_t n, int64_t k, int slice_format, int num_slices, int64_t k_block) {
    Plan pl;
    if (make_plan(m, n, k, slice_format, num_slices, k_block, false, pl) != 0) return 0;
    return recommended_bytes(pl) + product_bytes(pl);
}

int ozaki_split(int is_B, int64_t rows, int64_t k, const double* X, int64_t ldx, int slice_format, int num_slices,
                int64_t k_block, void* slices_out, int32_t* exps_out) {
    if (is_B != 0 && is_B != 1) return -1;
    if (rows < 0) return -2;
    if (k < 0) return -3;
    if (num_slices < 1) return -7;
    Plan pl;
    // plan with the operand in the role it has in the product; the other dimension is irrelevant here
    const int st = make_plan(is_B ? 0 : rows, is_B ? rows : 0, k, slice_format, num_slices, k_block, false, pl);
    if (st < 0) return st == -10 ? -6 : st == -12 ? -8 : st;
    if (st != 0) return st;
    if (rows == 0 || k == 0) return 0;
    if (!X) return -4;
    if (ldx < (is_B ? (k > 1 ? k : 1) : (rows > 1 ? rows : 1))) return -5;
    if (!slices_out) return -9;
    if (!exps_out) return -10;
    Carve c;
    if (!carve(pl, c, false, 1, context_workspace())) return OZAKI_STATUS_WORKSPACE;
    int rc = run_split(pl, c, X, ldx, X, ldx, !is_B, is_B != 0);
    if (rc) return rc;
    hipStream_t stream = ctx().stream;
    const Operand& op = is_B ? c.B : c.A;
    HIP_TRY(launch_export_slices(pl, op, slices_out, stream));
    // exponents: [T][s][rows_pad] -> [T][s][rows]
    HIP_TRY(hipMemcpy2DAsync(exps_out, (size_t)rows * sizeof(int32_t), op.exps, (size_t)op.rows_pad * sizeof(int32_t),
                             (size_t)rows * sizeof(int32_t), (size_t)pl.T * pl.s, hipMemcpyDeviceToDevice, stream));
    return 0;
}

int ozaki_count_slices(int is_B, int64_t rows, int64_t k, const double* X, int64_t ldx, int slice_format, int64_t k_block,
                       int* count_out) {
    if (is_B != 0 && is_B != 1) return -1;
    if (rows < 0) return -2;
    if (k < 0) return -3;
    if (!count_out) return -8;
    Plan pl;
    const int st = make_plan(is_B ? 0 : rows, is_B ? rows : 0, k, slice_format, 1, k_block, false, pl);
    if (st < 0) return st == -10 ? -6 : st == -12 ? -7 : st;
    if (st != 0) return st;
    *count_out = 0;
    if (rows == 0 || k == 0) return 0;
    if (!X) return -4;
    if (ldx < (is_B ? (k > 1 ? k : 1) : (rows > 1 ? rows : 1))) return -5;
    // needs the flag block, for A room for its transpose, and for long blocks the reserve of the documented size
    Context& c = ctx();
    const size_t at_bytes = is_B ? 0 : align_up((size_t)rows * k * sizeof(double));
    const size_t need = FLAG_BYTES + at_bytes + long_block_reserve(pl);
    if (!c.ws || c.ws_bytes < need) return OZAKI_STATUS_WORKSPACE;
    int* flags = reinterpret_cast<int*>(c.ws);
    HIP_TRY(hipMemsetAsync(flags + 1, 0, sizeof(int), c.stream));
    const double* vecs = X;
    int64_t ldv = ldx;
    if (!is_B) {
        double* At = reinterpret_cast<double*>(c.ws + FLAG_BYTES);
        HIP_TRY(launch_transpose(X, ldx, rows, k, At, c.stream));
        vecs = At;
        ldv = k;
    }
    HIP_TRY(launch_count_slices(vecs, ldv, pl, rows, flags, c.stream));
    int count = 0;
    HIP_TRY(hipMemcpyAsync(&count, flags + 1, sizeof(int), hipMemcpyDeviceToHost, c.stream));
    HIP_TRY(hipStreamSynchronize(c.stream));
    *count_out = count;
    return 0;
}

int ozaki_pair_products(int64_t m, int64_t n, int64_t k, const double* A, int64_t lda, const double* B, int64_t ldb,
                        int slice_format, int num_slices, int64_t k_block, int pair_set, int chained, void* P_out,
                        uint8_t* run_len_out) {
    if (pair_set != OZAKI_PAIRS_TRIANGLE && pair_set != OZAKI_PAIRS_ALL) return -11;
    Plan plan;
    int st = make_plan(m, n, k, slice_format, num_slices, k_block, pair_set == OZAKI_PAIRS_ALL, plan);
    if (st < 0) return st == -10 ? -8 : st == -11 ? -9 : st == -12 ? -10 : st;
    if (st != 0) return st;
    if (num_slices < 1) return -9;
    if (m == 0 || n == 0 || k == 0) return 0;
    if (!A) return -4;
    if (lda < m) return -5;
    if (!B) return -6;
    if (ldb < k) return -7;
    if (!P_out) return -13;
    Route r;
    if (!place_call(plan, false, 1, chained != 0, chained == 2, context_workspace(), r)) return OZAKI_STATUS_WORKSPACE;
    const Plan& pl = r.pl;
    const Carve& c = r.c;
    hipStream_t stream = ctx().stream;
    const PairOrder order = order_of(pl);
    int rc = run_split(pl, c, A, lda, B, ldb, true, true);
    if (rc) return rc;
    // the export reads the links from the deltas also where the GEMM kernel formed them itself
    Operand ea = c.A, eb = c.B;
    ea.deltas = r.deltas_a;
    eb.deltas = r.deltas_b;
    if (c.A.deltas == nullptr) HIP_TRY(launch_deltas(pl, &ea, &eb, NO_LADDER, stream));
    for (int64_t t = 0; t < pl.T; ++t) {
        int z0 = 0;
        for (int g_hi = order_top_diag(order); g_hi >= 2;) {
            const Pass ps = next_pass(order, g_hi, c.chunk_pairs);
            const size_t at = ((size_t)t * pl.npairs + z0) * (size_t)m * n;
            HIP_TRY(launch_pair_gemm(pl, c.A, c.B, order, ps, chained != 0, r.check, NO_LADDER, t, c.P, stream));
            HIP_TRY(launch_export_products(pl, ea, eb, order, ps, chained != 0, r.check.starts, t, c.P, static_cast<float*>(P_out) + at,
                                           run_len_out ? run_len_out + at : nullptr, stream));
            z0 += ps.npairs;
            g_hi = ps.g_lo - 1;
        }
    }
    return 0;
}

int ozaki_fp64_add_emulated(const double* a, const double* b, double* out, int64_t n) {
    if (n < 0) return -4;
    if (n == 0) return 0;
    if (!a) return -1;
    if (!b) return -2;
    if (!out) return -3;
    HIP_TRY(launch_add_emulated(a, b, out, n, ctx().stream));
    return 0;
}

}  // extern "C"
