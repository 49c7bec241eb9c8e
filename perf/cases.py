"""What is measured: calls of the DGEMM entry points as programs make them, from the smallest sizes to the largest.

A case names the entry point, the problem (m, n, k), the slice format and count, the block length of the inner dimension,
the accumulation, the pair set and the distribution of the entries.  Sizes, slice counts and distributions are those of
paper_2508_00441_amd/inputs.py and of the tests, or generic ones between them.  The library's results are defined bit for
bit (each accumulation mode has one order of its roundings), so every case is compared exactly.
"""
import math

import torch

from paper_2508_00441_amd import binding as lib

# slices for full FP64 accuracy at phi <= 2 and, for all pairs, the counts of the paper's Table 2
SLICES = {"fp8": 13, "fp6": 13, "fp6_e3m2": 16, "int8": 9, "fp16": 8}
SLICES_ALL = {"fp8": 11, "fp6": 11, "fp6_e3m2": 14, "int8": 8, "fp16": 7}
MOST_SLICE_FLOPS = 1.4e14        # a drawn case costs no more than the largest listed ones
MOST_WORKSPACE = 40 << 30


def _case(name, entry, m, n, k, fmt, s, accum, k_block=0, pairs="triangle", dist="phi", phi=1.0, pad=0):
    return dict(name=name, entry=entry, m=m, n=n, k=k, fmt=fmt, s=s, accum=accum, k_block=k_block, pairs=pairs, dist=dist,
                phi=float(phi), pad=pad)


def listed():
    return [
        # a call so small that launches and latency are all of it: the smallest benchmark configuration
        _case("small_256_fp8", "dgemm", 256, 256, 256, "fp8", 12, "hw", phi=0.5),
        # a serving loop that may not allocate: the entry point with its own fixed work memory, near its limit
        _case("static_600_fp8_emu", "static", 600, 600, 1000, "fp8", 11, "emu"),
        # the residual R = C - A B of an iterative refinement: odd sizes, padded leading dimensions, integer-only
        _case("residual_1000x777x1301_fp8", "scaled", 1000, 777, 1301, "fp8", 12, "emu", pad=3),
        # the paper's own workload (entries U(1,10), every slice pair) at its smallest size
        _case("paper_1024_fp8_all", "ex", 1024, 1024, 1024, "fp8", 11, "hw", pairs="full", dist="u110"),
        # the paper's FP16 comparison with blocks of 1024
        _case("paper_2048_fp16_kb1024_all", "ex", 2048, 2048, 2048, "fp16", 7, "hw", k_block=1024, pairs="full", dist="u110"),
        # the longest unblocked inner dimension of the paper's Table 2 with a small result, summed without rounding
        _case("long_256x320x65536_fp8_exact", "ex", 256, 320, 65536, "fp8", 11, "exact", pairs="full", dist="u110"),
        # a block of a few vectors against a large matrix, odd inner dimension
        _case("skinny_96x6000x4097_int8", "dgemm", 96, 6000, 4097, "int8", 9, "hw"),
        # the ordinary square size, full accuracy
        _case("square_4096_fp8", "dgemm", 4096, 4096, 4096, "fp8", 13, "hw"),
        # the paper's workload on the FP6 path, with the additions emulated
        _case("paper_4096_fp6_all_emu", "ex", 4096, 4096, 4096, "fp6", 11, "emu", pairs="full", dist="u110"),
        # the headline configuration: wide exponent range, integer-only
        _case("headline_8192_fp8_emu", "dgemm", 8192, 8192, 8192, "fp8", 16, "emu", phi=4.0),
        # a rank-1024 update of a large matrix: short inner dimension, large result
        _case("update_16384x8192x1024_fp8", "dgemm", 16384, 8192, 1024, "fp8", 13, "emu", phi=2.0),
        # the largest: k-blocked FP16 at 16384
        _case("large_16384_fp16_kb4096", "dgemm", 16384, 16384, 16384, "fp16", 9, "hw", k_block=4096),
    ]


def _pairs(case):
    return case["s"] ** 2 if case["pairs"] == "full" else case["s"] * (case["s"] + 1) // 2


def _workspace_bytes(case):
    a = (case["m"], case["n"], case["k"], lib.SLICE_FORMATS[case["fmt"]], case["s"], case["k_block"])
    if case["entry"] == "scaled":
        return lib.ozaki_workspace_bytes_scaled(*a)
    return lib.ozaki_workspace_bytes_ex(*a, lib.PAIR_SETS[case["pairs"]], False)


def draw(rng):
    def size(lo, hi):
        v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
        return v | 1 if rng.random() < 0.4 else max(lo, v // 16 * 16)

    while True:
        m, n, k = size(64, 8192), size(64, 8192), size(64, 8192)
        fmt = rng.choice(["fp8", "fp8", "fp8", "fp6", "fp6_e3m2", "int8", "fp16"])
        if fmt == "fp16":
            k_block = rng.choice([1024, 2048, 4096])
        else:
            k_block = rng.choice([0, 0, 0, 2048])
            if rng.random() < 0.1:
                k = size(16384, 65536)                      # unblocked beyond the register-resident slicer
        entry = rng.choice(["dgemm", "dgemm", "ex", "ex", "scaled", "static"])
        pairs = rng.choice(["full", "triangle"]) if entry == "ex" else "triangle"
        dist = "u110" if pairs == "full" else "phi"
        s = SLICES_ALL[fmt] if pairs == "full" else SLICES[fmt] + rng.choice([-1, 0, 0, 1])
        accum = rng.choice(["hw", "hw", "emu", "emu", "exact"])
        c = _case("", entry, m, n, k, fmt, s, accum, k_block, pairs, dist, rng.choice([0.5, 1.0, 2.0]), rng.choice([0, 0, 0, 1, 8]))
        del c["name"]
        if 2.0 * _pairs(c) * m * n * k > MOST_SLICE_FLOPS or _workspace_bytes(c) > MOST_WORKSPACE:
            continue
        if entry == "static":
            a = (m, n, k, lib.SLICE_FORMATS[fmt], s, k_block)
            if lib.ozaki_workspace_min_bytes(*a) > lib.STATIC_SCRATCH_BYTES:
                continue
        return c


def _matrix(rows, cols, pad, case, gen):
    """Column-major rows x cols with leading dimension rows + pad: a tensor of shape (cols, rows + pad)."""
    shape = (cols, rows + pad)
    x = torch.rand(shape, dtype=torch.float64, device="cuda", generator=gen)
    if case["dist"] == "u110":
        return x.mul_(9.0).add_(1.0)
    z = torch.randn(shape, dtype=torch.float64, device="cuda", generator=gen)
    return x.sub_(0.5).mul_(z.mul_(case["phi"]).exp_())


def _inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    m, n, k, pad = case["m"], case["n"], case["k"], case["pad"]
    A, B = _matrix(m, k, pad, case, gen), _matrix(k, n, pad, case, gen)
    R = _matrix(m, n, pad, case, gen) if case["entry"] == "scaled" else None
    return A, B, R


class _Caller:
    """What a program keeps between its calls: a context with its stream and work memory, the operands and the result."""

    def __init__(self, case, seed):
        self.case = case
        self.A, self.B, self.R = _inputs(case, seed)
        self.C = torch.zeros((case["n"], case["m"] + case["pad"]), dtype=torch.float64, device="cuda")
        self.ws = None
        self.context = lib.ozaki_context_create()
        lib.ozaki_context_use(self.context)
        lib.ozaki_set_stream(torch.cuda.current_stream().cuda_stream)
        if case["entry"] != "static":
            self.ws = torch.empty(max(_workspace_bytes(case), 256), dtype=torch.uint8, device="cuda")
            lib.ozaki_set_workspace(self.ws, self.ws.numel())

    def __del__(self):
        if getattr(self, "context", None):
            lib.ozaki_context_destroy(self.context)


def prepare(case, seed):
    return _Caller(case, seed)


def run(state):
    c = state.case
    m, n, k, pad = c["m"], c["n"], c["k"], c["pad"]
    fmt, acc = lib.SLICE_FORMATS[c["fmt"]], lib.ACCUM_MODES[c["accum"]]
    A, B, C = state.A, state.B, state.C
    lib.ozaki_context_use(state.context)
    if c["entry"] == "static":
        lib.ozaki_dgemm_static(m, n, k, A, m + pad, B, k + pad, C, m + pad, fmt, c["s"], c["k_block"], acc)
    elif c["entry"] == "scaled":
        C.copy_(state.R)                                    # the right-hand side stays as it is: C = R - A B
        lib.ozaki_dgemm_scaled(m, n, k, -1.0, A, m + pad, B, k + pad, 1.0, C, m + pad, fmt, c["s"], c["k_block"], acc)
    elif c["entry"] == "ex":
        lib.ozaki_dgemm_ex(m, n, k, A, m + pad, B, k + pad, C, m + pad, fmt, c["s"], c["k_block"], acc, lib.PAIR_SETS[c["pairs"]],
                           lib.SUM_RUNS, 0)
    else:
        lib.ozaki_dgemm(m, n, k, A, m + pad, B, k + pad, C, m + pad, fmt, c["s"], c["k_block"], acc)
    return C[:, :m]


def work(case):
    m, n, k = case["m"], case["n"], case["k"]
    c_passes = 2 if case["entry"] == "scaled" else 1
    return {"bytes": 8.0 * (m * k + k * n + c_passes * m * n), "flops": 2.0 * _pairs(case) * m * n * k}


def tolerance(case):
    return "exact"                                          # the order of every rounding is part of the definition


def exact(case, seed):
    A, B, R = _inputs(case, seed)
    m, k = case["m"], case["k"]
    C = torch.matmul(B[:, :k].contiguous(), A[:, :m].contiguous())
    return C if R is None else R[:, :m] - C
