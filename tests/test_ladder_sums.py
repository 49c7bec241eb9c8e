"""Products and sums of a tile in one kernel (csrc/ladder_sums.hpp): its branch-free emulated sum against the general one on the host, the calls
that take it, no FP64 instruction in its integer-only forms, and its results bit for bit the oracle's at the edges of tiles, slice
counts, blocks and stages, with vectors that run out and with vectors off the ladder (which leave the call to the other kernels)."""
import ctypes
import os
import re
import subprocess

import numpy as np
import pytest

from oracle import ozaki_oracle as oz
from paper_2508_00441_amd import binding as lib, inputs
import planner
from test_no_fp64_instructions import F64, HIPCC, _kernel_bodies

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FMT, ACC = lib.SLICE_FORMATS, lib.ACCUM_MODES


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    out = tmp_path_factory.mktemp("ladder") / "libladder.so"
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-o", str(out), os.path.join(ROOT, "tests", "host_ladder_add_harness.cpp")])
    return ctypes.CDLL(str(out))


@pytest.mark.parametrize("terms,step,bits,narrow", [(13, 5, 24, 1), (13, 5, 12, 1), (9, 7, 31, 1), (6, 5, 24, 1), (23, 5, 24, 0), (17, 7, 31, 0), (29, 4, 16, 0),
                                                    (23, 5, 3, 0)])
def test_branch_free_sum_equals_the_general_one(host, terms, step, bits, narrow):
    rng = np.random.default_rng(terms * step + bits)
    n = 200000
    v = rng.integers(-(1 << bits) + 1, 1 << bits, (n, terms))
    v = np.where(rng.random((n, terms)) < 0.2, 0, v >> rng.integers(0, bits, (n, terms)))                # zeros, short terms
    cancel = rng.random(n) < 0.5                                                                         # sums that almost vanish on the way
    i = rng.integers(1, terms, n)
    low = v[np.arange(n), i - 1] >> step
    v[cancel, i[cancel]] = -low[cancel] + rng.integers(-1, 2, n)[cancel]
    v = np.ascontiguousarray(v.astype(np.int32))
    a, b = np.empty(n, np.uint64), np.empty(n, np.uint64)
    host.host_ladder_sums(v.ctypes.data_as(ctypes.c_void_p), ctypes.c_size_t(n), terms, -70, step, narrow, a.ctypes.data_as(ctypes.c_void_p),
                          b.ctypes.data_as(ctypes.c_void_p))
    assert np.array_equal(a, b), np.nonzero(a != b)[0][:5]


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
@pytest.mark.parametrize("mode", ["emu", "exact", "hw"])
def test_integer_only_forms_use_no_fp64(tmp_path, mode):
    bodies = {n: b for n, b in _kernel_bodies(f"ladder_sums_int8_{mode}.hip", tmp_path).items() if "ladder_sums_kernel" in n}
    assert len(bodies) >= 6
    for n, body in bodies.items():
        used = set(re.findall(F64, body))
        assert "v_mfma_i32_32x32x32_i8" in body
        assert all(re.match(r"v_(add|ldexp|cvt|mul)_", u) for u in used) if mode == "hw" else not used, (n, used)


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_few_elements_behind_the_pass_are_accumulated_by_forms_for_few(tmp_path):
    """One element per thread (a quarter of the work) also where the vectors turn out to be off the ladder, in every mode, plain and scaled."""
    acc = _kernel_bodies("accumulate.hip", tmp_path)
    for name in ("accumulate_fine_rest_kernel", "accumulate_scaled_fine_rest_kernel"):
        for pint in ("Lb0E", "Lb1E"):
            for mode in (0, 1, 2):
                body = [b for n, b in acc.items() if f"{name}ILi{mode}E{pint}" in n]
                assert len(body) == 1 and (mode == 0 or not re.search(F64, body[0])), (name, mode, pint)


def test_eight_slices_take_the_pass_in_large_results_as_others_do():
    for fmt in ("fp8", "fp6", "int8"):
        assert all(planner.ladder(4096, 4096, k, fmt, s).starts for s in (6, 7, 8, 9) for k in (1024, 4096)), fmt


def test_no_launch_in_front_of_the_pass_for_the_vectors_off_the_ladder():
    """Where a wave can look at all vectors, whether the other kernels use the deltas or not."""
    for m, n, k, fmt, s, pairs, small in ((600, 600, 1000, "fp8", 11, "triangle", 1), (640, 640, 600, "fp6", 13, "triangle", 1), (640, 600, 700, "fp8", 10, "full", 1),
                                          (96, 6000, 4097, "int8", 9, "triangle", 1), (1000, 777, 1301, "fp8", 12, "triangle", 0), (1024, 1024, 1024, "fp8", 11, "full", 0),
                                          (4096, 4096, 1024, "fp6", 13, "triangle", 0)):
        assert planner.route(m, n, k, fmt, s, mode=pairs).small == small
        vectors = sum((x + 255) // 256 * 256 for x in (m, n))
        assert planner.ladder(m, n, k, fmt, s, mode=pairs) == planner.Ladder(1, 0, 1, 0, vectors)
    assert planner.ladder(4096, 4096, 1024, "fp8", 13) == planner.Ladder(1, 64, 1, 0, 8192)                    # up to 64 of each listed
    assert planner.ladder(64, 9000, 600, "fp6", 13) == planner.Ladder(1, 0, 0, 1, 256 + 9216)                  # more vectors than a wave looks at
    assert planner.ladder(600, 8000, 513, "fp8", 6) == planner.Ladder(1, 64, 0, 1, 768 + 8192)
    assert planner.ladder(600, 600, 400, "fp8", 11).starts == 0 and planner.ladder(600, 600, 1000, "fp16", 7).mark_bytes == 0


def _off_ladder(X, fmt, s, k_block):
    """How many rows of X, block by block, have a slice other than zeros more than b + 1 places below the one before."""
    plan, count = oz.make_plan(X.shape[1], fmt, k_block), 0
    for t in range(plan.num_blocks):
        slices, c, _ = oz.slice_rows(X[:, t * plan.k_block:(t + 1) * plan.k_block], plan.rho, s)
        off = np.zeros(len(X), bool)
        for p in range(1, s):
            off |= slices[p].any(axis=1) & (c[p - 1] - c[p] > plan.b + 1)
        count += int(off.sum())
    return count


def _matrices(m, n, k, fmt, s):
    """More slices than a mantissa and the spread of the entries fill would leave the ladder at its end: then a third of the entries lie lower."""
    A, B = inputs.phi_pair(m, n, k, 1.0, seed=m + n + k)
    if s * (oz.make_plan(k, fmt).b + 1) > 66:
        A[:, ::3] *= 2.0 ** -24
        B[::3, :] *= 2.0 ** -24
    return A, B


def _operands(m, n, k, fmt, s, off):
    A, B = _matrices(m, n, k, fmt, s)
    rng = np.random.default_rng(k)
    A[3, :] = 0.0
    A[m - 1, :] = np.ldexp(rng.integers(-7, 8, k).astype(np.float64), -30)             # runs out after a slice or two
    B[:, 1] = np.ldexp(rng.integers(-1000, 1001, k).astype(np.float64), -12)
    B[:, n - 2] *= 2.0 ** 300
    if off in ("A", "both"):
        A[m - 2, :] = 0.0
        A[m - 2, [0, k // 2, k - 1]] = 1.0 + 2.0 ** -50, 3.0 * 2.0 ** -23, -5.0 * 2.0 ** -41
    if off in ("B", "both"):
        B[:, 5] = 0.0
        B[[1, 2], 5] = 1.0, 2.0 ** -19
    return A, B


gpu_cases = pytest.mark.parametrize("fmt,m,n,k,k_block,s,pairs", [
    ("fp8", 513, 577, 512, 0, 13, "triangle"),          # 9 x 10 tiles, ragged; the shortest block, the fewest tiles
    ("fp8", 640, 577, 1031, 0, 6, "triangle"),          # the fewest slices, odd number of stages
    ("fp8", 833, 800, 4600, 0, 14, "triangle"),         # the most; the window's edge; 14 x 13 tiles
    ("fp8", 65, 3000, 600, 0, 8, "triangle"),
    ("fp8", 640, 577, 600, 0, 7, "triangle"),
    ("fp8", 641, 580, 512, 0, 9, "triangle"),
    ("fp8", 1000, 777, 1150, 600, 12, "triangle"),      # two blocks, the second one shorter: the scaled call's product so far is not C
    ("fp8", 512, 770, 1100, 550, 11, "full"),           # two blocks, both halves of the pairs
    ("fp8", 640, 600, 700, 0, 10, "full"),
    ("fp6", 641, 530, 600, 0, 14, "triangle"),
    ("fp6", 640, 580, 1600, 800, 6, "triangle"),
    ("fp6", 640, 580, 600, 0, 10, "triangle"),
    ("fp6", 640, 570, 600, 0, 12, "full"),
    ("fp6_e3m2", 640, 580, 700, 0, 15, "triangle"),
    ("fp6_e3m2", 640, 580, 640, 0, 13, "full"),
    ("fp6_e3m2", 640, 580, 520, 0, 10, "triangle"),
    ("fp6_e3m2", 640, 580, 1300, 650, 12, "triangle"),
    ("int8", 640, 576, 300, 0, 11, "triangle"),
    ("int8", 640, 580, 300, 0, 7, "triangle"),
    ("int8", 640, 580, 580, 290, 8, "triangle"),
    ("int8", 640, 580, 600, 0, 10, "triangle"),
    ("int8", 641, 576, 20000, 0, 6, "triangle"),        # a block that is sliced exponents first
    ("int8", 660, 640, 520, 260, 9, "full"),
    ("int8", 512, 511, 300, 0, 11, "triangle"),         # 64 tiles: the other kernels
])


@pytest.mark.gpu
@pytest.mark.parametrize("off", ["", "A", "both"])
@gpu_cases
def test_results_are_the_oracles(fmt, m, n, k, k_block, s, pairs, off):
    torch = pytest.importorskip("torch")
    from paper_2508_00441_amd import device
    A, B = _operands(m, n, k, fmt, s, off)
    route = planner.ladder(m, n, k, fmt, s, k_block, pairs)
    vectors_off = [_off_ladder(A, fmt, s, k_block), _off_ladder(B.T, fmt, s, k_block)]
    assert route.starts == (min(m, n) != 511) and route.limit == 0
    assert [c > 0 for c in vectors_off] == [off != "", off == "both"]                    # off == "": the one pass does the call
    rows = sorted({0, 3, 31, 32, 63, 64, m // 2, m - 2, m - 1} & set(range(m)))
    cols = sorted({0, 1, 5, 31, 32, 63, 64, n // 2, n - 2, n - 1})
    ldc = m + 3
    Ad, Bd = device.to_device_colmajor(A), device.to_device_colmajor(B)
    ws = device.Workspace(max(lib.ozaki_workspace_bytes_ex(m, n, k, FMT[fmt], s, k_block, lib.PAIR_SETS[pairs], False),
                              lib.ozaki_workspace_bytes_scaled(m, n, k, FMT[fmt], s, k_block)))
    for accum, rule in (("hw", "runs"), ("emu", "runs"), ("exact", "exact")):
        want = oz.ozaki_dgemm(A[rows], B[:, cols], fmt, s, k_block, mode=pairs, accumulate=rule)
        C = torch.full((n, ldc), float("nan"), dtype=torch.float64, device="cuda")
        lib.ozaki_dgemm_ex(m, n, k, Ad, m, Bd, k, C, ldc, FMT[fmt], s, k_block, ACC[accum], lib.PAIR_SETS[pairs], lib.SUM_RUNS, 0)
        assert lib.ozaki_last_device_status() == 0
        if planner.ladder(m, n, k, fmt, s, k_block, pairs, exact=accum == "exact").starts:
            counts = ws.buf[:32].cpu().numpy().view(np.int32)[4:6].tolist()
            assert (sum(counts) > 0) == (sum(vectors_off) > 0), counts                     # the kernels' choice rests on these
        got = C.cpu().numpy()
        assert np.all(np.isnan(got[:, m:])) and not np.any(np.isnan(got[:, :m]))
        part = np.ascontiguousarray(got[:, :m].T[np.ix_(rows, cols)])
        assert np.array_equal(part.view(np.uint64), want.view(np.uint64)), accum
        if pairs == "triangle":
            # scaled: one rounding per operation on the plain product, on C as it is
            C0 = inputs.phi_matrix(n, ldc, 2.0, np.random.default_rng(m * n))
            D = torch.from_numpy(C0).cuda()
            lib.ozaki_dgemm_scaled(m, n, k, -1.5, Ad, m, Bd, k, 0.3, D, ldc, FMT[fmt], s, k_block, ACC[accum])
            assert lib.ozaki_last_device_status() == 0
            scaled = D.cpu().numpy()
            assert np.array_equal(scaled[:, m:], C0[:, m:])
            assert np.array_equal(np.ascontiguousarray(scaled[:, :m]).view(np.uint64), (-1.5 * got[:, :m] + 0.3 * C0[:, :m]).view(np.uint64)), accum
    ws.close()


LARGE = [("fp8", 2050, 2082, 513, 13), ("fp8", 1100, 4000, 640, 6), ("int8", 2049, 2050, 261, 9)]
# The other slice counts that have a kernel, each with a table of its own and from 11 on products in ordinary registers
OTHERS = [("fp8", 2049, 2050, 513, s) for s in range(7, 13)] + [("int8", 2050, 2049, 261 + 64 * (s % 2), s) for s in (6, 7, 8, 10, 11)]


@pytest.mark.gpu
@pytest.mark.parametrize("fmt,m,n,k,s,rows_off,cols_off", [c + o for c in LARGE for o in ((0, 0), (1, 0), (0, 33), (32, 3), (64, 64), (65, 1), (2, 65))] +
                         [c + (33, 2) for c in OTHERS] + [("fp8", 600, 8000, 513, 6) + o for o in ((0, 0), (33, 64), (65, 1))])      # counted by a launch of its own
def test_vectors_off_the_ladder_in_large_results(fmt, m, n, k, s, rows_off, cols_off):
    """Up to 64 of each operand are done by a kernel of their own, more leave the call to the general kernels; plain and scaled."""
    torch = pytest.importorskip("torch")
    from paper_2508_00441_amd import device
    A, B = _matrices(m, n, k, fmt, s)
    assert planner.ladder(m, n, k, fmt, s)[:2] == (1, 64)
    rng = np.random.default_rng(rows_off * 100 + cols_off)
    odd_rows, odd_cols = rng.permutation(m)[:rows_off], rng.permutation(n)[:cols_off]
    for X, at in ((A, odd_rows), (B.T, odd_cols)):
        X[at, :] = 0.0
        for i in at:
            X[i, rng.permutation(k)[:3]] = 1.0 + 2.0 ** -50, 3.0 * 2.0 ** -23, -5.0 * 2.0 ** -41
    rows = sorted({0, 31, 32, m - 1} | set(odd_rows[:6].tolist()))
    cols = sorted({0, 63, 64, n - 1} | set(odd_cols[:6].tolist()))
    Ad, Bd = device.to_device_colmajor(A), device.to_device_colmajor(B)
    ws = torch.zeros(lib.ozaki_workspace_bytes_scaled(m, n, k, FMT[fmt], s, 0), dtype=torch.uint8, device="cuda")
    lib.ozaki_set_stream(torch.cuda.current_stream().cuda_stream)
    lib.ozaki_set_workspace(ws, ws.numel())
    C0 = inputs.phi_matrix(n, m, 2.0, np.random.default_rng(m * n))
    for accum, rule in (("hw", "runs"), ("emu", "runs"), ("exact", "exact")):
        want = oz.ozaki_dgemm(A[rows], B[:, cols], fmt, s, 0, accumulate=rule)
        C = torch.full((n, m), float("nan"), dtype=torch.float64, device="cuda")
        lib.ozaki_dgemm(m, n, k, Ad, m, Bd, k, C, m, FMT[fmt], s, 0, ACC[accum])
        assert lib.ozaki_last_device_status() == 0
        counts = ws[:32].cpu().numpy().view(np.int32)[4:6].tolist()
        assert counts == [rows_off, cols_off], counts                                # the kernels' choice rests on these
        got = C.cpu().numpy()
        assert not np.any(np.isnan(got))
        part = np.ascontiguousarray(got.T[np.ix_(rows, cols)])
        assert np.array_equal(part.view(np.uint64), want.view(np.uint64)), accum
        D = torch.from_numpy(C0).cuda()
        lib.ozaki_dgemm_scaled(m, n, k, -1.5, Ad, m, Bd, k, 0.3, D, m, FMT[fmt], s, 0, ACC[accum])
        assert lib.ozaki_last_device_status() == 0
        assert np.array_equal(D.cpu().numpy().view(np.uint64), (-1.5 * got + 0.3 * C0).view(np.uint64)), accum
    lib.ozaki_set_workspace(None, 0)


@pytest.mark.gpu
@pytest.mark.parametrize("fmt,m,n,k,k_block,s", [("fp8", 640, 577, 600, 0, 11), ("int8", 640, 577, 600, 300, 9), ("fp6", 700, 600, 1200, 0, 13),
                                                 ("int8", 600, 640, 20000, 0, 7), ("fp8", 2050, 2082, 513, 0, 13)])
@pytest.mark.parametrize("scale", [0, 20, -300])
def test_vectors_that_run_out_are_on_the_ladder_at_any_scale(fmt, m, n, k, k_block, s, scale):
    """Integers of ten bits times a power of two, whose later slices are zeros; a vector that runs out behind a gap is off the ladder, also where the
    slice behind the gap has the exponent of one without a remainder (zero)."""
    torch = pytest.importorskip("torch")
    from paper_2508_00441_amd import device
    rng = np.random.default_rng(m + k)
    A, B = (np.ldexp(rng.integers(-1000, 1001, shape).astype(np.float64), scale) for shape in ((m, k), (k, n)))
    rows, cols = [0, 7, 63, 64, m - 1], [0, 5, 63, 64, n - 1]
    f = FMT[fmt]
    ws = torch.zeros(lib.ozaki_workspace_bytes_scaled(m, n, k, f, s, k_block), dtype=torch.uint8, device="cuda")
    lib.ozaki_set_stream(torch.cuda.current_stream().cuda_stream)
    lib.ozaki_set_workspace(ws, ws.numel())
    for gap in (False, True):
        if gap:
            A[7, :] = 0.0
            A[7, [1, k - 1]] = 2.0 ** 20, 1.0
        want = oz.ozaki_dgemm(A[rows], B[:, cols], fmt, s, k_block, accumulate="runs")
        C = torch.full((n, m), float("nan"), dtype=torch.float64, device="cuda")
        lib.ozaki_dgemm(m, n, k, device.to_device_colmajor(A), m, device.to_device_colmajor(B), k, C, m, f, s, k_block, ACC["emu"])
        assert lib.ozaki_last_device_status() == 0
        counts = ws[:32].cpu().numpy().view(np.int32)[4:6].tolist()
        got = np.ascontiguousarray(C.cpu().numpy().T[np.ix_(rows, cols)])
        assert np.array_equal(got.view(np.uint64), want.view(np.uint64))
        off = gap and k_block == 0                                    # (in two blocks the row's entries lie in different ones)
        assert counts == [int(off), 0], counts
    lib.ozaki_set_workspace(None, 0)


@pytest.mark.gpu
@pytest.mark.parametrize("fmt,m,n,k,s,pairs", [("fp8", 640, 600, 700, 10, "full"), ("int8", 2049, 2050, 261, 9, "triangle"), ("fp8", 600, 8000, 513, 6, "triangle")])
def test_a_captured_call_decides_anew_on_every_replay(fmt, m, n, k, s, pairs):
    """None off the ladder, a few, too many, none again: counted by the pass itself, with a list, and by a launch in front."""
    torch = pytest.importorskip("torch")
    from paper_2508_00441_amd import device
    A, B = _matrices(m, n, k, fmt, s)
    Ad, Bd = device.to_device_colmajor(A), device.to_device_colmajor(B)
    C = torch.zeros((n, m), dtype=torch.float64, device="cuda")
    f, ps = FMT[fmt], lib.PAIR_SETS[pairs]
    ws = torch.zeros(lib.ozaki_workspace_bytes_ex(m, n, k, f, s, 0, ps, False), dtype=torch.uint8, device="cuda")
    call = lambda: lib.ozaki_dgemm_ex(m, n, k, Ad, m, Bd, k, C, m, f, s, 0, ACC["emu"], ps, lib.SUM_RUNS, 0)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        lib.ozaki_set_stream(side.cuda_stream)
        lib.ozaki_set_workspace(ws, ws.numel())
        call()
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            call()
        rows, cols = [0, 1, 31, 64, m - 1], [0, 63, n - 1]
        whole = Ad.clone()
        for count in (0, 3, 80, 0, 3):
            Ad.copy_(whole)
            if count:
                Ad[:, :count] *= 2.0 ** -45
                Ad[5, :count] = 3.0
            C.fill_(float("nan"))
            graph.replay()
            side.synchronize()
            got = C.clone()
            counts = ws[:32].cpu().numpy().view(np.int32)[4:6].tolist()
            assert (counts[0] > 0) == (count > 0) and counts[1] == 0, counts
            want = oz.ozaki_dgemm(device.from_device_colmajor(Ad)[rows], B[:, cols], fmt, s, 0, mode=pairs, accumulate="runs")
            assert np.array_equal(np.ascontiguousarray(got.cpu().numpy().T[np.ix_(rows, cols)]).view(np.uint64), want.view(np.uint64)), count
            C.fill_(float("nan"))
            call()
            side.synchronize()
            assert torch.equal(got.view(torch.int64), C.view(torch.int64)), count
        lib.ozaki_set_workspace(None, 0)
    lib.ozaki_set_stream(torch.cuda.current_stream().cuda_stream)
