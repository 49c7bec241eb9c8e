"""The slice-pair GEMMs' work decomposition (groups of pairs, order of the workgroups, 128 x 128 and 256 x 256 blocks):
every item once, on the host; and C bit-identical to the oracle at the edges of the blocks, on the GPU."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from oracle import ozaki_oracle as oz
from paper_2508_00441_amd import binding as lib, inputs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def host_order(tmp_path_factory):
    out = tmp_path_factory.mktemp("order") / "libhostorder.so"
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-w", "-o", str(out),
                           os.path.join(ROOT, "tests", "host_work_order_harness.cpp")])
    return ctypes.CDLL(str(out))


def test_every_workgroup_takes_one_item(host_order):
    for unit, height in ((0, 0), (32, 8), (32, 4), (64, 8), (64, 4)):
        for bm in (1, 2, 3, 4, 7, 8, 9, 16, 31, 32, 33):
            for bn in (1, 2, 5, 8, 31):
                for groups in (1, 3, 10, 37):
                    assert host_order.work_items_cover(groups, bm, bn, unit, height) == 0, (unit, height, bm, bn, groups)


def test_groups_of_a_pass_hold_every_pair_once(host_order):
    for s in (1, 2, 3, 7, 12, 13, 32):
        for full in (0, 1):
            top = 2 * s if full else s + 1
            for length in sorted({1, 2, 3, 4, 6, s}):
                for g_hi in sorted({top, max(2, top - 1), max(2, s + 1), max(2, s // 2)}):
                    for g_lo in sorted({2, g_hi, max(2, g_hi - 3)}):
                        assert host_order.groups_cover(s, full, length, g_hi, g_lo) == 0, (s, full, length, g_hi, g_lo)


# m, n around the block edges; k of one chunk, an odd and an even number of chunks, a ragged last one.  Which blocks these few
# tiles take is the planner's choice; test_large_blocks_match_oracle has the shapes that take 256 x 256
SHAPES = [(127, 129, 64), (128, 128, 65), (129, 127, 200), (1, 385, 320), (257, 100, 33), (96, 1500, 1000), (520, 500, 2100), (700, 900, 800)]


@pytest.mark.gpu
@pytest.mark.parametrize("fmt", ["fp8", "fp6", "fp6_e3m2", "int8", "fp16"])
@pytest.mark.parametrize("m,n,k", SHAPES)
def test_block_edges_match_oracle(fmt, m, n, k):
    torch = pytest.importorskip("torch")
    from paper_2508_00441_amd import device
    s = 6
    fid = lib.SLICE_FORMATS[fmt]
    A, B = inputs.phi_pair(m, n, k, 2.0, seed=m + 3 * n + k)
    Ad, Bd = device.to_device_colmajor(A), device.to_device_colmajor(B)
    want = {rule: oz.ozaki_dgemm(A, B, fmt, s, 0, accumulate=rule) for rule in ("runs", "plain")}
    for minimum in (False, True):                     # all products resident, and one pass per anti-diagonal
        ws = device.Workspace.for_problem(m, n, k, fid, s, 0, minimum=minimum)
        ws.buf.fill_(0xFF)                            # NaN patterns wherever nothing is written
        ws.buf[:256].zero_()
        for accum, rule in (("hw", "runs"), ("emu", "plain")):
            Cd = torch.full((n, m), float("nan"), dtype=torch.float64, device="cuda")
            print(f"{fmt} {m}x{n}x{k} minimum={minimum} {accum} {rule}", flush=True)
            lib.ozaki_dgemm_ex(m, n, k, Ad, m, Bd, k, Cd, m, fid, s, 0, lib.ACCUM_MODES[accum], lib.PAIRS_TRIANGLE, lib.SUM_RULES[rule], 0)
            assert lib.ozaki_last_device_status() == 0
            got = np.ascontiguousarray(Cd.cpu().numpy().T)
            assert np.array_equal(got.view(np.uint64), want[rule].view(np.uint64)), (minimum, accum, rule)
        ws.close()


@pytest.mark.gpu
@pytest.mark.parametrize("fmt", ["fp8", "fp6", "fp6_e3m2", "int8", "fp16"])
@pytest.mark.parametrize("m,n,k,s,mode", [(4097, 3900, 300, 6, "triangle"), (3969, 4225, 129, 5, "full"), (8191, 2049, 64, 7, "triangle")])
def test_large_blocks_match_oracle(fmt, m, n, k, s, mode):
    """256 x 256 blocks in every format, from 256 tiles on: numbers of 128 x 128 blocks odd (waves without a block to store), odd,
    even and single stages per pair, a ragged last one; strips and the plain order (32 block rows).  Rows and columns from both
    sides of the tile edges are compared: a vector is sliced on its own, so is every entry of the product."""
    torch = pytest.importorskip("torch")
    import planner
    from paper_2508_00441_amd import device
    rng = np.random.default_rng(m + n + k)
    A, B = inputs.phi_pair(m, n, k, 2.0, seed=m + 3 * n + k)
    sample = lambda count: np.unique(np.concatenate([np.arange(0, 3), [127, 128, 255, 256, count - 130, count - 129, count - 1], rng.integers(0, count, 30)]))
    rows, cols = sample(m), sample(n)
    A[m // 2:, :] = np.ldexp(inputs.full_mantissa_one_binade(m - m // 2, k, rng), 3)           # half of the tiles with long runs
    B[:, n // 2:] = inputs.full_mantissa_one_binade(k, n - n // 2, rng)
    Ad, Bd = device.to_device_colmajor(A), device.to_device_colmajor(B)
    fid, ps = lib.SLICE_FORMATS[fmt], lib.PAIR_SETS[mode]
    want = {rule: oz.ozaki_dgemm(A[rows], B[:, cols], fmt, s, 0, mode=mode, accumulate=rule) for rule in ("runs", "plain")}
    for minimum in (False, True):
        assert planner.route(m, n, k, fmt, s, 0, mode, minimum=minimum).small == 0
        ws = device.Workspace.for_problem(m, n, k, fid, s, 0, pair_set=ps, minimum=minimum)
        ws.buf.fill_(0xFF)                            # NaN patterns wherever nothing is written
        ws.buf[:256].zero_()
        for accum, rule in (("hw", "runs"), ("emu", "plain")):
            Cd = torch.full((n, m), float("nan"), dtype=torch.float64, device="cuda")
            print(f"{fmt} {m}x{n}x{k} minimum={minimum} {accum} {rule}", flush=True)
            lib.ozaki_dgemm_ex(m, n, k, Ad, m, Bd, k, Cd, m, fid, s, 0, lib.ACCUM_MODES[accum], ps, lib.SUM_RULES[rule], 0)
            assert lib.ozaki_last_device_status() == 0
            got = Cd[torch.from_numpy(cols).cuda()[:, None], torch.from_numpy(rows).cuda()[None, :]].cpu().numpy().T
            assert np.array_equal(np.ascontiguousarray(got).view(np.uint64), want[rule].view(np.uint64)), (minimum, accum, rule)
            assert bool(torch.isfinite(Cd).all())
        ws.close()


def test_small_block_kernels_use_no_fp64(tmp_path):
    import re
    from test_no_fp64_instructions import F64, HIPCC, _kernel_bodies
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    bodies = {n: b for n, b in _kernel_bodies("pair_gemm_small.hip", tmp_path).items() if "pair_gemm_small_kernel" in n}
    assert len(bodies) == 5
    for body in bodies.values():
        assert "v_mfma_" in body and not re.search(F64, body)
    measured = {n: b for n, b in _kernel_bodies("pair_gemm_measured.hip", tmp_path).items() if "pair_gemm_measured_kernel" in n}
    assert len(measured) == 4
    for body in measured.values():
        assert "v_mfma_" in body and not re.search(F64, body) and "scratch_" not in body      # nothing spilled
    slicing = _kernel_bodies("split.hip", tmp_path)
    for name, count in (("long_exponents_kernel", 1), ("slice_short_kernel", 4)):
        hit = [b for n, b in slicing.items() if name in n]
        assert len(hit) == count and not any(re.search(F64, b) for b in hit)
    fine = {n: b for n, b in _kernel_bodies("accumulate.hip", tmp_path).items() if "accumulate_fine_kernel" in n}
    assert len(fine) == 6
    for name, body in fine.items():
        if "ILi0E" not in name:                          # mode 0 is the hardware FP64 sum
            assert not re.search(F64, body), name


@pytest.mark.gpu
@pytest.mark.parametrize("fmt,m,n,k,s,mode", [("fp8", 130, 70, 100, 20, "triangle"), ("fp8", 65, 97, 200, 12, "full"), ("fp6", 33, 160, 64, 20, "triangle"),
                                              ("int8", 128, 31, 300, 18, "triangle"), ("fp8", 31, 33, 17, 32, "triangle")])
def test_long_groups_of_regular_ladders_match_oracle(fmt, m, n, k, s, mode):
    """One-binade rows (every scale difference the same) with an irregular row and column among them, the last tile partly
    padding: runs as long as the groups, formed from exponents that the GEMM kernel compares itself."""
    torch = pytest.importorskip("torch")
    from paper_2508_00441_amd import device
    rng = np.random.default_rng(m + n + k)
    A = inputs.full_mantissa_one_binade(m, k, rng) * np.where(rng.random((m, k)) < 0.5, -1.0, 1.0) * np.ldexp(1.0, rng.integers(-9, 9, m))[:, None]
    B = inputs.full_mantissa_one_binade(k, n, rng) * np.where(rng.random((k, n)) < 0.5, -1.0, 1.0)
    A[m // 2, :] = inputs.phi_matrix(1, k, 3.0, rng)[0]
    B[:, n - 1] = inputs.phi_matrix(1, k, 3.0, rng)[0]
    Ad, Bd = device.to_device_colmajor(A), device.to_device_colmajor(B)
    fid, ps = lib.SLICE_FORMATS[fmt], lib.PAIR_SETS[mode]
    ws = device.Workspace.for_problem(m, n, k, fid, s, 0, pair_set=ps)
    for accum, rule in (("hw", "runs"), ("emu", "runs"), ("exact", "exact")):
        Cd = torch.full((n, m), float("nan"), dtype=torch.float64, device="cuda")
        lib.ozaki_dgemm_ex(m, n, k, Ad, m, Bd, k, Cd, m, fid, s, 0, lib.ACCUM_MODES[accum], ps, lib.SUM_RUNS, 0)
        assert lib.ozaki_last_device_status() == 0
        want = oz.ozaki_dgemm(A, B, fmt, s, 0, mode=mode, accumulate=rule)
        assert np.array_equal(np.ascontiguousarray(Cd.cpu().numpy().T).view(np.uint64), want.view(np.uint64)), accum
    ws.close()
