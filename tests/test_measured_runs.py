"""Block lengths and slice counts around the window: inputs whose products fill it exactly, random ones, every route to the
accumulation.  These problems have few tiles, so that the planner mostly keeps their groups within the worst case; the
cases whose groups pass it, so that the accumulators are looked at, are in test_exported_runs.py."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import ozaki_oracle as oz  # noqa: E402
from paper_2508_00441_amd import binding as lib, device, inputs  # noqa: E402


def _run(A, B, fmt, s, kb, accum, pairs, minimum=False):
    m, k = A.shape
    n = B.shape[1]
    fid = lib.SLICE_FORMATS[fmt]
    Ad, Bd = device.to_device_colmajor(A), device.to_device_colmajor(B)
    Cd = torch.full((n, m), float("nan"), dtype=torch.float64, device="cuda")
    ws = device.Workspace.for_problem(m, n, k, fid, s, kb, pair_set=lib.PAIR_SETS[pairs], minimum=minimum)
    lib.ozaki_dgemm_ex(m, n, k, Ad, m, Bd, k, Cd, m, fid, s, kb, lib.ACCUM_MODES[accum], lib.PAIR_SETS[pairs], lib.SUM_RUNS, 0)
    assert lib.ozaki_last_device_status() == 0
    ws.close()
    return np.ascontiguousarray(Cd.cpu().numpy().T)


def _check(A, B, fmt, s, kb, accum, pairs):
    want = oz.ozaki_dgemm(A, B, fmt, s, kb, mode=pairs, accumulate="exact" if accum == "exact" else "runs")
    for minimum in (False, True):
        got = _run(A, B, fmt, s, kb, accum, pairs, minimum)
        assert np.array_equal(got.view(np.uint64), want.view(np.uint64)), minimum


def _full_slices(rows, k, b, count, rng):
    """Entries whose slices are all +-2^b: 1 - 2^-(b+1) + 2^-2(b+1) - ..., a tie at every slice that rounds up to 2^b."""
    v = sum((-1.0) ** i * 2.0 ** (-i * (b + 1)) for i in range(count))
    X = np.full((rows, k), v)
    X[1::3] *= np.where(rng.random((len(X[1::3]), k)) < 0.5, 1.0, -1.0)       # some rows that cancel
    X[2::3, ::2] *= -1.0
    return X


@pytest.mark.parametrize("fmt,k,kb,b", [("fp16", 1024, 0, 7), ("fp16", 4096, 1024, 7), ("fp16", 4096, 0, 6), ("fp16", 2048, 0, 6), ("fp16", 1500, 0, 6),
                                        ("fp8", 32768, 0, 4), ("fp8", 16384, 0, 4), ("fp6", 16384, 0, 4), ("fp6_e3m2", 65536, 0, 3)])
def test_products_that_fill_the_window(fmt, k, kb, b):
    assert oz.make_plan(k, fmt, kb).b == b
    rng = np.random.default_rng(k)
    A, B = _full_slices(70, k, b, 5, rng), _full_slices(40, k, b, 5, rng).T.copy()
    for pairs in ("triangle", "full"):
        _check(A, B, fmt, 5, kb, "emu", pairs)


@pytest.mark.parametrize("fmt,m,n,k,kb,s,dist,accum,pairs", [
    ("fp16", 300, 270, 2048, 1024, 8, "phi", "hw", "triangle"), ("fp16", 129, 400, 3000, 1024, 7, "u110", "emu", "full"),
    ("fp16", 260, 130, 1100, 512, 7, "u110", "exact", "full"), ("fp16", 200, 200, 20000, 0, 9, "phi", "hw", "triangle"),
    ("fp16", 70, 1000, 700, 100, 6, "phi", "hw", "triangle"), ("fp16", 1000, 20, 64, 16, 6, "phi", "emu", "triangle"),
    ("fp8", 200, 150, 16384, 0, 11, "u110", "hw", "full"), ("fp8", 300, 270, 9000, 0, 13, "phi", "emu", "triangle"),
    ("fp6", 130, 300, 8192, 0, 13, "phi", "exact", "triangle"), ("fp6_e3m2", 64, 64, 70000, 0, 12, "u110", "emu", "triangle"),
    ("fp16", 1700, 1600, 1024, 0, 4, "u110", "hw", "full"), ("fp8", 1500, 1300, 16384, 0, 6, "phi", "hw", "triangle")])
def test_long_runs_match_oracle(fmt, m, n, k, kb, s, dist, accum, pairs):
    rng = np.random.default_rng(m + n + k)
    if dist == "u110":
        A, B = inputs.uniform_1_10(m, k, rng), inputs.uniform_1_10(k, n, rng)
    else:
        A, B = inputs.phi_pair(m, n, k, 2.0, seed=m + n + k)
    _check(A, B, fmt, s, kb, accum, pairs)
