"""Runs beyond the window's worst case, in the launch configuration of ozaki_dgemm (product export with chained = 2) and in the DGEMM
itself.  The cases take the route that they are for, which the planner says on the host: 256 x 256 or 128 x 128 blocks, groups
longer than the worst case allows, bounds from the slices or the same for every pair.  One half of the vectors are regular
(long runs must form), the other half have slices that fill the window (runs must break).  Sampled rows and columns from both
halves and from the edges are compared with the oracle: a vector is sliced on its own, so is every entry of the product."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import planner  # noqa: E402
from oracle import formats  # noqa: E402
from oracle import ozaki_oracle as oz  # noqa: E402
from paper_2508_00441_amd import binding as lib, device  # noqa: E402
from test_gpu_parity import _as_device_words, _recipe  # noqa: E402


def _vectors(count, k, b, gen):
    """count x k: regular vectors (one binade, full significands, random signs), from count // 2 on vectors whose slices are all
    +-2^b: 1 - 2^-(b+1) + 2^-2(b+1) - ..., a tie at every slice that rounds up to 2^b; every third of those cancels half way."""
    X = (torch.randint(0, 1 << 52, (count, k), generator=gen, device="cuda") | (1023 << 52)).view(torch.float64)
    X *= torch.randint(0, 2, (count, k), generator=gen, device="cuda", dtype=torch.int8) * 2 - 1
    half = count // 2
    X[half:] = sum((-1.0) ** i * 2.0 ** (-i * (b + 1)) for i in range(5))
    X[half + 2::3, : k // 2] *= -1.0
    return X


def _sample(count, rng):
    half = count // 2
    fixed = [0, min(31, half - 1), half - 1, half, count - 1]
    return np.unique(fixed + list(rng.integers(0, half, 9)) + list(rng.integers(half, count, 9)))


def check_export(Pn, Ln, Ah, Bh, fmt, s, k_block, mode, counted):
    """Words and run lengths [T][pairs][n][m] of the columns of Bh and the rows of Ah: every run joins consecutive pairs of one
    anti-diagonal and equal scale, its word is the exact sum, no partial sum leaves the window, every pair is in one run.
    Returns the longest run among the entries `counted` and the largest sum."""
    plan = oz.make_plan(Ah.shape[1], fmt, k_block)
    pairs, window = oz.pair_order(s, mode), formats.EXACT_WINDOW[fmt]
    _, blocks = oz.ozaki_dgemm(Ah, Bh, fmt, s, k_block, mode=mode, return_blocks=True)
    longest = largest = 0
    for t, br in enumerate(blocks):
        covered = np.zeros(Ln.shape[1:], dtype=np.int64)
        for z, (p, q) in enumerate(pairs):
            run = Ln[t, z]
            longest = max(longest, int(run[counted].max()))
            scale = br.c_a[p - 1][None, :] + br.c_b[q - 1][:, None]
            total = np.zeros(run.shape, dtype=np.int64)
            for j in range(int(run.max())):
                inside = run > j
                pj, qj = pairs[z + j]
                assert (pj, qj) == (p + j, q - j), (t, z, j)
                assert np.array_equal((br.c_a[pj - 1][None, :] + br.c_b[qj - 1][:, None])[inside], scale[inside]), (t, z, j)
                total += np.where(inside, br.products[z + j].T, 0)
                assert np.abs(total).max() <= window, (t, z, j)
                covered[z + j] += inside
            largest = max(largest, int(np.abs(total).max()))
            assert np.array_equal(Pn[t, z], _as_device_words(total.T, fmt, plan.b)), (t, z)
        assert covered.min() == 1 and covered.max() == 1, t
    return longest, largest


# format, m, n, k, k_block, s, mode, 128 x 128 blocks?, bounds from the slices?
BEYOND = [
    ("fp16", 700, 650, 600, 256, 7, "triangle", 1, 1), ("fp16", 1300, 1200, 1024, 0, 7, "full", 0, 1), ("fp16", 1300, 1200, 2048, 0, 7, "full", 0, 0),
    ("fp16", 2900, 380, 2048, 0, 9, "full", 1, 0), ("fp16", 2100, 1100, 4096, 0, 8, "full", 0, 1),
    ("fp8", 2010, 1900, 32768, 0, 7, "triangle", 0, 0), ("fp8", 900, 120, 32768, 0, 11, "triangle", 1, 0), ("fp8", 100, 2600, 32768, 0, 7, "full", 1, 0),
    ("fp6", 2010, 1900, 32768, 0, 7, "triangle", 0, 0), ("fp6", 900, 120, 32768, 0, 11, "triangle", 1, 0),
    ("fp6_e3m2", 3000, 384, 65536, 0, 11, "full", 0, 0), ("fp6_e3m2", 100, 2600, 131072, 0, 7, "full", 1, 0),
]


@pytest.mark.parametrize("fmt,m,n,k,k_block,s,mode,small,from_slices", BEYOND)
def test_runs_beyond_the_worst_case(fmt, m, n, k, k_block, s, mode, small, from_slices):
    way = planner.route(m, n, k, fmt, s, k_block, mode)
    assert way.measured and way.small == small and way.bounds_from_slices == from_slices and way.group_len > way.run_limit, way
    assert from_slices == (way.run_limit == 1)
    plan = oz.make_plan(k, fmt, k_block)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(m + 2 * n + k)
    A, Bt = _vectors(m, k, plan.b, gen), _vectors(n, k, plan.b, gen)
    rng = np.random.default_rng(k)
    rows, cols = _sample(m, rng), _sample(n, rng)
    Ah, Bh = A[torch.from_numpy(rows).cuda()].cpu().numpy(), Bt[torch.from_numpy(cols).cuda()].cpu().numpy().T.copy()
    pick = (torch.from_numpy(cols).cuda()[:, None], torch.from_numpy(rows).cuda()[None, :])
    Ad = A.T.contiguous()
    del A
    fid, ps = lib.SLICE_FORMATS[fmt], lib.PAIR_SETS[mode]
    ws = device.Workspace.for_problem(m, n, k, fid, s, k_block, pair_set=ps)
    C = {}
    for accum in ("hw", "exact"):
        Cd = torch.full((n, m), float("nan"), dtype=torch.float64, device="cuda")
        print(f"{fmt} {m}x{n}x{k} {accum}", flush=True)
        lib.ozaki_dgemm_ex(m, n, k, Ad, m, Bt, k, Cd, m, fid, s, k_block, lib.ACCUM_MODES[accum], ps, lib.SUM_RUNS, 0)
        assert lib.ozaki_last_device_status() == 0
        C[accum] = Cd[pick].cpu().numpy().T
    pairs = oz.pair_order(s, mode)
    P = torch.full((plan.num_blocks, len(pairs), n, m), -77.0, dtype=torch.float32, device="cuda")
    L = torch.full((plan.num_blocks, len(pairs), n, m), 99, dtype=torch.uint8, device="cuda")
    print(f"{fmt} {m}x{n}x{k} export", flush=True)
    lib.ozaki_pair_products(m, n, k, Ad, m, Bt, k, fid, s, k_block, P, pair_set=ps, chained=2, run_len_out=L)
    assert lib.ozaki_last_device_status() == 0
    Pn, Ln = P[:, :, pick[0], pick[1]].cpu().numpy(), L[:, :, pick[0], pick[1]].cpu().numpy().astype(np.int64)
    ws.close()

    for accum, rule in (("hw", "runs"), ("exact", "exact")):
        want = oz.ozaki_dgemm(Ah, Bh, fmt, s, k_block, mode=mode, accumulate=rule)
        assert np.array_equal(np.ascontiguousarray(C[accum]).view(np.uint64), want.view(np.uint64)), accum
    regular = np.outer(cols < n // 2 // 32 * 32, rows < m // 2 // 32 * 32)            # 32 x 32 tiles of regular vectors only
    longest, largest = check_export(Pn, Ln, Ah, Bh, fmt, s, k_block, mode, regular)
    assert longest > way.run_limit, (longest, way)
    assert 2 * largest >= formats.EXACT_WINDOW[fmt], largest                         # sums that fill the window were there


@pytest.mark.parametrize("fmt,m,n,k,s,mode", [("int8", 257, 100, 3000, 8, "full"), ("fp8", 130, 70, 8192, 12, "triangle"), ("fp16", 70, 130, 512, 5, "triangle")])
def test_runs_of_the_worst_case_are_as_long_as_it_allows(fmt, m, n, k, s, mode):
    """chained = 1: groups of as many pairs as surely fit the window, whatever groups the DGEMM would take."""
    plan = oz.make_plan(k, fmt, 0)
    limit = max(1, min(s, formats.EXACT_WINDOW[fmt] // (plan.k_block << (2 * plan.b))))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(k)
    A, Bt = _vectors(m, k, plan.b, gen), _vectors(n, k, plan.b, gen)
    Ad = A.T.contiguous()
    pairs = oz.pair_order(s, mode)
    for minimum in (False, True):
        ws = device.Workspace.for_problem(m, n, k, lib.SLICE_FORMATS[fmt], s, 0, pair_set=lib.PAIR_SETS[mode], minimum=minimum)
        P = torch.empty((1, len(pairs), n, m), dtype=torch.float32, device="cuda")
        L = torch.full((1, len(pairs), n, m), 99, dtype=torch.uint8, device="cuda")
        lib.ozaki_pair_products(m, n, k, Ad, m, Bt, k, lib.SLICE_FORMATS[fmt], s, 0, P, pair_set=lib.PAIR_SETS[mode], chained=1, run_len_out=L)
        assert lib.ozaki_last_device_status() == 0
        ws.close()
        regular = L[0, :, : n // 2 // 32 * 32, : m // 2 // 32 * 32].amax(dim=(1, 2)).cpu().numpy()
        for z, (p, q) in enumerate(pairs):
            first = p - max(1, p + q - s)                      # position in the anti-diagonal
            left = min(s, p + q - 1) - p + 1                   # pairs from here to its end
            if first % limit == 0:
                assert 1 <= regular[z] <= min(limit, left), (z, p, q)
        assert regular.max() == limit, (regular.max(), limit)


@pytest.mark.parametrize("fmt,m,n,k,k_block,s,mode,recipe", [
    ("fp8", 300, 270, 520, 0, 8, "triangle", "phi4"), ("fp8", 130, 100, 200, 0, 12, "full", "binade"), ("fp6", 257, 130, 1000, 384, 9, "full", "u110"),
    ("fp6_e3m2", 130, 300, 64, 0, 14, "triangle", "binade"), ("int8", 130, 257, 300, 0, 8, "full", "binade"), ("fp16", 260, 130, 700, 256, 5, "triangle", "u110")])
def test_groups_of_the_dgemm(fmt, m, n, k, k_block, s, mode, recipe):
    """chained = 2 on few tiles: links that the 128 x 128 kernel forms from the exponents, irregular vectors among regular ones, one
    pass and several."""
    A, B = _recipe(recipe, m, n, k, seed=m + 2 * n + k)
    Ad, Bd = device.to_device_colmajor(A), device.to_device_colmajor(B)
    fid, ps = lib.SLICE_FORMATS[fmt], lib.PAIR_SETS[mode]
    shape = (oz.make_plan(k, fmt, k_block).num_blocks, len(oz.pair_order(s, mode)), n, m)
    for minimum in (False, True):
        assert planner.route(m, n, k, fmt, s, k_block, mode, minimum=minimum).small
        ws = device.Workspace.for_problem(m, n, k, fid, s, k_block, pair_set=ps, minimum=minimum)
        P = torch.full(shape, -77, dtype=torch.int32 if fmt == "int8" else torch.float32, device="cuda")
        L = torch.full(shape, 99, dtype=torch.uint8, device="cuda")
        lib.ozaki_pair_products(m, n, k, Ad, m, Bd, k, fid, s, k_block, P, pair_set=ps, chained=2, run_len_out=L)
        assert lib.ozaki_last_device_status() == 0
        ws.close()
        check_export(P.cpu().numpy(), L.cpu().numpy().astype(np.int64), A, B, fmt, s, k_block, mode, np.ones((n, m), dtype=bool))
