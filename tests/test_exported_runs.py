"""The product export in the launch configuration of ozaki_dgemm (chained = 2): runs beyond the window's worst case, blocks and
groups as the DGEMM takes them.  Every run joins consecutive pairs of equal scale, its stored word is the exact sum, and no
partial sum leaves the window."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import formats  # noqa: E402
from oracle import ozaki_oracle as oz  # noqa: E402
from paper_2508_00441_amd import binding as lib, device  # noqa: E402
from test_gpu_parity import _as_device_words, _oracle_products, _recipe  # noqa: E402


def export(A, B, fmt, s, k_block, mode, chained, minimum=False):
    """(products, run lengths) as numpy arrays [T][pairs][n][m]"""
    m, k = A.shape
    n = B.shape[1]
    T, npairs = oz.make_plan(k, fmt, k_block).num_blocks, len(oz.pair_order(s, mode))
    Ad, Bd = device.to_device_colmajor(A), device.to_device_colmajor(B)
    ws = device.Workspace.for_problem(m, n, k, lib.SLICE_FORMATS[fmt], s, k_block, pair_set=lib.PAIR_SETS[mode], minimum=minimum)
    P = torch.full((T, npairs, n, m), -77, dtype=torch.int32 if fmt == "int8" else torch.float32, device="cuda")
    L = torch.full((T, npairs, n, m), 99, dtype=torch.uint8, device="cuda")
    lib.ozaki_pair_products(m, n, k, Ad, m, Bd, k, lib.SLICE_FORMATS[fmt], s, k_block, P, pair_set=lib.PAIR_SETS[mode], chained=chained, run_len_out=L)
    assert lib.ozaki_last_device_status() == 0
    ws.close()
    return P.cpu().numpy(), L.cpu().numpy().astype(np.int64)


# fmt, m, n, k, k_block, s, mode, inputs, runs beyond the worst case expected (None: as the groups allow)
CASES = [
    ("fp16", 260, 130, 700, 256, 5, "triangle", "u110", True),     # a pair may fill the window: bounds from the slices
    ("fp16", 130, 70, 2048, 1024, 6, "full", "binade", True),
    ("fp16", 100, 150, 4096, 0, 5, "triangle", "u110", True),      # window of one pair at b = 6
    ("fp16", 100, 150, 2100, 0, 5, "triangle", "u110", True),
    ("fp8", 70, 140, 32768, 0, 7, "triangle", "binade", None),     # window of two pairs: bounds k_block 4^b; few tiles, short groups
    ("fp6", 140, 70, 32768, 0, 7, "triangle", "binade", None),
    ("fp6_e3m2", 70, 40, 65536, 0, 9, "triangle", "binade", None),  # four pairs
    ("fp8", 300, 270, 520, 0, 8, "triangle", "phi1", False),       # windows that hold every anti-diagonal
    ("fp8", 130, 100, 200, 0, 12, "full", "binade", False),
    ("int8", 130, 100, 520, 0, 7, "triangle", "phi1", False),
]


@pytest.mark.parametrize("fmt,m,n,k,k_block,s,mode,recipe,beyond", CASES)
def test_runs_of_the_dgemm_are_exact(fmt, m, n, k, k_block, s, mode, recipe, beyond):
    A, B = _recipe(recipe, m, n, k, seed=m + 2 * n + k)
    plan, blocks = _oracle_products(A, B, fmt, s, k_block, mode)
    pairs = oz.pair_order(s, mode)
    window = formats.EXACT_WINDOW[fmt]
    limit = max(1, min(32, window // (plan.k_block << (2 * plan.b))))
    for minimum in (False, True):                     # all products resident, and one pass per anti-diagonal
        Pn, Ln = export(A, B, fmt, s, k_block, mode, 2, minimum)
        longest = 0
        for t, br in enumerate(blocks):
            covered = np.zeros((len(pairs), n, m), dtype=np.int64)
            for z, (p, q) in enumerate(pairs):
                run = Ln[t, z]
                longest = max(longest, int(run.max()))
                scale = br.c_a[p - 1][None, :] + br.c_b[q - 1][:, None]
                total = np.zeros((n, m), dtype=np.int64)
                for j in range(int(run.max())):
                    inside = run > j
                    pj, qj = pairs[z + j]
                    assert (pj, qj) == (p + j, q - j), (t, z, j)                         # one anti-diagonal, consecutive
                    assert np.array_equal((br.c_a[pj - 1][None, :] + br.c_b[qj - 1][:, None])[inside], scale[inside]), (t, z, j)
                    total += np.where(inside, br.products[z + j].T, 0)
                    assert np.abs(total).max() <= window, (t, z, j)
                    covered[z + j] += inside
                assert np.array_equal(Pn[t, z], _as_device_words(total.T, fmt, plan.b)), (t, z)
            assert covered.min() == 1 and covered.max() == 1, t                          # every pair in exactly one run
        assert beyond is None or (longest > limit) == beyond, (longest, limit)
