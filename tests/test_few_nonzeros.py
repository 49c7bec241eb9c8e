"""Vectors whose units leave the regular ladder at every other slice (few non-zero elements, narrow bands, lone outliers hundreds of
binades away) through every form of the slicing kernels: codes and exponents bit-identical to the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import ozaki_oracle as oz  # noqa: E402
from test_gpu_parity import _gpu_split  # noqa: E402


def _sparse_rows(k, seed):
    rng = np.random.default_rng(seed)
    X = np.zeros((14, k))
    for r, nonzeros in enumerate((0, 1, 1, 1, 2, 2, 3, 4, 8, 16)):
        at = rng.permutation(k)[:nonzeros]
        X[r, at] = (rng.random(at.size) - 0.5) * np.exp(rng.normal(0.0, 2.0, at.size))
    X[10, k // 2 : k // 2 + 5] = rng.normal(size=5)                       # a band
    X[11, [0, k - 1]] = 1.0 + rng.random(2)                              # below the 96 bits of the number: two of them, three
    X[11, k - 1] *= 2.0 ** -70
    X[12, [0, k // 3, k - 1]] = np.ldexp(1.0 + rng.random(3), [400, 20, -300])
    X[13, [1, k - 2]] = np.ldexp(1.0 + rng.random(2), [-1020, -1068])      # down to subnormal numbers
    return X


# one wave per vector with four elements per lane, with eight, workgroups of 2 .. 16 waves, sixteen elements per thread, streamed blocks
@pytest.mark.parametrize("fmt", ["fp8", "fp6", "fp6_e3m2", "int8", "fp16"])
@pytest.mark.parametrize("k,k_block", [(100, 0), (300, 0), (1000, 0), (1000, 60), (1900, 0), (4000, 0), (6100, 0), (8000, 0), (12200, 0), (16384, 0), (20000, 0)])
def test_units_off_the_ladder(fmt, k, k_block):
    X = _sparse_rows(k, 900 + k)
    s = 20
    ref_codes, ref_exps, plan = oz.split_operand(X, fmt, s, k_block)
    for is_B in (0, 1):
        got_codes, got_exps = _gpu_split(X, is_B, fmt, s, k_block)
        for t in range(plan.num_blocks):
            for p in range(s):
                assert np.array_equal(got_exps[t][p], ref_exps[t][p]), (is_B, t, p)
                assert np.array_equal(got_codes[t][p], ref_codes[t][p]), (is_B, t, p)
