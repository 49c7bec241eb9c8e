"""Blocks of at most 256 elements (four elements per lane): codes and exponents bit-identical to the oracle, at the edges of the
lanes and chunks, for whole operands and blocked ones, contiguous vectors and rows of a column-major matrix."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import ozaki_oracle as oz  # noqa: E402
from paper_2508_00441_amd import inputs  # noqa: E402
from test_gpu_parity import _gpu_split  # noqa: E402


@pytest.mark.parametrize("fmt", ["fp8", "fp6", "fp6_e3m2", "int8"])
@pytest.mark.parametrize("rows,k,k_block", [(12, 16, 0), (300, 63, 0), (12, 64, 0), (70, 65, 0), (13, 129, 0), (257, 255, 0), (12, 256, 0), (12, 700, 256),
                                            (33, 500, 100), (20, 257, 256)])
def test_short_blocks_are_bit_exact(fmt, rows, k, k_block):
    X = inputs.nasty_rows(np.random.default_rng(rows + k), rows, k)
    s = 14
    ref_codes, ref_exps, plan = oz.split_operand(X, fmt, s, k_block)
    for is_B in (0, 1):
        got_codes, got_exps = _gpu_split(X, is_B, fmt, s, k_block)
        for t in range(plan.num_blocks):
            for p in range(s):
                assert np.array_equal(got_exps[t][p], ref_exps[t][p]), (is_B, t, p)
                assert np.array_equal(got_codes[t][p], ref_codes[t][p]), (is_B, t, p)
