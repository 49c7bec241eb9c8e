"""Vector lengths at the edges of the slicing kernel's thread and octet ranges (a wave without elements in its second octet,
fewer waves than the widest, whole workgroups of padding vectors) and rows 8 bytes off a 16-byte boundary: codes and
exponents bit-identical to the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import ozaki_oracle as oz  # noqa: E402
from paper_2508_00441_amd import inputs  # noqa: E402
from test_gpu_parity import _gpu_split  # noqa: E402


@pytest.mark.parametrize("fmt", ["fp8", "fp6", "fp6_e3m2", "int8", "fp16"])
@pytest.mark.parametrize("rows,k", [(3, 511), (5, 513), (7, 1025), (2, 1537), (3, 2047), (3, 2049), (2300, 1025), (2300, 2049), (2100, 4097), (4, 4608),
                                    (3, 8193), (2, 8705), (2, 16383)])
def test_lengths_at_the_thread_edges(fmt, rows, k):
    X = inputs.phi_matrix(rows, k, 2.0, np.random.default_rng(rows + k))
    X[0, k - 1] = 2.0 ** 30                                  # the maximum sits in the last place
    s = 5
    ref_codes, ref_exps, _ = oz.split_operand(X, fmt, s, 0)
    for is_B in (0, 1):
        got_codes, got_exps = _gpu_split(X, is_B, fmt, s, 0)
        for p in range(s):
            assert np.array_equal(got_exps[0][p], ref_exps[0][p]), (is_B, p)
            assert np.array_equal(got_codes[0][p], ref_codes[0][p]), (is_B, p)


@pytest.mark.parametrize("fmt", ["fp8", "fp6", "fp6_e3m2", "int8", "fp16"])
@pytest.mark.parametrize("k", [12289, 16384])
def test_many_vectors_at_sixteen_elements_per_thread(fmt, k):
    """The longest blocks that stay in registers, with more workgroups than the chip holds at once."""
    X = inputs.phi_matrix(24, k, 2.0, np.random.default_rng(k))
    X[5, :] = np.where(np.arange(k) % 4000 == 7, X[5, :], 0.0)
    X[6, :] *= np.ldexp(1.0, -(np.arange(k) // 200))
    s, rows = 4, 2050
    ref_codes, ref_exps, _ = oz.split_operand(X, fmt, s, 0)
    which = np.arange(rows) % 24
    got_codes, got_exps = _gpu_split(np.ascontiguousarray(X[which]), 1, fmt, s, 0)
    for p in range(s):
        assert np.array_equal(got_exps[0][p], ref_exps[0][p][which]), p
        assert np.array_equal(got_codes[0][p], ref_codes[0][p][which]), p
