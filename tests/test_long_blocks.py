"""Slicing of blocks beyond the register-resident kernel: the exponents of all slices come from readings of the block that
follow the regular ladder of units as far as it holds.  The vectors here leave the ladder in every way: remainders that
vanish, that are exact powers of two, that lie more than 32 bits below the unit, lone elements, wide outliers."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import ozaki_oracle as oz  # noqa: E402
from paper_2508_00441_amd import binding as lib, inputs  # noqa: E402
from test_gpu_parity import _gpu_split  # noqa: E402


def _vectors(k, rng):
    X = inputs.nasty_rows(rng, 24, k)
    X[9, :] = 1.0 + 2.0 ** -45                                # after the first slice every remainder is 2^-45
    X[10, :] = 0.0
    X[10, k - 1] = 1.0 + 2.0 ** -50                           # one element, in the last place of the block
    X[11, :] = 0.0
    X[11, 17] = 2.0 ** -1030                                  # one subnormal
    X[12, :] = np.where(rng.random(k) < 0.5, 1.0, 2.0 ** -40)             # remainders that are powers of two, 40 bits down
    X[13, :] = 1.0
    X[13, 5] = 1.0 + 2.0 ** -33 + 2.0 ** -52                  # just above a power of two in the upper word of the key
    X[14, :] = np.ldexp(1.0, -rng.integers(0, 600, k))        # powers of two over 600 binades
    X[15, :] = inputs.phi_matrix(1, k, 12.0, rng)[0]          # very wide
    X[16, :] = 3.0
    X[16, ::2] = -3.0 * 2.0 ** -60
    X[17, :] = np.nextafter(1.0, 0.0)
    X[18, :] = 2.0 ** 900
    X[18, 3] = 2.0 ** -1000
    return X


@pytest.mark.parametrize("fmt,k,k_block,s", [("fp8", 16385, 0, 20), ("fp8", 40001, 0, 14), ("fp6", 33000, 16500, 13), ("fp6_e3m2", 24640, 0, 32),
                                             ("int8", 50000, 0, 12), ("fp16", 65536, 0, 9), ("fp16", 20000, 0, 6)])
@pytest.mark.parametrize("is_B", [0, 1])
def test_long_blocks_are_bit_exact(fmt, k, k_block, s, is_B):
    X = _vectors(k, np.random.default_rng(k))
    ref_codes, ref_exps, plan = oz.split_operand(X, fmt, s, k_block)
    got_codes, got_exps = _gpu_split(X, is_B, fmt, s, k_block)
    for t in range(plan.num_blocks):
        for p in range(s):
            bad = np.nonzero(got_exps[t][p] != ref_exps[t][p])[0]
            assert bad.size == 0, (t, p, bad, got_exps[t][p][bad], ref_exps[t][p][bad])
            assert np.array_equal(got_codes[t][p], ref_codes[t][p]), (t, p)


def test_slice_count_of_long_blocks():
    """Vector by vector, against the number of slices after which the oracle's codes are all zero."""
    k = 17000
    X = _vectors(k, np.random.default_rng(3))
    codes, _, _ = oz.split_operand(X, "fp8", 33, 0)
    lib.ozaki_set_stream(torch.cuda.current_stream().cuda_stream)
    ws = torch.zeros(64 << 20, dtype=torch.uint8, device="cuda")
    lib.ozaki_set_workspace(ws, ws.numel())
    for r in range(X.shape[0]):
        nonzero = [p for p in range(33) if np.any(codes[0][p][r] & 0x7F)]
        want = nonzero[-1] + 1 if nonzero else 0
        Xd = torch.from_numpy(np.ascontiguousarray(X[r:r + 1, :])).cuda()
        assert lib.ozaki_count_slices(1, 1, k, Xd, k, lib.SLICE_FP8_E4M3, 0) == want, r
    lib.ozaki_set_workspace(None, 0)
