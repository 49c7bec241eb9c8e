"""Slicing along ladders of units (csrc/slice_digits.hpp) on the host: slice integers and exponents equal to the oracle's for
vectors that keep to the ladder, leave it, run out, are exact halves of their units, and reach below the 96-bit number."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from oracle import ozaki_oracle as oo
from paper_2508_00441_amd import inputs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def digits(tmp_path_factory):
    out = tmp_path_factory.mktemp("digits") / "libdigits.so"
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-o", str(out), os.path.join(ROOT, "tests", "host_slice_digits_harness.cpp")])
    return ctypes.CDLL(str(out))


def _halves(rng, rows, k, b):
    """Sums of signed multiples of ladder units whose last digit is the exact half: every tie, either sign, even and odd floors."""
    step = b + 1
    X = np.zeros((rows, k))
    for j in range(rows):
        depth = rng.integers(0, 52 // step, k)
        lead = rng.integers(-(1 << b), (1 << b) + 1, k).astype(np.float64)
        mid = rng.integers(-(1 << (b - 1)) if b > 0 else 0, (1 << b >> 1) + 1, k).astype(np.float64)
        X[j] = lead + np.ldexp(mid, -step * np.maximum(depth - 1, 0)) + np.ldexp(rng.choice([-0.5, 0.5, 1.0], k), -step * depth)
    X[:, 0] = 1 << b
    return X


@pytest.mark.parametrize("b", [0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11])
def test_ladder_slices_equal_the_oracle(digits, b):
    rng = np.random.default_rng(300 + b)
    k, s = 180, 18
    X = np.vstack([
        inputs.nasty_rows(rng, 40, k), _halves(rng, 12, k, b), -_halves(rng, 4, k, b),
        inputs.phi_matrix(8, k, 0.5, rng), inputs.phi_matrix(6, k, 6.0, rng), inputs.phi_matrix(4, k, 20.0, rng),
        inputs.uniform_1_10(6, k, rng),
        rng.integers(-1000, 1001, (4, k)).astype(np.float64),
        np.ldexp(rng.integers(-(1 << 20), 1 << 20, (4, k)).astype(np.float64), -30) + 3.0,
        np.ldexp(1.0, rng.integers(-40, 40, (4, k))) * np.where(rng.random((4, k)) < 0.5, -1, 1),
        inputs.phi_matrix(4, k, 1.0, rng) * 2.0 ** -1040, inputs.phi_matrix(4, k, 6.0, rng) * 2.0 ** -1015,
        np.ldexp(1.0 + rng.random((4, k)), rng.integers(-1070, 900, (4, k))),
    ])
    X[:, 5:9] = -0.0                                         # the sign of a zero is no part of its number
    slices, cs, _ = oo.slice_rows(X, 53 - b, s)
    want_q = np.stack([oo.slice_integers(v, b) for v in slices]).astype(np.int64)
    want_c = np.stack(cs)
    ladders = 0
    for r in range(X.shape[0]):
        x = np.ascontiguousarray(X[r])
        q, c = np.empty((s, k), dtype=np.int32), np.empty(s, dtype=np.int32)
        ladders += digits.host_slice_vector_digits(x.ctypes.data_as(ctypes.c_void_p), ctypes.c_size_t(k), b, s, q.ctypes.data_as(ctypes.c_void_p),
                                                   c.ctypes.data_as(ctypes.c_void_p))
        assert np.array_equal(c, want_c[:, r]), (r, c, want_c[:, r])
        assert np.array_equal(q, want_q[:, r, :]), r
    assert ladders > X.shape[0]                              # some vectors needed more than one


@pytest.mark.parametrize("b", [2, 3, 4, 6, 7, 8, 11])
@pytest.mark.parametrize("nonzeros", [1, 2, 4, 16])
def test_few_nonzeros_take_one_number(digits, b, nonzeros):
    """Vectors of few non-zero elements leave the ladder at every other unit; their slices still come from one reading of the vector,
    as long as its bits fit into 96, and one more for each further 96."""
    rng = np.random.default_rng(700 + 10 * b + nonzeros)
    k, rows, s = 64, 60, 33
    X = np.zeros((rows, k))
    for j in range(rows):
        X[j, rng.permutation(k)[:nonzeros]] = (rng.random(nonzeros) - 0.5) * np.exp(rng.normal(0.0, 2.0 if j < rows - 8 else 30.0, nonzeros))
    slices, cs, _ = oo.slice_rows(X, 53 - b, s)
    want_q = np.stack([oo.slice_integers(v, b) for v in slices]).astype(np.int64)
    want_c = np.stack(cs)
    for r in range(rows):
        x = np.ascontiguousarray(X[r])
        q, c = np.empty((s, k), dtype=np.int32), np.empty(s, dtype=np.int32)
        digits.host_slice_vector_digits(x.ctypes.data_as(ctypes.c_void_p), ctypes.c_size_t(k), b, s, q.ctypes.data_as(ctypes.c_void_p),
                                        c.ctypes.data_as(ctypes.c_void_p))
        assert np.array_equal(c, want_c[:, r]), (r, c, want_c[:, r])
        assert np.array_equal(q, want_q[:, r, :]), r
        used = np.abs(x[x != 0])
        span = int(np.log2(used.max() / used.min())) + 1 + 53 + 2 * (b + 1)
        assert digits.host_numbers_of_last_vector() <= 1 + span // 80, (r, span)
        if span <= 96:
            assert digits.host_numbers_of_last_vector() == 1, (r, span)
