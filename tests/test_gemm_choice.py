"""The choices of the planner that decide how long the slice-pair GEMMs take, against measured times: the order of the
workgroups; 256 x 256 or 128 x 128 blocks and the length of the groups."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def planner(tmp_path_factory):
    out = tmp_path_factory.mktemp("plan") / "libhostplan.so"
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-w", "-o", str(out),
                           os.path.join(ROOT, "tests", "host_plan_harness.cpp")])
    return ctypes.CDLL(str(out))


# 128 x 128 blocks?, groups, block rows, block columns, stages per pair, GEMM microseconds in the plain order and in strips (MI355X)
ORDERS = [
    (1, 21, 5, 23, 24, 576, 290), (0, 26, 5, 10, 118, 2738, 1778), (1, 26, 13, 4, 82, 879, 608), (1, 26, 6, 18, 30, 374, 282),
    (1, 24, 19, 7, 19, 491, 274), (0, 27, 10, 5, 59, 922, 766), (0, 26, 3, 12, 24, 311, 270), (0, 66, 6, 5, 156, 2148, 1520),
    (1, 23, 15, 7, 8, 121, 102), (1, 9, 6, 34, 24, 209, 174), (1, 27, 4, 7, 54, 238, 280), (0, 18, 19, 1, 33, 191, 227),
    (0, 75, 2, 2, 192, 338, 399), (0, 21, 1, 19, 50, 279, 363), (1, 11, 30, 2, 72, 164, 206), (1, 15, 1, 29, 58, 232, 298),
    (1, 51, 6, 1, 154, 140, 182), (0, 22, 2, 12, 6, 69, 76), (0, 13, 4, 15, 2, 69, 77), (0, 17, 20, 3, 4, 84, 97),
]


@pytest.mark.parametrize("small,groups,blocks_m,blocks_n,chunks,plain,strips", ORDERS)
def test_order_of_the_workgroups(planner, small, groups, blocks_m, blocks_n, chunks, plain, strips):
    chosen = planner.order_of_launch(small, *[ctypes.c_int64(v) for v in (groups, blocks_m, blocks_n, chunks)])
    assert (strips if chosen else plain) <= 1.05 * min(plain, strips)
