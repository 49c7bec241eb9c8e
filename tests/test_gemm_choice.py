"""The choices of the planner that decide how long the slice-pair GEMMs take, against measured times: the order of the
workgroups; 256 x 256 or 128 x 128 blocks and the length of the groups."""
import ctypes

import pytest

import planner


# 128 x 128 blocks?, slices, all pairs?, group length, block rows, block columns, stages per pair, GEMM microseconds in the plain order
# and in strips (MI355X)
ORDERS = [
    (1, 11, 1, 11, 5, 23, 24, 576, 290), (0, 11, 1, 8, 5, 10, 118, 2738, 1778), (1, 11, 1, 8, 13, 4, 82, 879, 608), (1, 11, 1, 8, 6, 18, 30, 374, 282),
    (1, 11, 1, 9, 19, 7, 19, 491, 274), (0, 16, 0, 7, 10, 5, 59, 922, 766), (0, 11, 1, 8, 3, 12, 24, 311, 270), (0, 11, 1, 2, 6, 5, 156, 2148, 1520),
    (1, 16, 0, 9, 15, 7, 8, 121, 102), (1, 8, 0, 7, 6, 34, 24, 209, 174), (1, 14, 1, 14, 4, 7, 54, 238, 280), (0, 13, 0, 8, 19, 1, 33, 191, 227),
    (0, 14, 1, 3, 2, 2, 192, 338, 399), (0, 16, 0, 11, 1, 19, 50, 279, 363), (1, 8, 0, 5, 30, 2, 72, 164, 206), (1, 13, 0, 11, 1, 29, 58, 232, 298),
    (1, 16, 0, 3, 6, 1, 154, 140, 182), (0, 11, 1, 10, 2, 12, 6, 69, 76), (0, 13, 0, 13, 4, 15, 2, 69, 77), (0, 13, 0, 9, 20, 3, 4, 84, 97),
    (1, 8, 0, 1, 3, 10, 64, 535, 351), (1, 8, 0, 2, 7, 4, 64, 226, 165), (1, 7, 1, 1, 3, 3, 128, 316, 209),
]


@pytest.mark.parametrize("small,s,full,length,blocks_m,blocks_n,chunks,plain,strips", ORDERS)
def test_order_of_the_workgroups(small, s, full, length, blocks_m, blocks_n, chunks, plain, strips):
    chosen = planner.load().order_of_launch(small, s, full, length, *[ctypes.c_int64(v) for v in (blocks_m, blocks_n, chunks)])
    assert (strips if chosen else plain) <= 1.05 * min(plain, strips)
