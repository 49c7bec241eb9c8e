"""The library's planner compiled for the host: which route a call takes (tests/host_plan_harness.cpp)."""
import collections
import ctypes
import functools
import os
import subprocess
import tempfile

from paper_2508_00441_amd import binding as lib

HERE = os.path.dirname(os.path.abspath(__file__))
Ladder = collections.namedtuple("Ladder", "starts limit reads_marks delta_launch mark_bytes")
Route = collections.namedtuple("Route", "small group_len run_limit measured bounds_from_slices pairs_per_pass")


@functools.lru_cache(maxsize=None)
def load() -> ctypes.CDLL:
    with tempfile.TemporaryDirectory() as d:
        out = os.path.join(d, "libhostplan.so")
        subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-w", "-o", out,
                               os.path.join(HERE, "host_plan_harness.cpp")])
        return ctypes.CDLL(out)


def route(m, n, k, fmt, s, k_block=0, mode="triangle", chained=True, minimum=False) -> Route:
    """The route of a DGEMM in a workspace of the documented (minimum) size."""
    r = (ctypes.c_int64 * 6)()
    i64 = ctypes.c_int64
    assert load().plan_route(i64(m), i64(n), i64(k), lib.SLICE_FORMATS[fmt], s, i64(k_block), lib.PAIR_SETS[mode], int(chained),
                             i64(-1 if minimum else 0), r) == 0
    return Route(*r)


def ladder(m, n, k, fmt, s, k_block=0, mode="triangle", exact=False) -> Ladder:
    """How a DGEMM begins: with the one pass over all pairs?"""
    r = (ctypes.c_int64 * 5)()
    i64 = ctypes.c_int64
    assert load().ladder_route(i64(m), i64(n), i64(k), lib.SLICE_FORMATS[fmt], s, i64(k_block), lib.PAIR_SETS[mode], int(exact), r) == 0
    return Ladder(*r)
