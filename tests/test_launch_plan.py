"""The host-side rules of the launches (csrc/launch_plan.h), compiled with the host compiler and checked without a GPU."""
import ctypes as C
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
OUT = os.path.join(ROOT, "_build", "host_plan")
pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host C++ compiler")


@pytest.fixture(scope="module")
def plan():
    os.makedirs(OUT, exist_ok=True)
    so = os.path.join(OUT, "plan.so")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-o", so,
                           "-I", os.path.join(ROOT, "paper_2605_10501_amd", "csrc"), os.path.join(ROOT, "tests", "host_plan", "plan_abi.cpp")])
    lib = C.CDLL(so)
    lib.plan_matrix_extent.restype = C.c_long
    return lib


OUT_OF_RANGE = 0xFFFFF000                      # the byte offset that a load of nothing uses (kOob)


def extent(plan, outer, inner, ld):
    return plan.plan_matrix_extent(C.c_long(outer), C.c_long(inner), C.c_long(ld))


@pytest.mark.parametrize("outer,inner", [(1, 1), (1, 7), (5, 8), (33, 64), (0, 8), (0, 1), (4, 0), (0, 0)])
@pytest.mark.parametrize("pad", [0, 1, 16, 1023, 100_000])
def test_descriptor_range_is_the_matrix(plan, outer, inner, pad):
    """No element past the last one, and nothing at all for an empty operand (K = 0, in either layout, with padded rows)."""
    ld = inner + pad
    last = max((r * ld + c for r in range(outer) for c in range(inner)), default=-1)
    n = extent(plan, outer, inner, ld)
    assert n == last + 1
    for es in (2, 4):
        assert (n * es) % (1 << 32) <= OUT_OF_RANGE        # as the unsigned range the descriptor holds


def test_what_a_descriptor_cannot_address(plan):
    ok = lambda outer, inner, ld, es: plan.plan_buffer_range_ok(C.c_long(outer), C.c_long(inner), C.c_long(ld), es)
    assert ok(1 << 14, 1 << 14, 1 << 14, 4) and not ok(1 << 15, 1 << 15, 1 << 15, 4)
    assert ok(1, 1 << 29, 0, 4) and not ok(1, 1 << 30, 0, 4)          # one long row counts with a zero stride as well
    assert ok(4, 8, 0, 4) and not ok(4, 8, -8, 4) and ok(1, 8, -8, 4)  # rows that go backwards are outside the range
    assert ok(0, 8, 8, 4) and ok(8, 0, 8, 4)


@pytest.mark.parametrize("wgs", [1, 255, 1 << 20, (1 << 24) - 1, 1 << 24, (1 << 24) + 1, 3 * (1 << 24) + 7, (1 << 31) - 1])
def test_grids_stay_below_the_thread_limit(plan, wgs):
    xy = (C.c_uint * 2)()
    plan.plan_fold_grid(C.c_long(wgs), 256, xy)
    x, y = xy
    assert x * 256 < 1 << 32 and y <= 65535 and wgs <= x * y < wgs + (1 << 20)
    assert (y == 1) == (wgs < 1 << 24) == bool(plan.plan_launch_fits(C.c_long(wgs), 256))


def test_fp32_attention_tiles_only_where_the_grid_can_be_launched(plan):
    f = lambda n, seqs, longest, hd=64, nq=4, nkv=4, heads=4: bool(
        plan.plan_f32_attention_tiles(hd, C.c_long(n), C.c_long(seqs), C.c_long(longest), nq, nkv, heads))
    assert f(293, 4, 128) and f(8192, 1, 8192) and f(8192, 1, 8192, 80) and f(8192, 1, 8192, 128)
    assert not f(293, 4, 128, 96) and not f(293, 4, 0) and not f(293, 4, 128, heads=65536)
    assert not f(104_096, 100_001, 4096) and f(104_096, 65_535, 4096) and not f(104_096, 65_536, 4096)   # 2^24 workgroups
    assert not f(1 << 21, 1 << 11, 1024, 128, 8, 8, 8)                                                   # qkv above 4 GB
