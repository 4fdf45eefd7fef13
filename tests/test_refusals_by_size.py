"""Grids whose bricked form is too large are refused whatever walk a call of so
few rays would take: the refusal does not depend on the number of rays."""
import ctypes as C

import pytest

from paper_1410_1629_amd import binding as B
from paper_1410_1629_amd import workloads as W

# 2^31 - 88049 cells, with whole bricks more than 2^31 - 1
PROB = {"box": (-1, 1, -1, 1, -1, 1), "n": (46339, 46341, 1)}
DUMMY = C.c_void_p(256)  # never read: the call is refused before any device work


@pytest.mark.parametrize("n", [1, 1 << 30])
def test_peel_off(n):
    lib, grid, det = B.load(), B.make_grid(PROB), B.make_detectors([W.frame(10.0, 30.0, 8, 8, 1.0, 1.0)])
    rc = lib.peel_off(C.byref(grid), DUMMY, 1.0, 0.0, 0, n, DUMMY, DUMMY, DUMMY, 1, det, DUMMY, None)
    assert rc == -1 and "bricked grid" in lib.mcrt_last_error().decode()


@pytest.mark.parametrize("entry", ["trace_path", "trace_path_noalloc"])
@pytest.mark.parametrize("n", [1, 1 << 30])
def test_trace_path(entry, n):
    lib, grid = B.load(), B.make_grid(PROB)
    rc = getattr(lib, entry)(C.byref(grid), DUMMY, 1.0, 0, n, DUMMY, DUMMY, DUMMY, 0, None, None, None, None, None)
    assert rc == -1 and "bricked grid" in lib.mcrt_last_error().decode()
