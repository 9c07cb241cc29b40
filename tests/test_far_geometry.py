"""The far field's geometry on the host: over every leaf that a window can
touch, a cell's lines arrive exactly once -- whole through one tile's expansion,
through a tile that the window may cut, or point by point; a tile takes lines
whole only where every window covers it, and only beyond the leaf's gap."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def far(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("far") / "far_host.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", os.path.join(HERE, "far_host.cpp"), "-o", so],
                   check=True)
    lib = C.CDLL(so)
    p = C.POINTER(C.c_int32)
    i64, i32, d = C.c_int64, C.c_int32, C.c_double
    lib.far_count.argtypes = [i64, i64, i32, i32, d, d, i32, i32, i32, p, p, p, p, p]
    return lib


# W, cells, log2 of a leaf's points, gap in cells at cell 0 and its growth per cell
CASES = [(2498, 469, 6, 0.3, 0.0, 1), (2498, 300, 6, 0.1, 0.005, 1), (9998, 500, 6, 0.0, 0.01, 1),
         (600, 64, 6, 0.5, 0.001, 1), (319, 50, 6, 0.5, 0.0, 0), (49998, 1700, 6, 1.2, 0.01, 1),
         (2498, 3, 6, 0.5, 0.0, 1), (2498, 2, 6, 0.5, 0.0, 0), (100000, 130, 6, 2.0, 0.0, 1),
         (1000, 97, 6, 3.2, 0.0, 1), (1300, 97, 6, 8.0, 0.0, 1), (2303, 211, 6, 0.5, 0.0, 1),
         (2304, 211, 6, 0.5, 0.0, 1), (1152, 90, 6, 6.1, 0.0, 1), (2498, 300, 6, 39.0, 0.0, 0),
         (2498, 937, 5, 0.2, 0.003, 1), (2498, 1700, 4, 0.4, 0.002, 1), (600, 301, 4, 2.0, 0.01, 1),
         (577, 120, 5, 0.5, 0.0, 1), (575, 120, 5, 0.5, 0.0, 0), (9998, 2200, 4, 0.0, 0.02, 1)]


@pytest.mark.parametrize("W,nf,sh,g0,g1,on", CASES)
@pytest.mark.parametrize("row_points", [256, 64])
def test_every_leaf_once(far, W, nf, sh, g0, g1, on, row_points):
    Wx, n = W + 4, 1 << sh
    rng = np.random.default_rng(W + nf)
    cells = sorted(set([0, 1, 2, 3, nf - 1, nf - 2, nf // 2] + list(rng.integers(0, nf, 25))))
    ptr = lambda a: a.ctypes.data_as(C.POINTER(C.c_int32))
    for f in cells:
        if f < 0 or f >= nf:
            continue
        fr, cu, di, gap = (np.zeros(nf, np.int32) for _ in range(4))
        info = np.zeros(5, np.int32)
        far.far_count(W, Wx, nf, sh, g0, g1, row_points >> sh, int(f), (Wx + n - 1) // n + 1, ptr(fr), ptr(cu),
                      ptr(di), ptr(gap), ptr(info))
        assert info[0] == on
        leaf = np.arange(nf)
        # inside every window of the cell / possibly inside one of them
        covered = (n * leaf >= n * f + n - 1 - W) & (n * leaf + n - 1 <= n * f + W)
        touched = (n * leaf + n - 1 >= n * f - Wx) & (n * leaf <= n * f + n - 1 + Wx)
        if f in (0, nf - 1) or not on:  # lines beyond the grid: all point by point
            assert fr.sum() == 0 and cu.sum() == 0
            assert np.all(di[touched] == 1)
            continue
        assert np.all((fr + cu + di)[touched] == 1), (W, nf, sh, f)
        assert np.all(fr[~covered] == 0)
        near = np.abs(leaf - f) <= gap
        assert np.all((fr + cu)[near] == 0)
        assert np.array_equal(near, (leaf >= info[2]) & (leaf <= info[3]))
        assert info[4] == 0
        assert np.all(di[~near] == 0)
        # as many cells as the lines of the cell need
        assert np.all((gap >= g0 + g1 * f)[touched]) and np.all(gap >= 1)
        # a cut tile is at least 17 of its half-widths from the line's cell
        if cu.any():
            assert (n * np.abs(leaf[cu > 0] - f)).min() + n >= 17 * info[1] // 2 - info[1] // 2
