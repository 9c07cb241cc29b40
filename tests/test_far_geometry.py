"""The far field's geometry on the host: over every leaf that a window can
touch, a cell's lines arrive exactly once -- whole through one tile's expansion,
through a tile that the window may cut, or point by point; a tile takes lines
whole only where every window covers it, and only away from the near leaves."""
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
    lib.far_count.argtypes = [C.c_int64, C.c_int64, C.c_int32, C.c_int64, C.c_int32, C.c_int32, C.c_int32, p, p, p]
    return lib


@pytest.mark.parametrize("W,nf,gap,on", [(2498, 469, 1, 1), (2498, 300, 2, 1), (9998, 500, 5, 1), (600, 64, 1, 1),
                                         (319, 50, 1, 0), (49998, 1700, 23, 1), (2498, 3, 1, 1), (2498, 2, 1, 0),
                                         (100000, 130, 3, 1), (1000, 97, 4, 1), (1300, 97, 9, 1), (1300, 97, 19, 1),
                                         (2303, 211, 1, 1), (2304, 211, 1, 1), (1152, 90, 7, 1), (2498, 300, 40, 0)])
@pytest.mark.parametrize("row", [4, 16])
def test_every_leaf_once(far, W, nf, gap, on, row):
    Wx = W + 4
    rng = np.random.default_rng(W + nf)
    cells = sorted(set([0, 1, 2, 3, nf - 1, nf - 2, nf // 2] + list(rng.integers(0, nf, 25))))
    ptr = lambda a: a.ctypes.data_as(C.POINTER(C.c_int32))
    for f in cells:
        if f < 0 or f >= nf:
            continue
        fr, cu, di = (np.zeros(nf, np.int32) for _ in range(3))
        assert far.far_count(W, Wx, nf, gap, row, int(f), (Wx + 63) // 64 + 1, ptr(fr), ptr(cu), ptr(di)) == on
        leaf = np.arange(nf)
        # inside every window of the cell / possibly inside one of them
        covered = (64 * leaf >= 64 * f + 63 - W) & (64 * leaf + 63 <= 64 * f + W)
        touched = (64 * leaf + 63 >= 64 * f - Wx) & (64 * leaf <= 64 * f + 63 + Wx)
        if f in (0, nf - 1) or not on:  # lines beyond the grid: all point by point
            assert fr.sum() == 0 and cu.sum() == 0
            assert np.all(di[touched] == 1)
            continue
        assert np.all((fr + cu + di)[touched] == 1), (W, nf, row, f)
        assert np.all(fr[~covered] == 0)
        near = np.abs(leaf - f) <= gap
        assert np.all((fr + cu)[near] == 0)
        assert np.all(di[~near] == 0)
        # a cut tile is at least 18 of its half-widths from the line
        if cu.any():
            width = min(4, max(1, int(cu.sum())))
            assert 64 * np.abs(leaf[cu > 0] - f).min() >= 18 * 8 * width
