"""Cells and levels of the far field's moments (plain integer functions, CPU)."""
import ctypes
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = r"""
#include "far_geometry.h"
using namespace xs;
extern "C" int widest(int lo, int hi, int l) { return far_widest(lo, hi, l); }
extern "C" long long before(int n, int l) { return far_cells_before(n, l); }
extern "C" int tiles(int n, int l) { return far_tiles(n, l); }
extern "C" int mom_level(int sh, double g) { return far_mom_level(sh, g); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("far_moments")
    src, so = d / "m.cpp", d / "m.so"
    src.write_text(SRC)
    inc = os.path.join(os.path.dirname(HERE), "paper_2609_17273_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", inc, str(src), "-o", str(so)], check=True)
    L = ctypes.CDLL(str(so))
    L.before.restype = ctypes.c_longlong
    L.mom_level.argtypes = [ctypes.c_int, ctypes.c_double]
    return L


@pytest.mark.parametrize("lo, hi", [(1, 1), (1, 2), (2, 3), (1, 62), (63, 64), (64, 127), (5, 1000), (1023, 1025)])
@pytest.mark.parametrize("l", [0, 1, 3, 7])
def test_cells_make_up_a_range(lib, lo, hi, l):
    at, n = lo, 0
    while at <= hi:
        w = lib.widest(at, hi, l)
        assert 0 <= w <= l and at % (1 << w) == 0 and at + (1 << w) - 1 <= hi
        at += 1 << w
        n += 1
    assert at == hi + 1
    assert n <= (hi - lo + 1 >> l) + 2 * l + 1


def test_rows_and_levels(lib):
    for n in (1, 2, 31, 64, 65, 12500):
        assert [lib.before(n, k + 1) - lib.before(n, k) for k in range(8)] == [lib.tiles(n, k) for k in range(8)]
    for sh in (4, 6):
        assert lib.mom_level(sh, 0.0) == 0 and lib.mom_level(sh, 0.5 * (1 << sh)) == 0
        assert lib.mom_level(sh, 0.51 * (1 << sh)) == 1
        for g in (3.0, 77.0, 5000.0):
            k = lib.mom_level(sh, g)
            assert g <= 0.5 * (1 << sh + k) and (k == 0 or g > 0.5 * (1 << sh + k - 1))
        assert lib.mom_level(sh, float("inf")) == lib.mom_level(sh, float("nan")) == 16
