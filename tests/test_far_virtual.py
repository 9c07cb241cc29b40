"""Cells of lines beyond the grid (far_geometry.h): over every leaf of the grid
that a window can touch, the lines of a cell inside or outside the grid arrive exactly once -- whole
through one tile, through a tile that the window may cut, or point by point -- and
never through tiles closer than the leaf's gap; the outermost cells go point
by point."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = r"""
#include "far_geometry.h"
using namespace xs;
extern "C" int virt(int sh, int lmax, long long Wx) { return far_virtual(sh, lmax, Wx); }
// as the device: tiles of the grid, cells [-v, n_fine + v); info: on, v, near leaves, a bad candidate count
extern "C" void count(long long W, long long Wx, int n_fine, int sh, double g0, double g1, int most, int f, int reach,
                      int* far, int* cut, int* direct, int* gap, int* info) {
  FarCond c = far_make(W, Wx, n_fine, sh, g0, g1);
  c.v = c.on ? far_virtual(sh, c.lmax, Wx) : 0;
  if (most >= 0 && c.v > most) c.v = most >> c.lmax << c.lmax;
  info[0] = c.on; info[1] = c.v; info[2] = 0; info[3] = -1; info[4] = 0; info[5] = c.lmax;
  for (int i = 0; i < n_fine; ++i) {
    far[i] = cut[i] = direct[i] = 0;
    gap[i] = c.on ? far_gap(c, 0, i) : 0;
  }
  if (!c.on) return;
  far_near(c, f, info[2], info[3]);
  for (int l = 0; l <= c.lmax; ++l)
    for (int t = 0; t < far_tiles(n_fine, l); ++t) {
      CellRange r[4], e[2], cc[2];
      far_tile_ranges(c, l, t, r);
      const CellRange cand = far_candidates(c, l, f, f);
      for (auto& q : r) {
        if (q.lo > q.hi) continue;
        if (q.lo < 1 - c.v || q.hi > n_fine - 2 + c.v) info[4]++;
        if (q.lo > f || q.hi < f) continue;
        if (t < cand.lo || t > cand.hi) info[4]++;
        for (int leaf = t << l; leaf < ((t + 1) << l) && leaf < n_fine; ++leaf) far[leaf]++;
      }
      if (l != c.end) continue;
      far_cut(c, t, e);
      far_cut_candidates(c, f, f, cc);
      for (int k = 0; k < 2; ++k) {
        if (e[k].lo > e[k].hi || e[k].lo > f || e[k].hi < f) continue;
        if (t < cc[k].lo || t > cc[k].hi) info[4]++;
        for (int leaf = t << l; leaf < ((t + 1) << l) && leaf < n_fine; ++leaf) cut[leaf]++;
      }
    }
  const int rl = 256 >> sh;
  for (int a = 0; a < n_fine; a += rl) {
    const int b = a + rl - 1;
    const int clo = far_max(a - reach, -c.v), chi = far_min(b + reach, n_fine - 1 + c.v);
    CellRange s[kSegs];
    far_segments(c, a, b, clo, chi, s);
    const int g = far_gap(c, 0, a);
    for (int k = 0; k < kSegs; ++k) {
      if (f < s[k].lo || f > s[k].hi) continue;
      for (int leaf = a; leaf <= b && leaf < n_fine; ++leaf)
        if (k != 0 || (leaf >= f - g && leaf <= f + g)) direct[leaf]++;
    }
  }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("far_virtual")
    src, so = d / "v.cpp", d / "v.so"
    src.write_text(SRC)
    inc = os.path.join(os.path.dirname(HERE), "paper_2609_17273_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", "-I", inc, str(src), "-o", str(so)], check=True)
    L = C.CDLL(str(so))
    p, i64, i32, dd = C.POINTER(C.c_int32), C.c_longlong, C.c_int, C.c_double
    L.count.argtypes = [i64, i64, i32, i32, dd, dd, i32, i32, i32, p, p, p, p, p]
    L.virt.argtypes = [i32, i32, i64]
    return L


# W, cells, log2 of a leaf's points, gap at cell 0 and its growth, most cells beyond the grid (-1: all)
CASES = [(2498, 313, 4, 0.3, 0.0, -1), (2498, 32, 4, 0.3, 1e-4, -1), (2498, 8, 6, 0.2, 0.0, -1),
         (2498, 80, 6, 0.1, 0.005, -1), (9998, 100, 4, 2.0, 0.01, -1), (49998, 64, 4, 30.0, 1e-4, -1),
         (2498, 100, 4, 0.3, 0.0, 64), (2498, 100, 4, 0.3, 0.0, 0), (700, 33, 4, 1.0, 0.001, -1),
         (2498, 3, 6, 0.5, 0.0, -1), (1300, 97, 6, 8.0, 0.0, -1)]


@pytest.mark.parametrize("W, nf, sh, g0, g1, most", CASES)
def test_every_leaf_once(lib, W, nf, sh, g0, g1, most):
    Wx, n = W + 4, 1 << sh
    ptr = lambda a: a.ctypes.data_as(C.POINTER(C.c_int32))
    fr, cu, di, gap = (np.zeros(nf, np.int32) for _ in range(4))
    info = np.zeros(6, np.int32)
    go = lambda f: lib.count(W, Wx, nf, sh, g0, g1, most, int(f), (Wx + n - 1) // n + 2, ptr(fr), ptr(cu), ptr(di),
                             ptr(gap), ptr(info))
    go(0)
    assert info[0] == 1
    v = int(info[1])
    assert v % (1 << info[5]) == 0
    if most < 0:
        assert v * n > Wx + n
    rng = np.random.default_rng(W + nf)
    cells = set([-v, 1 - v, 2 - v, -2, -1, 0, 1, nf - 1, nf, nf + 1, nf + v - 2, nf + v - 1])
    cells |= set(int(q) for q in rng.integers(-v, nf + v, 40))
    leaf = np.arange(nf)
    for f in sorted(c for c in cells if -v <= c < nf + v):
        go(f)
        covered = (n * leaf >= n * f + n - 1 - W) & (n * leaf + n - 1 <= n * f + W)
        touched = (n * leaf + n - 1 >= n * f - Wx) & (n * leaf <= n * f + n - 1 + Wx)
        assert info[4] == 0
        if f in (-v, nf - 1 + v):
            assert fr.sum() == 0 and cu.sum() == 0
            assert np.all(di[touched] == 1)
            continue
        assert np.all((fr + cu + di)[touched] == 1), f
        assert np.all(fr[~covered] == 0), f
        near = np.abs(leaf - f) <= gap
        assert np.all((fr + cu)[near] == 0) and np.all(di[~near] == 0), f
        assert np.array_equal(near, (leaf >= info[2]) & (leaf <= info[3])), f


def test_number_of_cells(lib):
    for sh in (4, 6):
        for lmax in (0, 3, 6, 15):
            for Wx in (100, 2502, 25002, 1 << 20, 1 << 28):
                v = lib.virt(sh, lmax, Wx)
                assert v % (1 << lmax) == 0 and 0 < v <= 1 << 16
                assert v == 1 << 16 or v << sh > Wx + (1 << sh)
