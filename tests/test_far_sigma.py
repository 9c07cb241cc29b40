"""The Gaussian moments' range: with the level that far_sigma_level gives, the
recurrence of the moments stays finite in its own precision, with 32 lines a lane and
a factor of a hundred to spare; and it is the lowest such level."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = r"""
#include "far_geometry.h"
extern "C" int level(int sh, double sigma, int f32) {
  return xs::far_sigma_level(sh, sigma, f32 ? xs::kMomSigma32 : xs::kMomSigma64);
}
"""


@pytest.fixture(scope="module")
def level(tmp_path_factory):
    d = tmp_path_factory.mktemp("far_sigma")
    src, so = d / "m.cpp", d / "m.so"
    src.write_text(SRC)
    inc = os.path.join(os.path.dirname(HERE), "paper_2609_17273_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", inc, str(src), "-o", str(so)], check=True)
    f = ctypes.CDLL(str(so)).level
    f.argtypes = [ctypes.c_int, ctypes.c_double, ctypes.c_int]
    return f


def _largest(sigma, n, dt):
    """max |u_k|, u_(k+1) = s u_k + k sigma^2 u_(k-1), over the s of a line within half a cell."""
    worst = 0.0
    with np.errstate(all="ignore"):
        for a in (-0.5, 0.0, 0.5):
            for b in (1e-3, 0.1, 0.5):
                sr, si, e2 = dt(a), dt(b), dt(sigma * sigma)
                pr, pi, ur, ui = dt(1), dt(0), sr, si
                for k in range(1, n + 1):
                    worst = max(worst, abs(float(ur)), abs(float(ui)))
                    if not np.isfinite(worst) or np.isnan(ur) or np.isnan(ui):
                        return np.inf
                    e = dt(k) * e2
                    ur, ui, pr, pi = dt(sr * ur + (e * pr - si * ui)), dt(sr * ui + (si * ur + e * pi)), ur, ui
    return worst


@pytest.mark.parametrize("f32, sh, n, dt", [(1, 4, 28, np.float32), (0, 6, 48, np.float64)])
@pytest.mark.parametrize("sigma", [0.0, 0.3, 20.0, 64.0, 64.1, 150.0, 600.0, 5e4, 4e6, 6e6])
def test_moments_in_range(level, f32, sh, n, dt, sigma):
    l = level(sh, sigma, f32)
    if l == 16:  # no level: lines go one by one
        assert sigma > (4.0 if f32 else 65536.0) * (1 << sh + 15)
        return
    assert _largest(sigma / (1 << sh + l), n, dt) * 32 < np.finfo(dt).max / 100
    most = 4.0 if f32 else 65536.0
    assert l == 0 or sigma > most * (1 << sh + l - 1)


def test_not_finite(level):
    assert level(4, float("inf"), 1) == level(4, float("nan"), 1) == 16
