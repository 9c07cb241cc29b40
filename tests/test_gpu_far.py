"""Tile expansions against the point-by-point gather.

xs_cross_section_noalloc runs the same path without expansions, so the two
calls of one plan differ by the interpolation (3.4e-14 of a line's value with
20 nodes, 2.2e-8 with 12) and by rounding: in the FP64 form up to 3.2e-12, the
gather's stepping of x along a row, and 4e-12 is asked for; in the FP32 form
each side keeps a value within about 3e-6 (the hardware reciprocal and the
rounding of x^2), and 1e-5 is asked for.  Points that no window reaches are
exactly zero on both sides."""
import numpy as np
import pytest

import synth
from xs_helpers import X, gpu_inputs, log, workload

pytestmark = pytest.mark.gpu

FP64, FP32 = 0, 1
TOL = {FP64: 4e-12, FP32: 1e-5}
C = synth.Condition

# grid (nu0, dnu, points) and conditions: window ends on tiles of 256, 128 and
# 64 points, lines beyond both grid ends, windows wider than the grid and too
# narrow for expansions, near regions of several leaves, ragged last cells
CASES = {
    "wide": ((0.0, 0.01, 60001), [C(2000.0, 1.0, 25.0)]),
    "inside": ((200.37, 0.01, 20011), [C(1000.0, 0.3, 25.0)]),
    "mixed_cutoffs": ((100.0, 0.01, 30017), [C(300.0, 1e-4, 6.1), C(2500.0, 50.0, 100.0), C(800.0, 1.0, 2.0),
                                            C(800.0, 1.0, 12.5)]),
    "fine_step": ((500.0, 0.001, 30001), [C(5000.0, 0.01, 10.0)]),
    "short": ((300.0, 0.01, 259), [C(1500.0, 1.0, 25.0)]),
}


class _Grid:
    def __init__(self, nu0, dnu, n):
        self.nu0, self.dnu, self.n_bins = nu0, dnu, n


def _run(profile, prec, case, lines=None):
    import torch
    P = X()
    (nu0, dnu, n), conds = CASES[case]
    wl = workload("voigt_1e7", n_states=20000, n_lines=30011, nu_hi=600.0, seed=4242)
    ln = wl.lines() if lines is None else lines
    ds, dl = gpu_inputs(wl, ln)
    plan = P.Plan(profile, 0, 0, prec, _Grid(nu0, dnu, n), conds, ln.n, mass_amu=wl.mass_amu)
    start = torch.linspace(0.0, 1.0, n, dtype=torch.float64, device="cuda").repeat(len(conds), 1)
    got = plan.cross_section(ds, dl).clone()
    ref = plan.cross_section_noalloc(ds, dl, torch.empty_like(got)).clone()
    acc = plan.cross_section(ds, dl, out=start.clone(), accumulate=True)
    torch.cuda.synchronize()
    got, ref, acc, start = (t.cpu().numpy() for t in (got, ref, acc, start))
    plan.close()
    return got, ref, acc, start


@pytest.mark.parametrize("case", list(CASES))
@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("profile", [synth.LORENTZ, synth.VOIGT, synth.BIN_LORENTZ, synth.BIN_VOIGT])
def test_expansions_against_points(profile, prec, case):
    got, ref, acc, start = _run(profile, prec, case)
    assert np.all(np.isfinite(got))
    for c in range(got.shape[0]):
        m = ref[c] > 0.0
        assert m.any()
        assert np.all(got[c][~m] == 0.0)
        e = float(np.max(np.abs(got[c][m] - ref[c][m]) / ref[c][m]))
        log(f"[far] profile {profile} prec {prec} {case} c{c}: {e:.2e}")
        assert e <= TOL[prec]
    assert np.allclose(acc, start + got, rtol=1e-14, atol=0.0)


def test_lines_that_are_not_finite():
    """A line of infinite intensity reaches the points of its window and no
    others, as point by point (where a formula forms the infinity as a
    difference of infinities it is not a number; which points those are
    depends on the formula)."""
    wl = workload("voigt_1e7", n_states=20000, n_lines=30011, nu_hi=600.0, seed=4242)
    ln = wl.lines().take(np.arange(30011))
    ln.einstein_a = ln.einstein_a.copy()
    ln.einstein_a[17] = np.inf
    got, ref, _, _ = _run(synth.VOIGT, FP64, "wide", ln)
    assert not np.all(np.isfinite(ref))
    assert np.array_equal(np.isfinite(got), np.isfinite(ref))
    m = np.isfinite(ref)
    assert np.max(np.abs(got[m] - ref[m]) / ref[m]) <= TOL[FP64]


@pytest.mark.parametrize("case", list(CASES))
@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("profile", [synth.LORENTZ, synth.VOIGT])
def test_adjoint_against_points(profile, prec, case):
    """The adjoint with expansions (a gather plan's) against point by point (a
    scatter plan's).  Both sum the same terms; a term keeps about 3e-12 of
    itself in the FP64 form and 3e-6 in the FP32 form, and cotangents of random
    signs leave a gradient's norm at least a tenth of its terms' norm: 1e-10 and
    1e-4 of the norm are asked for."""
    import torch
    P = X()
    (nu0, dnu, n), conds = CASES[case]
    wl = workload("voigt_1e7", n_states=20000, n_lines=30011, nu_hi=600.0, seed=4242)
    ln = wl.lines()
    ds, dl = gpu_inputs(wl, ln)
    rng = np.random.default_rng(7)
    g = torch.as_tensor(rng.standard_normal((len(conds), n)), device="cuda")
    out = []
    for algo in (0, 1):
        plan = P.Plan(profile, 0, 0, prec, _Grid(nu0, dnu, n), conds, ln.n, mass_amu=wl.mass_amu, algo=algo)
        r = plan.adjoint(ds, dl, g)
        torch.cuda.synchronize()
        out.append({k: v.cpu().numpy() for k, v in r.items()})
        plan.close()
    tol = {FP64: 1e-10, FP32: 1e-4}[prec]
    for k in out[0]:
        e = float(np.linalg.norm(out[0][k] - out[1][k]) / max(np.linalg.norm(out[1][k]), 1e-300))
        log(f"[far adjoint] profile {profile} prec {prec} {case} {k}: {e:.2e}")
        assert np.all(np.isfinite(out[0][k]))
        assert e <= tol
        assert np.array_equal(out[0][k] == 0.0, out[1][k] == 0.0)
