"""Tiles through the moments of their cells, against the point-by-point gather.

Lists dense enough for the moments (24 lines to a leaf), as expansions against
points: the same tolerances, to which the moments add 4e-9 (FP32 form) and 4e-15.
Conditions reach from Doppler cores that keep several leaves near to lines wider
than every cell (no level by moments); windows from a few cells to more
than six levels, whose moments take two launches.
"""
import numpy as np
import pytest

import synth
from test_gpu_far import FP32, FP64, TOL, C, _Grid
from xs_helpers import X, gpu_inputs, log, workload

pytestmark = pytest.mark.gpu
CASES = {
    "widths": ((300.0, 0.01, 15001), [C(300.0, p, 25.0) for p in (1e-3, 0.4, 3.0, 20.0, 300.0)]),
    "hot": ((150.0, 0.003, 15011), [C(4000.0, 0.2, 7.3), C(4000.0, 40.0, 21.0)]),
    "levels": ((310.0, 0.001, 40003), [C(1200.0, 0.1, 25.0)]),
}


@pytest.mark.parametrize("case", list(CASES))
@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("profile", [synth.LORENTZ, synth.VOIGT, synth.BIN_LORENTZ, synth.BIN_VOIGT])
def test_moments_against_points(profile, prec, case):
    import torch
    P = X()
    (nu0, dnu, n), conds = CASES[case]
    wl = workload("voigt_1e7", n_states=20000, n_lines=70001, nu_hi=600.0, seed=99)
    ln = wl.lines()
    ds, dl = gpu_inputs(wl, ln)
    plan = P.Plan(profile, 0, 0, prec, _Grid(nu0, dnu, n), conds, ln.n, mass_amu=wl.mass_amu)
    got = plan.cross_section(ds, dl).clone()
    ref = plan.cross_section_noalloc(ds, dl, torch.empty_like(got)).clone()
    torch.cuda.synchronize()
    got, ref = got.cpu().numpy(), ref.cpu().numpy()
    plan.close()
    for c in range(len(conds)):
        m = ref[c] > 0.0
        e = float(np.max(np.abs(got[c][m] - ref[c][m]) / ref[c][m]))
        log(f"[moments] profile {profile} prec {prec} {case} c{c}: {e:.2e}")
        assert e <= TOL[prec]


@pytest.mark.parametrize("prec", [FP64, FP32])
def test_sticks_between_prepare_and_pass(prec):
    """A stick spectrum leaves the records of the last preparation, and with them
    the widest line's half-width that chooses the moments' levels: the pass after
    it gives the same bits as the one before."""
    import torch
    P = X()
    wl = workload("voigt_1e7", n_states=20000, n_lines=70001, nu_hi=600.0, seed=99)
    ln = wl.lines()
    ds, dl = gpu_inputs(wl, ln)
    plan = P.Plan(synth.VOIGT, 0, 0, prec, _Grid(300.0, 0.01, 15001), [C(300.0, p, 25.0) for p in (0.4, 20.0)], ln.n,
                  mass_amu=wl.mass_amu)
    plan.prepare(ds, dl)
    a = plan.profile().clone()
    plan.line_intensities(ds, dl)
    b = plan.profile().clone()
    torch.cuda.synchronize()
    assert torch.equal(a, b)
    plan.close()
