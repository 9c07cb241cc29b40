"""Doppler cores of many leaves: the moments of a Gaussian grow with the powers
of its standard deviation in cells, and stay in range because they begin at a level of cells
that are wide enough (far_sigma_level); FP32 ones of cells below a ninth of it would not.  The cases'
deviations are 9 to 36 leaves of 16 points; lists dense enough for the
moments.  Against the point-by-point gather's FP64 form at the tolerances of
test_gpu_far (its FP32 form is itself off by 6e-6 to 1.2e-5 where thousands of cores
overlap, the expansions by 2e-8 to 8e-8)."""
import numpy as np
import pytest

import synth
from test_gpu_far import FP32, FP64, TOL, C, _Grid
from xs_helpers import X, log

pytestmark = pytest.mark.gpu
CASES = {"hot": (19000.0, 5e-4, 2.0, C(5000.0, 0.05, 25.0)), "light": (20000.0, 0.001, 2.0, C(2000.0, 0.1, 25.0)),
         "edge": (19500.0, 5e-4, 18.0, C(2700.0, 0.05, 10.0))}


@pytest.mark.parametrize("case", list(CASES))
@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("profile", [synth.VOIGT, synth.BIN_VOIGT])
def test_wide_cores_against_points(profile, prec, case):
    import torch
    P = X()
    nu0, dnu, mass, cond = CASES[case]
    n, n_lines = 20011, 31001
    rng = np.random.default_rng(3)
    end = nu0 + (n - 1) * dnu
    nu = rng.uniform(nu0 - 2.0, end + 2.0, n_lines)
    El = np.concatenate([[0.0], rng.uniform(0.0, 8000.0, n_lines - 1)])
    st = synth.States(np.concatenate([El, El + nu]), np.ones(2 * n_lines))
    i = np.arange(n_lines, dtype=np.int32)
    ln = synth.Lines(i + np.int32(n_lines), i, (10.0 ** rng.uniform(-4, 2, n_lines)).astype(np.float32),
                     rng.uniform(0.02, 0.1, n_lines).astype(np.float32), rng.uniform(0.3, 0.8, n_lines).astype(np.float32))
    ds, dl = P.DeviceStates.from_numpy(st), P.DeviceLines.from_numpy(ln)
    plan, exact = (P.Plan(profile, 0, 0, q, _Grid(nu0, dnu, n), [cond], n_lines, mass_amu=mass) for q in (prec, FP64))
    got = plan.cross_section(ds, dl).clone()
    ref = exact.cross_section_noalloc(ds, dl, torch.empty_like(got)).clone()
    torch.cuda.synchronize()
    got, ref = got[0].cpu().numpy(), ref[0].cpu().numpy()
    plan.close()
    exact.close()
    assert np.all(np.isfinite(got)) and np.all(ref > 0.0)
    e = float(np.max(np.abs(got - ref) / ref))
    log(f"[wide cores] profile {profile} prec {prec} {case}: {e:.2e}")
    assert e <= TOL[prec]
