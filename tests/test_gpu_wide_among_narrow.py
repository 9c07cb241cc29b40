"""A line of enormous pressure width (y = gamma / (sg sqrt 2) of 1e6 to 1e8) among narrow ones:
a wave of tile expansions takes one rule for all of its lines, and the narrow
ones' nearest tiles take six node pairs, whose products of the wide one's
denominators must not leave FP64's range.  Against the gather at the tolerances of test_gpu_far."""
import numpy as np
import pytest

import synth
from test_gpu_far import FP32, FP64, TOL, C, _Grid
from xs_helpers import X, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gref", [1e7, 1e8, 1e9, 2e10])
@pytest.mark.parametrize("profile", [synth.VOIGT, synth.BIN_VOIGT])
def test_wide_among_narrow(profile, gref):
    import torch
    P = X()
    nu0, dnu, n, n_lines = 19000.0, 5e-4, 20011, 9001
    rng = np.random.default_rng(3)
    end = nu0 + (n - 1) * dnu
    nu = rng.uniform(nu0 - 2.0, end + 2.0, n_lines)
    El = np.concatenate([[0.0], rng.uniform(0.0, 8000.0, n_lines - 1)])
    st = synth.States(np.concatenate([El, El + nu]), np.ones(2 * n_lines))
    i = np.arange(n_lines, dtype=np.int32)
    gr = rng.uniform(0.02, 0.1, n_lines)
    gr[np.argsort(np.abs(nu - (nu0 + end) / 2))[:3]] = gref
    ln = synth.Lines(i + np.int32(n_lines), i, (10.0 ** rng.uniform(-4, 2, n_lines)).astype(np.float32),
                     gr.astype(np.float32), rng.uniform(0.3, 0.8, n_lines).astype(np.float32))
    ds, dl = P.DeviceStates.from_numpy(st), P.DeviceLines.from_numpy(ln)
    plan = P.Plan(profile, 0, 0, FP64, _Grid(nu0, dnu, n), [C(5000.0, 0.05, 25.0)], n_lines, mass_amu=2.0)
    got = plan.cross_section(ds, dl).clone()
    ref = plan.cross_section_noalloc(ds, dl, torch.empty_like(got)).clone()
    torch.cuda.synchronize()
    got, ref = got[0].cpu().numpy(), ref[0].cpu().numpy()
    plan.close()
    assert np.all(np.isfinite(ref)) and np.all(np.isfinite(got))
    e = float(np.max(np.abs(got - ref) / ref))
    log(f"[wide among narrow] profile {profile} {gref:.0e}: {e:.2e}")
    assert e <= TOL[FP64]
