"""Tables whose conditions differ in window: some take tile expansions, some go point by
point in the near kernel (narrow windows) or in the gather (400 points and more to
a side), each with the values that it has by itself.  Against the gather of the
allocation-free call at the tolerances of test_gpu_far, and added to what sigma held."""
import numpy as np
import pytest

import synth
from test_gpu_far import FP32, FP64, TOL, C, _Grid
from xs_helpers import X, gpu_inputs, log, workload

pytestmark = pytest.mark.gpu
CONDS = [C(300.0, 1.0, 25.0), C(500.0, 1.0, 5.0), C(700.0, 0.1, 0.7), C(900.0, 10.0, 5.7), C(1100.0, 1.0, 2.0),
         C(1300.0, 1.0, 25.0)]


@pytest.mark.parametrize("config", [dict(), dict(tile_bins=512, bucket_bins=64, persistent=0)])
@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("profile", [synth.LORENTZ, synth.VOIGT, synth.BIN_LORENTZ, synth.BIN_VOIGT])
def test_mixed_windows(profile, prec, config):
    import torch
    P = X()
    n = 20011
    wl = workload("voigt_1e7", n_states=20000, n_lines=30011, nu_hi=600.0, seed=4242)
    ln = wl.lines()
    ds, dl = gpu_inputs(wl, ln)
    plan = P.Plan(profile, 0, 0, prec, _Grid(200.37, 0.01, n), CONDS, ln.n, mass_amu=wl.mass_amu)
    if config:
        plan.set_config(**config)
    got = plan.cross_section(ds, dl).clone()
    again = plan.profile().clone()
    ref = plan.cross_section_noalloc(ds, dl, torch.empty_like(got)).clone()
    start = torch.linspace(0.0, 1.0, n, dtype=torch.float64, device="cuda").repeat(len(CONDS), 1)
    acc = plan.cross_section(ds, dl, out=start.clone(), accumulate=True)
    torch.cuda.synchronize()
    assert torch.equal(got, again)
    got, ref, acc, start = (t.cpu().numpy() for t in (got, ref, acc, start))
    plan.close()
    for c in range(len(CONDS)):
        m = ref[c] > 0.0
        assert m.any() and np.all(got[c][~m] == 0.0)
        e = float(np.max(np.abs(got[c][m] - ref[c][m]) / ref[c][m]))
        log(f"[mixed] profile {profile} prec {prec} c{c}: {e:.2e}")
        assert e <= TOL[prec]
    assert np.allclose(acc, start + got, rtol=1e-14, atol=0.0)


@pytest.mark.parametrize("profile", [synth.LORENTZ, synth.VOIGT])
def test_replayed(profile):
    """The same in a graph, several replays with eager work between them."""
    import torch
    P = X()
    wl = workload("voigt_1e7", n_states=20000, n_lines=30011, nu_hi=600.0, seed=4242)
    ln = wl.lines()
    ds, dl = gpu_inputs(wl, ln)
    plan = P.Plan(profile, 0, 0, FP32, _Grid(200.37, 0.01, 20011), CONDS, ln.n, mass_amu=wl.mass_amu)
    want = plan.cross_section(ds, dl).clone()
    out = torch.empty_like(want)
    plan.capture(ds, dl, out)
    for _ in range(4):
        out.fill_(-1.0)
        plan.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        assert torch.equal(plan.cross_section(ds, dl), want)
    plan.close()
