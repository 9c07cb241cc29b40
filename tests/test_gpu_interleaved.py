"""Stick spectra and partition functions of other lists and states between a
preparation and its passes: the prepared records keep their own scales, partition
functions and widths, so the pass and the adjoint after them give the same bits
as before."""
import numpy as np
import pytest

import synth
from test_gpu_far import FP32, FP64, C, _Grid
from xs_helpers import X, gpu_inputs, workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("between", ["sticks", "partition"])
@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("profile", [synth.VOIGT, synth.DOPPLER])
def test_records_outlive_other_calls(profile, prec, between):
    import torch
    P = X()
    wl = workload("voigt_1e7", n_states=20000, n_lines=30011, nu_hi=600.0, seed=99)
    other = synth.workload("voigt_1e7", n_states=3000, n_lines=7001, nu_hi=500.0, seed=5)
    la, lb = wl.lines(), other.lines()
    lb.einstein_a = lb.einstein_a * np.float32(1e6)   # another strongest line
    lb.gamma_ref = lb.gamma_ref * np.float32(50.0)    # and widest
    (sa, da), (sb, db) = gpu_inputs(wl, la), gpu_inputs(other, lb)
    n = 15001
    conds = [C(300.0, 0.4, 25.0), C(900.0, 20.0, 25.0)]
    plan = P.Plan(profile, 0, 0, prec, _Grid(300.0, 0.01, n), conds, la.n, mass_amu=wl.mass_amu)
    g = torch.as_tensor(np.random.default_rng(7).standard_normal((2, n)), device="cuda")
    plan.prepare(sa, da)
    sig = plan.profile().clone()
    adj = {k: v.clone() for k, v in plan.profile_adjoint(sa, da, g).items()}
    if between == "sticks":
        S, ls = plan.line_intensities(sb, db)
        assert prec == FP64 or ls.abs().min().item() > 0.0
    else:
        plan.partition_function(sb)
    sig2 = plan.profile().clone()
    adj2 = plan.profile_adjoint(sa, da, g)
    torch.cuda.synchronize()
    assert torch.equal(sig, sig2)
    assert all(torch.equal(adj[k], adj2[k]) for k in adj)
    plan.close()
