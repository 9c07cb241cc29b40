"""A table's conditions without tile expansions go through the gather or the near kernel,
all of them one way by the table's windows and the number of lines: both sides of that, against the
gather of the allocation-free call at the tolerances of test_gpu_far, replayed too."""
import numpy as np
import pytest

import synth
from test_gpu_far import FP32, FP64, TOL, C, _Grid
from xs_helpers import X, gpu_inputs, log, workload

pytestmark = pytest.mark.gpu
# 1620 points to a side without expansions: the gather's from 2.78e5 lines on (bin means from 5e4 and 1.1e5);
# the narrow ones take the second table to the near kernel
WIDE = [C(300.0, 1.0, 25.0), C(500.0, 1.0, 5.7), C(900.0, 0.1, 5.5), C(1100.0, 1.0, 5.0)]
NARROW = [C(300.0, 1.0, 25.0), C(500.0, 1.0, 5.7), C(900.0, 0.1, 0.5), C(1100.0, 1.0, 0.3)]


@pytest.mark.parametrize("table", ["wide", "narrow"])
@pytest.mark.parametrize("n_lines", [30011, 285011])
@pytest.mark.parametrize("profile,prec", [(synth.LORENTZ, FP64), (synth.LORENTZ, FP32), (synth.VOIGT, FP32), (synth.VOIGT, FP64),
                                          (synth.BIN_VOIGT, FP32), (synth.BIN_LORENTZ, FP64)])
def test_both_ways(profile, prec, n_lines, table):
    import torch
    P = X()
    conds = WIDE if table == "wide" else NARROW
    wl = workload("voigt_1e7", n_states=20000, n_lines=n_lines, nu_hi=600.0, seed=77)
    ln = wl.lines()
    ds, dl = gpu_inputs(wl, ln)
    plan = P.Plan(profile, 0, 0, prec, _Grid(200.37, 0.01, 20011), conds, ln.n, mass_amu=wl.mass_amu)
    got = plan.cross_section(ds, dl).clone()
    assert torch.equal(got, plan.profile())
    ref = plan.cross_section_noalloc(ds, dl, torch.empty_like(got)).clone()
    out = torch.empty_like(got)
    plan.capture(ds, dl, out)
    for _ in range(3):
        out.fill_(-1.0)
        plan.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, got)
    got, ref = got.cpu().numpy(), ref.cpu().numpy()
    plan.close()
    for c in range(len(conds)):
        m = ref[c] > 0.0
        assert m.any() and np.all(got[c][~m] == 0.0)
        e = float(np.max(np.abs(got[c][m] - ref[c][m]) / ref[c][m]))
        log(f"[mixed routes] profile {profile} prec {prec} {n_lines} {table} c{c}: {e:.2e}")
        assert e <= TOL[prec]
