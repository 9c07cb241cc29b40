"""The sort of 1025 lines, two blocks of 1024 keys, with 10-bit digits, whose
table lies in the records' wavenumbers; and the sizes around it that lie in the
partition function's partial sums (one block, few lines).  Spectra of one
intensity slot against the oracle at the tolerances of the parity tests, cooling functions as in
test_gpu_lines."""
import numpy as np
import pytest

import oracle
import synth
from xs_helpers import gpu_inputs, make_plan, rel_err

pytestmark = pytest.mark.gpu
FP64, FP32 = 0, 1


# 8192 to 16368 points: 512 to 1023 leaves of 16 points (FP32 Voigt), 10-bit keys
@pytest.mark.parametrize("n_lines", [300, 513, 514, 1024, 1025, 1026])
@pytest.mark.parametrize("prec", [FP64, FP32])
def test_spectrum(prec, n_lines):
    import torch
    wl = synth.workload("voigt_1e7", n_states=1000, n_lines=n_lines, nu_hi=120.0, seed=5 + n_lines)
    ln = wl.lines()
    plan = make_plan(wl, prec, ln.n)
    ds, dl = gpu_inputs(wl, ln)
    got = plan.cross_section(ds, dl)
    torch.cuda.synchronize()
    got = got[0].cpu().numpy()
    plan.close()
    ref = oracle.run_condition(wl, ln, wl.conditions[0]).sigma
    e, l1, _ = rel_err(got, ref)
    assert e <= {FP64: 1e-10, FP32: 1e-4}[prec]


@pytest.mark.parametrize("n_states, n_lines", [(600, 1025), (1000, 1025), (1000, 1026), (520, 400)])
def test_cooling(n_states, n_lines):
    wl = synth.workload("voigt_1e7", n_states=n_states, n_lines=n_lines, seed=n_states + n_lines)
    ln = wl.lines()
    T = np.array([40.0, 600.0, 3000.0])
    plan = make_plan(wl, FP64, ln.n)
    ds, dl = gpu_inputs(wl, ln)
    W, Q = (a.cpu().numpy() for a in plan.cooling_function(ds, dl, T))
    plan.close()
    Wr, Qr = oracle.cooling(wl.states, ln, T)
    assert np.max(np.abs(W - Wr) / Wr) <= 1e-12
    assert np.max(np.abs(Q - Qr) / Qr) <= 1e-12
