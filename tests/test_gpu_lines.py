"""Line passes on the GPU at the sizes where they change form.

Sorting by key: one to three passes of 8, 9 or 10 bits, 1024 or 4096 keys a
block, the digit table scanned or added up by each block, and its three places
in the workspace.  The cooling function sorts lines by upper state, so its sums
are wrong if a line lands in another state's run; the states' number sets the
key's bits, the lines' the blocks.  Tolerance 1e-12 relative: the exponent
-c2 E (1/T) is at most two roundings from the oracle's quotient, 2 |x| 1.1e-16 <=
1.7e-13 for |x| <= 745, and all terms are positive.

Stick spectra: FP64 totals come from the output pass, FP32 ones and those of a
cross section from the pass before it; both have to count alike.
"""
import numpy as np
import pytest

import oracle
import synth
from xs_helpers import gpu_inputs, make_plan

pytestmark = pytest.mark.gpu
FP64, FP32 = 0, 1


@pytest.mark.parametrize("n_states, n_lines", [
    (1000, 1), (1000, 300), (200, 1023), (1000, 1024), (3000, 1025), (1000, 65536), (1000, 65537),
    (120000, 65537), (300000, 5000), (300000, 1048576), (120000, 1048577), (700000, 1048577), (1100000, 70000)])
def test_sort_sizes(n_states, n_lines):
    wl = synth.workload("voigt_1e7", n_states=n_states, n_lines=n_lines, seed=n_states + n_lines)
    ln = wl.lines()
    T = np.array([40.0, 600.0, 3000.0])
    plan = make_plan(wl, FP64, ln.n)
    ds, dl = gpu_inputs(wl, ln)
    W, Q = (a.cpu().numpy() for a in plan.cooling_function(ds, dl, T))
    Wr, Qr = oracle.cooling(wl.states, ln, T)
    assert np.max(np.abs(W - Wr) / Wr) <= 1e-12
    assert np.max(np.abs(Q - Qr) / Qr) <= 1e-12
    st = plan.stats()
    assert st["lines_kept"] + st["lines_invalid"] <= ln.n and st["lines_in"] == ln.n
    plan.close()


@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("n_lines", [1, 255, 257, 600000])
def test_totals_of_sticks_and_spectra(prec, n_lines):
    import torch
    wl = synth.workload("voigt_1e7", n_states=4000, n_lines=n_lines, seed=71)
    ln = wl.lines()
    plan = make_plan(wl, prec, ln.n)
    ds, dl = gpu_inputs(wl, ln)
    plan.prepare(ds, dl)
    torch.cuda.synchronize()
    a = plan.stats()
    S, ls = plan.line_intensities(ds, dl)
    torch.cuda.synchronize()
    b = plan.stats()
    for k in ("lines_in", "lines_kept", "window_pairs", "lines_invalid"):
        assert a[k] == b[k], k
    if prec == FP64:
        assert ls.item() == 0.0
    else:  # the largest intensity is the scale (rounded to FP32)
        assert abs(S.max().item() - 1.0) <= 2.0 ** -23
    plan.close()
