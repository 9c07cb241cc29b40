"""Gaussian profiles a line to a lane, against the gather of the allocation-free call.

Both evaluate the same points with the same formula.  Far out a value magnifies
the error of x by 2 x^2 ln 2: FP64 form |x| <= 33, x stepped along a row by the
gather to about 1.5e-12 of itself, 2.3e-9 of the value, 1e-8 is asked for down to
1e-250 of the largest; FP32 form |x| <= 12.7, x and x^2 each to 1.2e-7 on either side,
5e-5 of the value and for bin means as much again for erfc, 2e-4 is asked for down to
1e-30.  Points that no line reaches are zero on both sides.
"""
import numpy as np
import pytest

import synth
from test_gpu_far import FP32, FP64, C, _Grid
from xs_helpers import X, gpu_inputs, workload

pytestmark = pytest.mark.gpu

# grid, conditions, lines, fixed half-width: a core inside one leaf, several leaves, more
# than a tile; a line or two to a tile, and tiles split into parts; a ragged end
CASES = {
    "narrow": ((250.3, 0.01, 20011), [C(300.0, 0.0, 25.0)], 30011, 0.004),
    "tiles": ((400.0, 0.001, 20001), [C(3000.0, 0.0, 25.0), C(200.0, 0.0, 0.7), C(900.0, 0.0, 25.0)], 60011, 0.21),
    "few": ((0.0, 0.01, 60001), [C(1000.0, 0.0, 25.0)] * 9, 37, 0.02),
    "short": ((300.0, 0.05, 7), [C(2000.0, 0.0, 5.0)], 30011, 0.3),
}


@pytest.mark.parametrize("case", list(CASES))
@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("profile", [0, 1, 4, 5])
def test_gaussians_against_gather(profile, prec, case):
    import torch
    P = X()
    (nu0, dnu, n), conds, n_lines, hwhm = CASES[case]
    wl = workload("voigt_1e7", n_states=20000, n_lines=n_lines, nu_hi=600.0, seed=17)
    ln = wl.lines()
    ds, dl = gpu_inputs(wl, ln)
    plan = P.Plan(profile, 0, 0, prec, _Grid(nu0, dnu, n), conds, ln.n, mass_amu=wl.mass_amu, hwhm_fixed=hwhm)
    got = plan.cross_section(ds, dl).clone()
    ref = plan.cross_section_noalloc(ds, dl, torch.empty_like(got)).clone()
    acc = plan.cross_section(ds, dl, out=got.clone(), accumulate=True)
    torch.cuda.synchronize()
    got, ref, acc = (t.cpu().numpy() for t in (got, ref, acc))
    plan.close()
    for c in range(len(conds)):
        m = ref[c] > {FP64: 1e-250, FP32: 1e-30}[prec] * ref[c].max()
        assert m.any()
        assert np.max(np.abs(got[c][m] - ref[c][m]) / ref[c][m]) <= {FP64: 1e-8, FP32: 2e-4}[prec]
        assert np.max(got[c][~m], initial=0.0) <= {FP64: 1e-249, FP32: 1e-29}[prec] * ref[c].max()
    assert np.allclose(acc, 2.0 * got, rtol=1e-14, atol=0.0)
