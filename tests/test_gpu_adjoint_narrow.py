"""FP32 adjoint of lines far narrower than the grid's step, whose sums are their nearest
point's: x there has to be as good as the offset from it, wherever a wave's loops begin
(windows cut by the grid's ends, clumps, and even lists).  Against FP64 point by point.

x carries 5e-7 at most (fours of points from one conversion), a Lorentzian's value 1e-6
of it, its derivatives 2e-6; FP32 sums of 256 terms 5e-7: 3e-6 of the norm is asked for."""
import numpy as np
import pytest

import synth
from test_gpu_far import FP32, FP64, C, _Grid
from xs_helpers import X, log

pytestmark = pytest.mark.gpu
CASES = {"cut": (299.3, 0.2, 99, 3638, "inside", [C(300.0, 0.074, 4.0), C(3000.0, 0.029, 0.6)]),
         "short": (82.7, 0.01, 47, 330, "inside", [C(3000.0, 0.00017, 0.03)]),
         "clump": (195.9, 0.05, 1344, 8354, "clump", [C(3000.0, 0.00043, 25.0)]),
         "even": (4423.9, 0.01, 6120, 1822, "inside", [C(3000.0, 0.013, 25.0), C(1000.0, 0.51, 1.0)])}


@pytest.mark.parametrize("seed", [1, 2, 3])
@pytest.mark.parametrize("case", list(CASES))
def test_narrow_lorentzians(case, seed):
    import torch
    P = X()
    nu0, dnu, nb, n, kind, conds = CASES[case]
    rng = np.random.default_rng(seed)
    L, cut = dnu * nb, max(c.cutoff for c in conds)
    if kind == "inside":
        nu = nu0 - cut + (L + 2 * cut) * rng.random(n)
    else:
        nu = nu0 + L * (0.3 + 0.01 * rng.random(n))
        nu[::7] = nu0 + L * rng.random(nu[::7].size)
    nu = np.maximum(nu, 1e-3)
    El = np.concatenate([[0.0], rng.uniform(0.0, 3000.0, n - 1)])
    ds = P.DeviceStates.from_numpy(synth.States(np.concatenate([El, El + nu]), np.ones(2 * n)))
    i = np.arange(n, dtype=np.int32)
    dl = P.DeviceLines.from_numpy(synth.Lines(i + np.int32(n), i, (10.0 ** rng.uniform(-3, 1, n)).astype(np.float32),
                                              rng.uniform(0.02, 0.1, n).astype(np.float32), rng.uniform(0.3, 0.8, n).astype(np.float32)))
    g = torch.as_tensor(10.0 ** rng.uniform(-2, 2, (len(conds), nb)), device="cuda")
    out = []
    for prec, algo in ((FP32, 0), (FP64, 1)):
        plan = P.Plan(synth.LORENTZ, 0, 0, prec, _Grid(nu0, dnu, nb), conds, n, mass_amu=30.0, algo=algo)
        out.append({k: v.cpu().numpy() for k, v in plan.adjoint(ds, dl, g).items()})
        plan.close()
    for k in ("d_log_scale", "d_gamma_ref", "d_n_exp"):
        e = float(np.linalg.norm(out[0][k] - out[1][k]) / np.linalg.norm(out[1][k]))
        log(f"[narrow adjoint] {case} {seed} {k}: {e:.2e}")
        assert e <= 3e-6
