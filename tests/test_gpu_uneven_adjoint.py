"""Adjoints of uneven lists: waves of crowded lines go through tiles, those whose lines lie
far apart point by point, with the same gradients as a scatter plan's at the tolerances of
test_gpu_far.  Lists with a crowded part and a few lines all over the grid, windows of
several sizes in a table, and the even lists around the line between the two."""
import numpy as np
import pytest

import synth
from test_gpu_far import FP32, FP64, C, _Grid
from xs_helpers import X, log

pytestmark = pytest.mark.gpu
CASES = {"crowded": (30011, 90, 900.0), "few": (20011, 1, 900.0), "even": (0, 20011, 200.0), "sparse": (0, 13001, 200.0)}
CONDS = [C(900.0, 1.0, 25.0), C(300.0, 0.2, 12.5), C(500.0, 1.0, 2.0)]


@pytest.mark.parametrize("case", list(CASES))
@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("profile", [synth.LORENTZ, synth.VOIGT])
def test_adjoint(profile, prec, case):
    import torch
    P = X()
    crowd, rest, hi = CASES[case]
    rng = np.random.default_rng(11)
    nu = np.concatenate([rng.uniform(0.4 * hi, 0.42 * hi, crowd), rng.uniform(0.5, hi, rest)])
    n = nu.size
    El = np.concatenate([[0.0], rng.uniform(0.0, 5000.0, n - 1)])
    st = synth.States(np.concatenate([El, El + nu]), np.ones(2 * n))
    i = np.arange(n, dtype=np.int32)
    ln = synth.Lines(i + np.int32(n), i, (10.0 ** rng.uniform(-4, 2, n)).astype(np.float32),
                     rng.uniform(0.02, 0.1, n).astype(np.float32), rng.uniform(0.3, 0.8, n).astype(np.float32))
    ds, dl = P.DeviceStates.from_numpy(st), P.DeviceLines.from_numpy(ln)
    nb = int(hi / 0.01) + 1
    g = torch.as_tensor(rng.standard_normal((len(CONDS), nb)), device="cuda")
    out = []
    for algo in (0, 1):
        plan = P.Plan(profile, 0, 0, prec, _Grid(0.0, 0.01, nb), CONDS, n, mass_amu=30.0, algo=algo)
        r = plan.adjoint(ds, dl, g)
        torch.cuda.synchronize()
        out.append({k: v.cpu().numpy() for k, v in r.items()})
        plan.close()
    for k in out[0]:
        e = float(np.linalg.norm(out[0][k] - out[1][k]) / max(np.linalg.norm(out[1][k]), 1e-300))
        log(f"[uneven] profile {profile} prec {prec} {case} {k}: {e:.2e}")
        assert np.all(np.isfinite(out[0][k])) and e <= {FP64: 1e-10, FP32: 1e-4}[prec]
        assert np.array_equal(out[0][k] == 0.0, out[1][k] == 0.0)
