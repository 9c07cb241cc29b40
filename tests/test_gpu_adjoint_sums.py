"""FP32 sums of the adjoint's far part, which goes over hundreds of tiles where windows
are long: no more additions in a row than the 256 of the point-by-point blocks, which pass
to FP64 then (a tile's terms first, then the tiles).

Loss weights of one sign and lines wide against the grid (every term of d_log_scale has
one sign, those of the widths' gradients change sign once): a sum of 256 FP32 terms
carries up to 256 / 2 roundings of 6e-8 / sqrt(256) of it on average, 5e-7; 2e-6 of the
norm is asked for."""
import numpy as np
import pytest

import synth
from test_gpu_far import FP32, FP64, C, _Grid
from xs_helpers import X, log

pytestmark = pytest.mark.gpu
CASES = {"21bar": (0.002, 241119, C(3000.0, 21.0, 25.0)), "100bar": (0.005, 200003, C(3000.0, 100.0, 100.0)),
         "60bar": (0.001, 300007, C(1500.0, 60.0, 25.0))}


@pytest.mark.parametrize("case", list(CASES))
@pytest.mark.parametrize("profile", [synth.VOIGT, synth.LORENTZ])
def test_long_windows(profile, case):
    import torch
    P = X()
    dnu, n, cond = CASES[case]
    rng = np.random.default_rng(21)
    m = 30011
    nu = rng.uniform(0.5, dnu * (n - 1), m)
    El = np.concatenate([[0.0], rng.uniform(0.0, 8000.0, m - 1)])
    st = synth.States(np.concatenate([El, El + nu]), np.ones(2 * m))
    i = np.arange(m, dtype=np.int32)
    ln = synth.Lines(i + np.int32(m), i, (10.0 ** rng.uniform(-4, 0, m)).astype(np.float32),
                     rng.uniform(0.02, 0.1, m).astype(np.float32), rng.uniform(0.3, 0.8, m).astype(np.float32))
    ds, dl = P.DeviceStates.from_numpy(st), P.DeviceLines.from_numpy(ln)
    g = torch.as_tensor(10.0 ** rng.uniform(-2, 2, (1, n)), device="cuda")
    out = []
    for prec, algo in ((FP32, 0), (FP64, 1)):
        plan = P.Plan(profile, 0, 0, prec, _Grid(0.0, dnu, n), [cond], m, mass_amu=30.0, algo=algo)
        r = plan.adjoint(ds, dl, g)
        torch.cuda.synchronize()
        out.append({k: v.cpu().numpy() for k, v in r.items()})
        plan.close()
    worst = 0.0
    for k in ("d_log_scale", "d_gamma_ref", "d_n_exp"):
        e = float(np.linalg.norm(out[0][k] - out[1][k]) / np.linalg.norm(out[1][k]))
        log(f"[adjoint sums] profile {profile} {case} {k}: {e:.2e}")
        worst = max(worst, e)
    assert worst <= 2e-6
