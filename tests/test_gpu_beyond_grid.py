"""Grids inside longer lists: lines up to a cut-off beyond either end, most of
the list beyond it, enter the tiles and moments like the others.  Sigma against
the point-by-point gather, the adjoint against a scatter plan's, at the
tolerances of test_gpu_far; the oracle at those of the parity tests."""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_far import FP32, FP64, TOL, C, _Grid
from xs_helpers import X, log, rel_err

pytestmark = pytest.mark.gpu

# first point, step, points, conditions, lines, states' lifetimes (no moments): grids of a few leaves, of half
# a cut-off, of two; windows of several sizes in one table; a window of more cells than are kept beyond the grid
CASES = {
    "few": (1000.0, 0.01, 601, [C(1000.0, 1.0, 25.0)], 20011, False),
    "half": (1000.0, 0.01, 1300, [C(700.0, 0.1, 25.0)], 20011, False),
    "two": (1500.0, 0.01, 5003, [C(1000.0, 1.0, 25.0), C(300.0, 1e-3, 6.1), C(2000.0, 20.0, 60.0), C(500.0, 1.0, 1.0)],
            20011, False),
    "lifetimes": (1500.0, 0.01, 2503, [C(1000.0, 0.3, 25.0)], 20011, True),
    "beyond": (1000.0, 2e-5, 3001, [C(1000.0, 0.01, 25.0)], 8009, False),
}


def _inputs(case):
    P = X()
    nu0, dnu, n, conds, n_lines, tau = CASES[case]
    rng = np.random.default_rng(n)
    cut = max(c.cutoff for c in conds)
    nu = rng.uniform(nu0 - cut - 1.0, nu0 + (n - 1) * dnu + cut + 1.0, n_lines)
    El = np.concatenate([[0.0], rng.uniform(0.0, 5000.0, n_lines - 1)])
    st = synth.States(np.concatenate([El, El + nu]), np.ones(2 * n_lines))
    if tau:
        st.lifetime = 10.0 ** rng.uniform(-12.0, -9.0, 2 * n_lines)
    i = np.arange(n_lines, dtype=np.int32)
    ln = synth.Lines(i + np.int32(n_lines), i, (10.0 ** rng.uniform(-4, 2, n_lines)).astype(np.float32),
                     rng.uniform(0.02, 0.1, n_lines).astype(np.float32), rng.uniform(0.3, 0.8, n_lines).astype(np.float32))
    return P, _Grid(nu0, dnu, n), conds, st, ln


@pytest.mark.parametrize("case", list(CASES))
@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("profile", [synth.LORENTZ, synth.VOIGT, synth.BIN_LORENTZ, synth.BIN_VOIGT])
def test_sigma_against_points(profile, prec, case):
    import torch
    P, grid, conds, st, ln = _inputs(case)
    ds, dl = P.DeviceStates.from_numpy(st), P.DeviceLines.from_numpy(ln)
    plan = P.Plan(profile, 0, 0, prec, grid, conds, ln.n, mass_amu=30.0)
    got = plan.cross_section(ds, dl).clone()
    ref = plan.cross_section_noalloc(ds, dl, torch.empty_like(got)).clone()
    torch.cuda.synchronize()
    got, ref = got.cpu().numpy(), ref.cpu().numpy()
    plan.close()
    assert np.all(np.isfinite(got))
    for c in range(len(conds)):
        m = ref[c] > 0.0
        assert m.any() and np.all(got[c][~m] == 0.0)
        e = float(np.max(np.abs(got[c][m] - ref[c][m]) / ref[c][m]))
        log(f"[beyond] profile {profile} prec {prec} {case} c{c}: {e:.2e}")
        assert e <= TOL[prec]


@pytest.mark.parametrize("case", list(CASES))
@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("profile", [synth.LORENTZ, synth.VOIGT])
def test_adjoint_against_points(profile, prec, case):
    import torch
    P, grid, conds, st, ln = _inputs(case)
    ds, dl = P.DeviceStates.from_numpy(st), P.DeviceLines.from_numpy(ln)
    g = torch.as_tensor(np.random.default_rng(7).standard_normal((len(conds), grid.n_bins)), device="cuda")
    out = []
    for algo in (0, 1):
        plan = P.Plan(profile, 0, 0, prec, grid, conds, ln.n, mass_amu=30.0, algo=algo)
        r = plan.adjoint(ds, dl, g)
        torch.cuda.synchronize()
        out.append({k: v.cpu().numpy() for k, v in r.items()})
        plan.close()
    for k in out[0]:
        e = float(np.linalg.norm(out[0][k] - out[1][k]) / max(np.linalg.norm(out[1][k]), 1e-300))
        log(f"[beyond adjoint] profile {profile} prec {prec} {case} {k}: {e:.2e}")
        assert np.all(np.isfinite(out[0][k])) and e <= {FP64: 1e-10, FP32: 1e-4}[prec]
        assert np.array_equal(out[0][k] == 0.0, out[1][k] == 0.0)


@pytest.mark.parametrize("prec", [FP64, FP32])
def test_against_oracle(prec):
    import torch
    P, grid, conds, st, ln = _inputs("half")
    ds, dl = P.DeviceStates.from_numpy(st), P.DeviceLines.from_numpy(ln)
    plan = P.Plan(synth.VOIGT, 0, 0, prec, grid, conds, ln.n, mass_amu=30.0)
    got = plan.cross_section(ds, dl)[0].cpu().numpy()
    plan.close()
    c = conds[0]
    Q, _ = oracle.partition(st, oracle.LTE, c.T)
    nu, S, keep = oracle.intensities(st, ln, 0, oracle.LTE, c.T, Q)
    al, ga = oracle.widths(nu, ln, synth.VOIGT, c.T, c.P, 30.0)
    ref = oracle.sigma(nu, S, al, ga, synth.VOIGT, grid, c.cutoff)
    e, _, _ = rel_err(got, ref)
    assert e <= {FP64: 1e-10, FP32: 1e-4}[prec]
