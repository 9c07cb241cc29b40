"""Expansions with what else a plan can be given: two-temperature and custom-density
populations, negative intensities among them, log scales, emission; and cotangents that are
not finite.  Against the gather and the scatter's adjoint.  Sigma with intensities of one sign at the
tolerances of test_gpu_far; with both signs their sums can cancel, and the error is measured
against the sum of magnitudes, which the same list with A of one sign bounds."""
import numpy as np
import pytest

import synth
from test_gpu_far import FP32, FP64, TOL, C, _Grid
from xs_helpers import X, log

pytestmark = pytest.mark.gpu


def _manifold(n_lines, density=False):
    P = X()
    rng = np.random.default_rng(31)
    ns = 4000
    v = rng.integers(0, 6, ns).astype(np.int32)
    ev = 1500.0 * np.arange(6) - 8.0 * np.arange(6) ** 2
    E = ev[v] + rng.uniform(0.0, 1200.0, ns)
    E[0], v[0] = 0.0, 0
    st = synth.States(E, 2.0 * rng.integers(0, 40, ns) + 1.0, v, ev)
    if density:
        st.n_vib = np.array([1.0, 3.0, 0.2, 5.0, 0.0, 1.0])
    up, lo = rng.integers(0, ns, (2, 40 * n_lines)).astype(np.int32)
    nu = E[up] - E[lo]
    k = np.flatnonzero((nu > 0.5) & (nu < 600.0))[:n_lines]
    assert k.size == n_lines
    ln = synth.Lines(up[k], lo[k], (10.0 ** rng.uniform(-4, 2, n_lines)).astype(np.float32),
                     rng.uniform(0.02, 0.1, n_lines).astype(np.float32), rng.uniform(0.3, 0.8, n_lines).astype(np.float32))
    return P, st, ln, rng


@pytest.mark.parametrize("mode", [synth.ABSORPTION, synth.EMISSION])
@pytest.mark.parametrize("pop", [synth.NLTE_2T, synth.NLTE_DENSITY])
@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("profile", [synth.VOIGT, synth.LORENTZ, synth.BIN_VOIGT])
def test_populations(profile, prec, pop, mode):
    import torch
    P, st, ln, rng = _manifold(30011, pop == synth.NLTE_DENSITY)
    conds = [synth.Condition(0.0, 1.0, 25.0, 6000.0, 500.0), synth.Condition(0.0, 0.1, 12.5, 300.0, 900.0)]
    ds = P.DeviceStates.from_numpy(st)
    dl = P.DeviceLines.from_numpy(ln, log_scale=rng.uniform(-3.0, 3.0, ln.n).astype(np.float32))
    plan = P.Plan(profile, mode, pop, prec, _Grid(0.0, 0.01, 60001), conds, ln.n, mass_amu=30.0)
    S, _ = plan.line_intensities(ds, dl)
    got = plan.cross_section(ds, dl).clone()
    ref = plan.cross_section_noalloc(ds, dl, torch.empty_like(got)).clone()
    torch.cuda.synchronize()
    got, ref = got.cpu().numpy(), ref.cpu().numpy()
    negative = bool((S < 0).any().item())
    plan.close()
    if pop == synth.NLTE_2T and mode == synth.ABSORPTION:
        assert negative
    for c in range(2):
        # the sum of magnitudes, from below: where intensities have both signs, the envelope over 41 points
        scale = np.abs(ref[c])
        if negative:
            scale = np.maximum.reduce([np.roll(scale, q) for q in range(-20, 21)])
        m = scale > 0.0
        e = float(np.max(np.abs(got[c][m] - ref[c][m]) / scale[m]))
        log(f"[populations] profile {profile} prec {prec} pop {pop} mode {mode} c{c} negative {negative}: {e:.2e}")
        assert e <= TOL[prec] * (10.0 if negative else 1.0)


@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("profile", [synth.VOIGT, synth.LORENTZ])
def test_cotangent_not_finite(profile, prec, bad):
    """Lines whose windows hold the point have gradients that are not finite, the others the
    scatter's."""
    import torch
    P, st, ln, rng = _manifold(30011)
    st = synth.States(st.energy, st.g_tot)
    ds, dl = P.DeviceStates.from_numpy(st), P.DeviceLines.from_numpy(ln)
    g = rng.standard_normal((1, 60001))
    g[0, [20000, 40003]] = bad
    g = torch.as_tensor(g, device="cuda")
    out = []
    for algo in (0, 1):
        plan = P.Plan(profile, 0, 0, prec, _Grid(0.0, 0.01, 60001), [C(700.0, 1.0, 25.0)], ln.n, mass_amu=30.0, algo=algo)
        r = plan.adjoint(ds, dl, g)
        torch.cuda.synchronize()
        out.append({k: v.cpu().numpy() for k, v in r.items()})
        plan.close()
    nu = st.energy[ln.upper] - st.energy[ln.lower]
    hit = np.minimum(np.abs(nu - 200.0), np.abs(nu - 400.03)) < 24.99
    clear = np.minimum(np.abs(nu - 200.0), np.abs(nu - 400.03)) > 25.01
    for k in ("d_log_scale", "d_gamma_ref", "d_n_exp"):
        a, b = out[0][k], out[1][k]
        assert not np.isfinite(a[hit]).any() and not np.isfinite(b[hit]).any()
        assert np.isfinite(a[clear]).all()
        e = float(np.linalg.norm(a[clear] - b[clear]) / np.linalg.norm(b[clear]))
        assert e <= {FP64: 1e-10, FP32: 1e-4}[prec], (k, e)
