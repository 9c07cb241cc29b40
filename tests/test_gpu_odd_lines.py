"""Lines whose intensities or widths are not finite among ordinary ones: they go point by
point over their windows, the others through expansions as without them (up to
1024 such lines; beyond that every line goes point by point).  The table's conditions take
expansions, the near kernel and the gather.  Against the gather and the
scatter's adjoint: the same points and gradients are finite, at the tolerances of
test_gpu_far."""
import numpy as np
import pytest

import synth
from test_gpu_far import FP32, FP64, TOL, C, _Grid
from xs_helpers import X, gpu_inputs, log, workload

pytestmark = pytest.mark.gpu
CONDS = [C(900.0, 1.0, 25.0), C(300.0, 0.2, 12.5), C(500.0, 1.0, 2.0), C(700.0, 1.0, 5.7)]


def _lines(kind):
    wl = workload("voigt_1e7", n_states=20000, n_lines=30011, nu_hi=600.0, seed=4242)
    ln = wl.lines().take(np.arange(30011))
    ln.einstein_a, ln.gamma_ref, ln.n_exp = (a.copy() for a in (ln.einstein_a, ln.gamma_ref, ln.n_exp))
    if kind == "inf":
        ln.einstein_a[[17, 5000]] = np.inf
    elif kind == "nan":
        ln.einstein_a[[17, 5000, 5001]] = np.nan
    elif kind == "widths":
        ln.gamma_ref[[11, 700]] = np.nan
        ln.gamma_ref[12] = np.inf
        ln.n_exp[13] = np.nan
        ln.n_exp[[14, 900, 901]] = np.inf   # widths of zero above T_ref, infinite below
        ln.n_exp[15] = -np.inf
    else:  # more than the list of them holds, in a part of the grid
        wl_nu = wl.states.energy[ln.upper] - wl.states.energy[ln.lower]
        i = np.flatnonzero(wl_nu < 60.0)[:1500]
        assert i.size == 1500
        ln.einstein_a[i] = np.nan
    return wl, ln


@pytest.mark.parametrize("kind", ["inf", "nan", "widths", "many"])
@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("profile", [synth.LORENTZ, synth.VOIGT, synth.BIN_VOIGT])
def test_sigma(profile, prec, kind):
    import torch
    if prec == FP32 and kind == "inf":
        pytest.skip("an infinite intensity is the FP32 form's scale: no point is finite with or without expansions")
    P = X()
    wl, ln = _lines(kind)
    ds, dl = gpu_inputs(wl, ln)
    plan = P.Plan(profile, 0, 0, prec, _Grid(0.0, 0.01, 60001), CONDS, ln.n, mass_amu=wl.mass_amu)
    got = plan.cross_section(ds, dl).clone()
    again = plan.cross_section(ds, dl).clone()
    ref = plan.cross_section_noalloc(ds, dl, torch.empty_like(got)).clone()
    torch.cuda.synchronize()
    assert torch.equal(torch.nan_to_num(got, nan=-1.0), torch.nan_to_num(again, nan=-1.0))
    got, ref = got.cpu().numpy(), ref.cpu().numpy()
    plan.close()
    for c in range(len(CONDS)):
        fin = np.isfinite(ref[c])
        assert 0 < fin.sum() < fin.size or kind == "widths"
        assert np.array_equal(np.isfinite(got[c]), fin)
        m = fin & (ref[c] > 0.0)
        e = float(np.max(np.abs(got[c][m] - ref[c][m]) / ref[c][m]))
        log(f"[odd] profile {profile} prec {prec} {kind} c{c}: {e:.2e}")
        assert e <= TOL[prec]


@pytest.mark.parametrize("kind", ["nan", "widths", "many"])
@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("profile", [synth.LORENTZ, synth.VOIGT])
def test_adjoint(profile, prec, kind):
    import torch
    P = X()
    wl, ln = _lines(kind)
    ds, dl = gpu_inputs(wl, ln)
    g = torch.as_tensor(np.random.default_rng(7).standard_normal((len(CONDS), 60001)), device="cuda")
    out = []
    for algo in (0, 1):
        plan = P.Plan(profile, 0, 0, prec, _Grid(0.0, 0.01, 60001), CONDS, ln.n, mass_amu=wl.mass_amu, algo=algo)
        r = plan.adjoint(ds, dl, g)
        torch.cuda.synchronize()
        out.append({k: r[k].cpu().numpy() for k in ("d_log_scale", "d_gamma_ref", "d_n_exp")})
        plan.close()
    for k in out[0]:
        a, b = out[0][k], out[1][k]
        fin = np.isfinite(b)
        assert np.array_equal(np.isfinite(a), fin) and fin.sum() > 28000
        e = float(np.linalg.norm(a[fin] - b[fin]) / np.linalg.norm(b[fin]))
        log(f"[odd adjoint] profile {profile} prec {prec} {kind} {k}: {e:.2e}")
        assert e <= {FP64: 1e-10, FP32: 1e-4}[prec]


@pytest.mark.parametrize("prec", [FP64, FP32])
def test_widths_from_lifetimes_alone(prec):
    """Lorentzians without pressure width whose lifetimes give them one are ordinary lines."""
    import torch
    P = X()
    wl, ln = _lines("widths")
    ln.gamma_ref = np.zeros_like(ln.gamma_ref)
    ln.n_exp = np.full_like(ln.n_exp, 0.5)
    st = synth.States(wl.states.energy, wl.states.g_tot,
                      lifetime=10.0 ** np.random.default_rng(2).uniform(-12.0, -9.0, wl.states.n))
    st.lifetime[ln.upper[[40, 41]]] = np.inf  # and a few of no width at all
    ds, dl = P.DeviceStates.from_numpy(st), P.DeviceLines.from_numpy(ln)
    plan = P.Plan(synth.LORENTZ, 0, 0, prec, _Grid(0.0, 0.01, 60001), CONDS[:2], ln.n, mass_amu=wl.mass_amu)
    got = plan.cross_section(ds, dl).clone()
    ref = plan.cross_section_noalloc(ds, dl, torch.empty_like(got)).clone()
    torch.cuda.synchronize()
    got, ref = got.cpu().numpy(), ref.cpu().numpy()
    plan.close()
    fin = np.isfinite(ref)
    assert fin.any() and np.array_equal(np.isfinite(got), fin)
    m = fin & (ref > 0.0)
    assert np.max(np.abs(got[m] - ref[m]) / ref[m]) <= TOL[prec]


@pytest.mark.parametrize("prec", [FP64, FP32])
def test_passes_and_adjoints_in_turn(prec):
    """A pass with expansions hides the lines in the records, the adjoint needs them: the
    same values whichever ran before."""
    import torch
    P = X()
    wl, ln = _lines("nan")
    ds, dl = gpu_inputs(wl, ln)
    n = 60001
    plan = P.Plan(synth.VOIGT, 0, 0, prec, _Grid(0.0, 0.01, n), CONDS, ln.n, mass_amu=wl.mass_amu)
    g = torch.as_tensor(np.random.default_rng(7).standard_normal((len(CONDS), n)), device="cuda")
    same = lambda a, b: torch.equal(a.view(torch.int64), b.view(torch.int64))
    plan.prepare(ds, dl)
    adj = {k: v.clone() for k, v in plan.profile_adjoint(ds, dl, g).items()}
    sig = plan.profile().clone()
    adj2 = {k: v.clone() for k, v in plan.profile_adjoint(ds, dl, g).items()}
    sig2 = plan.profile().clone()
    sig3 = plan.profile().clone()
    torch.cuda.synchronize()
    assert torch.isnan(adj["d_log_scale"]).sum().item() == 3 and torch.isnan(sig).any()
    assert same(sig, sig2) and same(sig, sig3)
    assert all(same(adj[k], adj2[k]) for k in adj)
    plan.close()
