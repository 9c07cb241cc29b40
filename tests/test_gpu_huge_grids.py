"""Outputs of more than 2^32 points, and conditions of more than 5e8: more blocks than
one dimension of a launch takes.  Parts of the spectrum against plans of these parts
alone, on steps that are powers of two, so that the grid points are the same numbers."""
import numpy as np
import pytest

import synth
from test_gpu_far import FP32, C, _Grid
from xs_helpers import X

pytestmark = pytest.mark.gpu


def _list(nu, seed):
    import torch
    P = X()
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    n = nu.shape[0]
    E = torch.cat([torch.zeros(1, dtype=torch.float64, device="cuda"), nu])
    A = (10.0 ** (torch.rand(n, device="cuda", generator=g) * 6.0 - 4.0)).float()
    i = torch.arange(1, n + 1, dtype=torch.int32, device="cuda")
    return P.DeviceStates(E, torch.ones_like(E)), P.DeviceLines(i, torch.zeros_like(i), A)


def _part(P, profile, conds, dnu, k0, k1, st, ln, mass=30.0):
    import torch
    plan = P.Plan(profile, 0, 0, FP32, _Grid(k0 * dnu, dnu, k1 - k0), conds, ln.n, mass_amu=mass)
    out = torch.empty((len(conds), k1 - k0), dtype=torch.float64, device="cuda")
    sig = plan.cross_section(st, ln, out=out)
    torch.cuda.synchronize()
    plan.close()
    return sig


def test_many_output_points():
    """16 conditions x 2.8e8 points, Doppler (a line to a lane)."""
    import torch
    P = X()
    dnu, n = 2.0 ** -14, 280_000_123
    nu = torch.linspace(1.0, n * dnu - 1.0, 4001, dtype=torch.float64, device="cuda")
    st, ln = _list(nu, 1)
    conds = [C(300.0 + 100.0 * i, 0.0, 1.0) for i in range(16)]
    plan = P.Plan(synth.DOPPLER, 0, 0, FP32, _Grid(0.0, dnu, n), conds, ln.n, mass_amu=30.0)
    sig = plan.cross_section(st, ln)
    torch.cuda.synchronize()
    for k0 in (0, 140_000_000, n - 300_011):
        ref = _part(P, synth.DOPPLER, conds, dnu, k0, k0 + 300_011, st, ln)
        got = sig[:, k0:k0 + 300_011]
        assert (ref > 0).any()
        m = ref > 1e-30 * ref.max()
        assert ((got - ref).abs()[m] / ref[m]).max().item() <= 2e-4
    plan.close()
    del sig
    torch.cuda.empty_cache()


@pytest.mark.parametrize("lifetimes", [False, True])
def test_many_points_of_one_condition(lifetimes):
    """6e8 points through expansions, with and without moments (lines with lifetimes go one by one)."""
    import torch
    P = X()
    dnu, n, n_lines = 2.0 ** -15, 600_000_077, 37_600_000
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    nu = 0.1 + (n * dnu - 0.2) * torch.rand(n_lines, dtype=torch.float64, device="cuda", generator=g)
    st, ln = _list(nu, 2)
    if lifetimes:
        st.lifetime = torch.full_like(st.energy, 1e-10)
    conds, mass = [C(300.0, 0.05, 0.05)], 3000.0  # cores of 650 points at the end, windows of 1638
    plan = P.Plan(synth.VOIGT, 0, 0, FP32, _Grid(0.0, dnu, n), conds, n_lines, mass_amu=mass)
    sig = plan.cross_section(st, ln)
    torch.cuda.synchronize()
    for k0 in (0, 300_000_000, n - 200_003):
        k1 = k0 + 200_003
        ref = _part(P, synth.VOIGT, conds, dnu, k0, k1, st, ln, mass)
        got = sig[:, k0:k1]
        m = ref > 0
        assert m.any() and ((got - ref).abs()[m] / ref[m]).max().item() <= 1e-5
    plan.close()
    del sig
    torch.cuda.empty_cache()
