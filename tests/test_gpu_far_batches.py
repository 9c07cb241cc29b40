"""The tile expansions' rows lie in the partial rows' space, for as many conditions at a time
as fit: tables of several batches give each condition the values it has by itself, and
the workspace of a plan with expansions is that of one without, but for the table of cells beyond
the grid, the odd lines' list and the partial sums."""
import numpy as np
import pytest

import synth
from test_gpu_far import FP32, FP64, C, _Grid
from xs_helpers import X

pytestmark = pytest.mark.gpu


def _list(n, hi, seed):
    import torch
    P = X()
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    U = lambda: torch.rand(n, dtype=torch.float64, device="cuda", generator=g)
    nu, El = 0.5 + (hi - 0.5) * U(), 5000.0 * U()
    El[0] = 0.0
    E = torch.cat([El, El + nu])
    i = torch.arange(n, dtype=torch.int32, device="cuda")
    A = (10.0 ** (6.0 * U() - 4.0)).float()
    return P.DeviceStates(E, torch.ones_like(E)), P.DeviceLines(i + n, i, A, (0.02 + 0.08 * U()).float(),
                                                               (0.3 + 0.5 * U()).float())


# points, conditions, lines: FP32 5 doubles a point and condition, FP64 2.1, of 1.3e8; the adjoint 1.1 and 2.1
@pytest.mark.parametrize("prec, n, nc, lines", [(FP32, 1_000_003, 40, 120_007), (FP64, 1_500_001, 60, 200_003)])
@pytest.mark.parametrize("profile", [synth.VOIGT, synth.LORENTZ])
def test_batches(profile, prec, n, nc, lines):
    import torch
    P = X()
    st, ln = _list(lines, 0.01 * (n - 1), 3)
    conds = [C(300.0 + 20.0 * i, 0.1 + 0.1 * i, 25.0 if i % 3 else 40.0) for i in range(nc)]
    plan = P.Plan(profile, 0, 0, prec, _Grid(0.0, 0.01, n), conds, lines, mass_amu=30.0)
    sig = plan.cross_section(st, ln)
    again = plan.cross_section(st, ln)
    assert torch.equal(sig, again)
    del again
    for c in (0, 1, nc // 2, nc - 1):
        one = P.Plan(profile, 0, 0, prec, _Grid(0.0, 0.01, n), [conds[c]], lines, mass_amu=30.0)
        want = one.cross_section(st, ln)[0]
        m = want > 0
        e = ((sig[c] - want).abs()[m] / want[m]).max().item()
        assert e <= {FP64: 1e-12, FP32: 1e-6}[prec], (c, e)
        one.close()
    plan.close()


@pytest.mark.parametrize("prec, n, nc, lines", [(FP32, 2_000_003, 64, 150_007), (FP64, 1_500_001, 48, 200_003)])
def test_adjoint_batches(prec, n, nc, lines):
    """The gradients of a table against the sums of its conditions' own."""
    import torch
    P = X()
    st, ln = _list(lines, 0.01 * (n - 1), 4)
    conds = [C(300.0 + 20.0 * i, 0.1 + 0.1 * i, 25.0) for i in range(nc)]
    g = torch.randn((nc, n), dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    plan = P.Plan(synth.VOIGT, 0, 0, prec, _Grid(0.0, 0.01, n), conds, lines, mass_amu=30.0)
    r = {k: v.clone() for k, v in plan.adjoint(st, ln, g).items()}
    plan.close()
    total = {k: torch.zeros_like(r[k]) for k in ("d_log_scale", "d_gamma_ref", "d_n_exp")}
    one = P.Plan(synth.VOIGT, 0, 0, prec, _Grid(0.0, 0.01, n), [conds[0]], lines, mass_amu=30.0)
    for c in range(nc):
        one.set_conditions([conds[c]])
        q = one.adjoint(st, ln, g[c:c + 1])
        for k in total:
            total[k] += q[k]
        if prec == FP64:
            for k in ("dT", "dP"):
                assert abs(q[k][0].item() - r[k][c].item()) <= 1e-9 * abs(r[k][c].item())
    one.close()
    for k in total:
        e = ((total[k] - r[k]).norm() / r[k].norm()).item()
        assert e <= {FP64: 1e-12, FP32: 1e-6}[prec], (k, e)


@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("n, nc", [(2_000_001, 1), (1_000_001, 48), (20_000_001, 2)])
def test_workspace(prec, n, nc):
    P = X()
    conds = [C(300.0, 1.0, 25.0)] * nc
    size = [P.Plan(synth.VOIGT, 0, 0, prec, _Grid(0.0, 0.01, n), conds, 1000, algo=a) for a in (0, 1)]
    gather, scatter = (p.ws.numel() for p in size)
    for p in size:
        p.close()
    assert gather - scatter <= (1 << 20) + n / 4 + 8192 + 1024 * 16


def test_one_long_condition():
    """A condition whose rows and moments do not fit together has rows of its own."""
    import torch
    P = X()
    n, lines = 40_000_001, 2_600_003
    dnu = 2.0 ** -11
    st, ln = _list(lines, dnu * (n - 1), 5)
    cond = [C(300.0, 0.3, 1.5)]
    plan = P.Plan(synth.VOIGT, 0, 0, FP32, _Grid(0.0, dnu, n), cond, lines, mass_amu=300.0)
    sig = plan.cross_section(st, ln)
    g = torch.randn((1, n), dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(2))
    r = {k: v.clone() for k, v in plan.adjoint(st, ln, g).items()}
    plan.close()
    for k0 in (0, 17_000_000, n - 100_003):
        part = P.Plan(synth.VOIGT, 0, 0, FP32, _Grid(k0 * dnu, dnu, 100_003), cond, lines, mass_amu=300.0)
        want = part.cross_section(st, ln)[0]
        got = sig[0, k0:k0 + 100_003]
        m = want > 0
        assert ((got - want).abs()[m] / want[m]).max().item() <= 1e-5
        part.close()
    other = P.Plan(synth.VOIGT, 0, 0, FP32, _Grid(0.0, dnu, n), cond, lines, mass_amu=300.0, algo=1)
    want = other.adjoint(st, ln, g)
    other.close()
    for k in r:
        assert ((r[k] - want[k]).norm() / want[k].norm()).item() <= 1e-4
