"""Intensities where the partition function is below 2^-1024, so that its
reciprocal is beyond FP64: a list whose lowest level lies far above zero (a part of
a molecule's states) at a low temperature.  Shifting all energies by the lowest one leaves
the intensities as they are and makes Q ordinary: that is the oracle's input.

Q is a sum of exponentials of up to 711 (each to 3 roundings of it, 2.4e-13) that
FP64 holds to 2e-15 here; the line's own power of two is exact to its own rounding: 1e-12
is asked for, FP32 form 1e-6."""
import numpy as np
import pytest

import oracle
import synth
from xs_helpers import X

pytestmark = pytest.mark.gpu
FP64, FP32 = 0, 1


@pytest.mark.parametrize("mode", [synth.ABSORPTION, synth.EMISSION])
@pytest.mark.parametrize("prec", [FP64, FP32])
def test_intensities(prec, mode):
    import torch
    P = X()
    T, n = 6.0, 2000
    E0 = 710.5 * T / oracle.c2()
    rng = np.random.default_rng(8)
    E = np.concatenate([[0.0], rng.uniform(200.0, 2500.0, n)])
    g = np.concatenate([[1.0], 2.0 * rng.integers(0, 50, n) + 1.0])
    up = np.arange(1, n + 1, dtype=np.int32)
    lo = np.zeros(n, np.int32)
    ln = synth.Lines(up, lo, (10.0 ** rng.uniform(-3, 3, n)).astype(np.float32))
    # (shifted as the library's FP64 inputs are: E + E0 rounded, less E0)
    Es = E + E0
    base = synth.States(Es - Es[0], g)
    Q, _ = oracle.partition(base, oracle.LTE, T)
    _, ref, _ = oracle.intensities(base, ln, mode, oracle.LTE, T, Q)
    st = synth.States(Es, g)
    class G:
        nu0, dnu, n_bins = 0.0, 1.0, 3001
    plan = P.Plan(synth.DOPPLER, mode, synth.LTE, prec, G, [synth.Condition(T, 0.0, 25.0)], n)
    ds, dl = P.DeviceStates.from_numpy(st), P.DeviceLines.from_numpy(ln)
    Qg, _ = plan.partition_function(ds)
    assert 0.0 < Qg.item() < 2.0 ** -1024
    S, ls = plan.line_intensities(ds, dl)
    torch.cuda.synchronize()
    S, ls = S[0].double().cpu().numpy(), ls.item()
    plan.close()
    assert np.all(np.isfinite(S))
    if prec == FP32:
        S, ref = S[S > 1e-30], ref[S > 1e-30]
        S = S * np.exp(ls) if np.isfinite(np.exp(ls)) else S
        tol = 1e-6
    else:
        big = ref > 1e-290
        S, ref, tol = S[big], ref[big], 1e-12
    assert S.size > 100
    assert np.max(np.abs(S - ref) / ref) <= tol
