#!/usr/bin/env python3
"""Benchmark of the line-list cross-section path on one MI355X.

Workload the metric is quoted on (the 1e7-line Voigt case): LTE absorption,
1e6 states (E exponential, mean 8000 cm^-1, cap 40000; J 0-120), 1e7
transitions (nu in (0, 20000], A 10^U(-8,3), gamma_ref 10^U(log 0.02, log 0.1),
n_exp U(0.3, 0.8)), T = 2000 K, P = 1 bar, mass 30 amu, Voigt profile, grid
0-20000 cm^-1 step 0.01 (2,000,001 points), cut-off 25 cm^-1.  Seeded
synthetic data (generator ``synth``), uploaded to HBM before timing.

One step = the whole hot path once, FP32 log-scaled form:
  prepare (Q(T), S_i, bucketing, records) -> profile pass (sigma) ->
  dL/dsigma of L = sum_k w_k (sigma_k - t_k)^2 (target t at 1700 K, 0.8 bar) ->
  adjoint pass (dL/dT, dL/dP, dL/dgamma_ref, dL/dn_exp, dL/dlog_scale).
``value`` = profile evaluations per second over the step (forward and
adjoint window evaluations: each kept line times its window bins on the
grid, counted exactly by the library).  Also reported: the same step in the
FP64 form (speedup FP32 / FP64, its own rooflines), the adjoint / forward
time ratio, the line-parallel atomic scatter, binned and pseudo-Voigt
profiles, lifetime widths, the cooling function, the roofline of the
dominant kernel, HBM figures against 8 TB/s and a measured device copy,
board power and shader clock sampled during the timed work, the 48-condition
grid at its full 1e8 lines (autotuned, captured graph, FP32 and FP64), the
two-temperature emission workload at its full 1e9 lines streamed in 10
chunks, and the oracle timed on the host (``cpu_baseline``).
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

# Algorithmic work per profile evaluation: the flops of the formula the method
# needs at that evaluation (FMA = 2; add, mul, reciprocal, division, exp2 = 1),
# by the Voigt region rho = x^2 + y^2 of the evaluation (the same regions the
# kernels use).  (rho threshold, flops) from the outermost region inward:
#   forward FP32: 1 node pair: x = fma(r,a,-b) 2, s = fma(x,x,h) 2,
#                 d = fma(s,s,c) 2, rcp 1, numerator fma 2, accumulate fma 2
#                 = 11; 2 pairs: x 2, per pair s, d, rcp, numerator, product 8,
#                 sum and accumulate 2 = 20;
#                 core: Weideman's rational approximation with N = 24 terms in
#                 FP64 (q and Z 14; the degree-23 polynomial by the real
#                 quadratic-divisor recurrence, 22 steps of 2 FMAs plus setup
#                 and the final product, 4 N + 1 = 97; Re w 11; x, scale and
#                 accumulate 4) = 126.
#   forward FP64: 1 pair 11; the three-point rule (one pair and the node at
#                 0, one division: x 2, s 2, N 4, D 5, division 1,
#                 accumulate 1) 15; 2 pairs (one division) 19; 3/4/6 pairs
#                 30/39/57; core N = 40: 14 + 161 + 11 + 4 = 190.
#   adjoint FP32: in a wave whose lines all have y^2 at most half the
#                 region's rho bound (the block-summed form), x 2 and per
#                 pair s 2, d 2, rcp 1, g/d and g/d^2 2, sums of g/d, g s/d,
#                 g/d^2, g s/d^2 6 = 13: 1 pair 15, 2 pairs 28 (3 pairs 41);
#                 in the other waves 1 pair takes the u-form: x 2, u 1, d 3,
#                 rcp 1, g/d 1, g u/d^2 2, sums of g/d, g u/d, g u/d^2,
#                 g u^2/d^2 6 = 16; 2 pairs the per-point form: x 2, u 1, per pair
#                 d, rcp, e, t 12 and their K-weighted sums 8, four
#                 accumulations 8 = 51; core: w (N = 24, both
#                 parts: 14 + 97 + 17), w' = -2zw + 2i/sqrt(pi) and Re G 13,
#                 x, |z|^2 5, three accumulations 6 = 152.
#   adjoint FP64: 1/2/3 pairs 15/28/41 (other waves 16/51/71); the
#                 three-point rule 22 (x 2, its pair 13, the node at 0: v 2,
#                 rcp 1, g/v 1, sums of g/v and g/v^2 3; per-point form, as
#                 two pairs, 51); 4/6 pairs (general form) 113/161;
#                 core N = 40: 14 + 161 + 17 + 24 = 216.
FLOP_REGIONS = {
    ("fwd", "f32"): [(900.0, 11), (64.0, 20), (0.0, 126)],
    ("fwd", "f64"): [(9.0e6, 11), (4.5e4, 15), (4000.0, 19), (400.0, 30), (144.0, 39), (64.0, 57), (0.0, 190)],
    ("adj", "f32"): [(900.0, 15), (64.0, 28), (0.0, 152)],
    ("adj", "f64"): [(9.0e6, 15), (4.5e4, 22), (4000.0, 28), (400.0, 41), (144.0, 113), (64.0, 161), (0.0, 216)],
}
# adjoint regions with a block-summed form (the table's figure): the flops of
# the per-point form used in the other waves
ADJ_POINT_FLOPS = {"f32": [16, 51], "f64": [16, 51, 51, 71]}
# MI355X vector peaks, no packed-FP32 (the kernels are compiled without packed FP32):
# 256 CU x 4 SIMD x 16 lanes x 2 flop (FMA) x 2.4 GHz = 78.6 TFLOP/s for FP32
# and FP64 alike.  The published 157.3 TFLOP/s FP32 figure needs packed math.
PEAK_TFLOPS = {"f32": 78.6, "f64": 78.6}
KERNEL_SOURCES = ["paper_2609_17273_amd/csrc/k_profile.hip", "paper_2609_17273_amd/csrc/k_adjoint.hip",
                  "paper_2609_17273_amd/csrc/k_common.h", "paper_2609_17273_amd/csrc/k_lines.hip",
                  "paper_2609_17273_amd/csrc/k_near.hip", "paper_2609_17273_amd/csrc/k_far.hip",
                  "paper_2609_17273_amd/csrc/k_voigt.h", "paper_2609_17273_amd/csrc/far_geometry.h",
                  "paper_2609_17273_amd/csrc/far_tables.h", "paper_2609_17273_amd/csrc/sort_plan.h",
                  "paper_2609_17273_amd/csrc/xsec_internal.h"]

# The Lorentzian and Voigt passes take the tiles away from a line through
# expansions and cells of lines, so they run far fewer operations than one
# evaluation per window point.  Rates and flops are reported per window point all
# the same (the work a caller asks for), which makes `frac` no utilisation: it can
# exceed 1.
EXPANSION_NOTE = ("flops of one evaluation per (line, window point); tiles away from a line are expanded, so far fewer "
                  "are run and frac is not a utilisation (it may exceed 1)")
FWD_KERNELS = "k_near + k_far_leaves/moments/cells + k_far_finish (%s, Voigt)"
ADJ_KERNELS = "k_adj_moments/cut + k_adjoint near and far (%s, Voigt)"


def region_fractions(wl, lines, cond):
    """Fraction of the window evaluations in each Voigt region, from the closed
    form of |x| < sqrt(rho - y^2) per line (grid clipping ignored)."""
    import numpy as np
    c, kb, amu = 2.99792458e10, 1.380649e-16, 1.66053906660e-24
    E = wl.states.energy
    nu = E[lines.upper] - E[lines.lower]
    pos = nu > 0
    nu = nu[pos]
    alpha = nu / c * np.sqrt(2.0 * kb * cond.T * np.log(2.0) / (wl.mass_amu * amu))
    s = alpha / np.sqrt(np.log(2.0))                 # sigma_G sqrt(2)
    gref = lines.gamma_ref.astype(np.float64)[pos]
    nexp = lines.n_exp.astype(np.float64)[pos]
    y = gref * (296.0 / cond.T) ** nexp * cond.P / s
    total = 2.0 * cond.cutoff * len(nu)

    def inside(rho):
        X = np.sqrt(np.maximum(rho - y * y, 0.0))
        return float(np.sum(2.0 * np.minimum(X * s, cond.cutoff))) / total

    out = {}
    for kind in FLOP_REGIONS:
        regs = FLOP_REGIONS[kind]
        fr = []
        for j, (rho, _) in enumerate(regs):
            outer = inside(regs[j - 1][0]) if j > 0 else 1.0
            inner = inside(rho) if rho > 0.0 else 0.0
            fr.append(max(outer - inner, 0.0))
        out[kind] = fr
    return out


def adj_block_share(wl, lines, cond, y2max):
    """Share of the adjoint's waves (64 neighbouring lines in wavenumber order)
    whose lines all have y^2 <= y2max, i.e. that take the block-summed form of
    a region whose rho bound is 2 y2max.  Every line has the same window, so
    it also approximates the share of that region's evaluations."""
    import numpy as np
    c, kb, amu = 2.99792458e10, 1.380649e-16, 1.66053906660e-24
    E = wl.states.energy
    nu = E[lines.upper] - E[lines.lower]
    pos = nu > 0
    order = np.argsort(nu[pos], kind="stable")
    nu = nu[pos][order]
    s = nu / c * np.sqrt(2.0 * kb * cond.T / (wl.mass_amu * amu))
    y = (lines.gamma_ref.astype(np.float64)[pos][order] * (296.0 / cond.T)
         ** lines.n_exp.astype(np.float64)[pos][order] * cond.P / s)
    n = len(y)
    pad = np.zeros((-n) % 64)
    wmax = np.concatenate([y * y, pad]).reshape(-1, 64).max(axis=1)
    return float(np.mean(wmax <= y2max))


def adj_block_shares(wl, lines, cond, prec="f32"):
    """adj_block_share for each adjoint region with a block-summed form."""
    regs = FLOP_REGIONS[("adj", prec)]
    return [adj_block_share(wl, lines, cond, 0.5 * regs[j][0]) for j in range(len(ADJ_POINT_FLOPS[prec]))]


def flops_per_eval(fracs, kind, block_shares=None):
    """Flops per evaluation averaged over the regions; for the adjoint the
    regions with a block-summed form weight it and the per-point form by the
    share of waves taking each (all block-summed when no shares are given)."""
    fl = [f for _, f in FLOP_REGIONS[kind]]
    if kind[0] == "adj" and block_shares is not None:
        for j, (sh, pt) in enumerate(zip(block_shares, ADJ_POINT_FLOPS[kind[1]])):
            fl[j] = sh * fl[j] + (1.0 - sh) * pt
    return sum(f * x for f, x in zip(fracs[kind], fl))


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def source_hash() -> str:
    h = hashlib.sha256()
    for p in KERNEL_SOURCES:
        with open(os.path.join(ROOT, p), "rb") as f:
            h.update(f.read())
    return h.hexdigest()[:16]


def traffic_from_profiles(kernel_key: str):
    """HBM bytes per launch from the committed rocprofv3 --pmc summary, if it
    was taken on the current kernel sources (else None)."""
    path = os.path.join(ROOT, "profiles", "pmc_traffic.json")
    if not os.path.exists(path):
        return None
    with open(path) as f:
        d = json.load(f)
    e = d.get(kernel_key)
    if not e or e.get("source_hash") != source_hash():
        return None
    return e.get("hbm_bytes_per_launch")


def valu_from_profiles(kernel_key: str, ms: float, sclk_mhz=None):
    """VALU issue of a kernel from the committed rocprofv3 SQ counters, if
    they were taken on the current kernel sources (else None): wave64 VALU
    instructions per launch, lane instructions per evaluation, and their
    share of the peak issue rate over the measured launch time: one wave64
    VALU instruction per 16-lane SIMD per 4 cycles at 2.4 GHz, the clock of
    the 78.6 TFLOP/s peak (transcendentals counted as one instruction).  A
    share near 1 means the kernel keeps the VALU saturated.  The share of
    all VALU instructions can exceed 1 (the FP32 adjoint read 1.00-1.05 point by point):
    transcendentals (reciprocals, exponentials) issue to a unit of their own
    and overlap the others, so issue_frac_excl_transcendental, the share of
    the rest, is reported too and stays at or below about 1.  The shader
    clock sampled from sysfs during the timed steps (the DPM level) is
    reported beside it, not used."""
    path = os.path.join(ROOT, "profiles", "pmc_valu.json")
    if not os.path.exists(path):
        return None
    with open(path) as f:
        d = json.load(f)
    e = d.get(kernel_key)
    if not e or e.get("source_hash") != source_hash():
        return None
    n = e["SQ_INSTS_VALU"]
    cycles = 256 * 4 * 2.4e9 * (ms / 1e3)
    return {"wave_instructions": n, "per_eval": round(n * 64 / e["evals"], 3),
            "transcendental_per_eval": round(e["SQ_INSTS_VALU_TRANS"] * 64 / e["evals"], 3),
            "issue_frac": round(4.0 * n / cycles, 4),
            "issue_frac_excl_transcendental": round(4.0 * (n - e["SQ_INSTS_VALU_TRANS"]) / cycles, 4),
            "sclk_MHz_sampled": round(sclk_mhz, 1) if sclk_mhz else None}


def issue_roofline(kernel_key: str, ms: float, kernel: str):
    """ALU roofline of a kernel whose per-evaluation formula has no flop
    count in the convention above (bin integrals through arctangents, error
    functions): VALU lane-instructions per second from the committed SQ
    counters against the peak issue rate 256 CU x 64 lanes x 2.4 GHz (as for
    the cooling function), or None when the counters were taken on other
    sources."""
    v = valu_from_profiles(kernel_key, ms)
    if v is None:
        return None
    ach = v["wave_instructions"] * 64 / (ms / 1e3)
    return {"bound": "alu", "achieved": round(ach / 1e12, 3), "peak": round(256 * 64 * 2.4e9 / 1e12, 3),
            "unit": "T VALU lane-instructions/s", "frac": round(ach / (256 * 64 * 2.4e9), 4), "kernel": kernel,
            "avg_launch_ms": round(ms, 3), "instr_per_eval": v["per_eval"],
            "frac_excl_transcendental": v["issue_frac_excl_transcendental"]}


def run_step(plan, ds, dl, sig, w, target, ev):
    import torch
    ev[0].record()
    plan.prepare(ds, dl)
    ev[1].record()
    plan.profile(out=sig)
    ev[2].record()
    g = (2.0 * w) * (sig - target)
    ev[3].record()
    r = plan.profile_adjoint(ds, dl, g)
    ev[4].record()
    return r


def time_steps(plan, ds, dl, sig, w, target, steps, warmup):
    import torch
    evs = [[torch.cuda.Event(enable_timing=True) for _ in range(5)] for _ in range(max(steps, 1))]
    for _ in range(warmup):
        run_step(plan, ds, dl, sig, w, target, evs[0])
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for k in range(steps):
        run_step(plan, ds, dl, sig, w, target, evs[k])
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    per = {"prepare": 0.0, "forward": 0.0, "loss_grad": 0.0, "adjoint": 0.0}
    for e in evs[:steps]:
        per["prepare"] += e[0].elapsed_time(e[1]) / steps
        per["forward"] += e[1].elapsed_time(e[2]) / steps
        per["loss_grad"] += e[2].elapsed_time(e[3]) / steps
        per["adjoint"] += e[3].elapsed_time(e[4]) / steps
    # per-step device times (first to last event of each step)
    tot = sorted(e[0].elapsed_time(e[4]) for e in evs[:steps])
    dist = {"median": round(tot[len(tot) // 2], 3), "min": round(tot[0], 3), "max": round(tot[-1], 3)} if tot else {}
    return (t1 - t0) * 1e3 / max(steps, 1), per, dist


def _sysfs_dir():
    """sysfs directory of the GPU torch uses (its PCI address)."""
    import torch
    p = torch.cuda.get_device_properties(0)
    return f"/sys/bus/pci/devices/{p.pci_domain_id:04x}:{p.pci_bus_id:02x}:{p.pci_device_id:02x}.0"


def _read(path):
    try:
        with open(path) as f:
            return f.read()
    except OSError:
        return None


def device_state():
    """The GPU's current shader, memory and fabric clock levels and board
    power, read in this process from its sysfs files (a process that uses the
    GPU starts no child process).  Best effort: missing files are left out."""
    import glob
    out = {}
    try:
        base = _sysfs_dir()
        out["pci"] = os.path.basename(base)
        for name in ("pp_dpm_sclk", "pp_dpm_mclk", "pp_dpm_fclk"):
            txt = _read(os.path.join(base, name))
            if txt:
                cur = [ln.strip() for ln in txt.splitlines() if ln.strip().endswith("*")]
                out[name] = cur[0] if cur else txt.strip()[:80]
        for hw in sorted(glob.glob(os.path.join(base, "hwmon", "hwmon*"))):
            for name in ("power1_average", "power1_input"):
                txt = _read(os.path.join(hw, name))
                if txt and txt.strip().lstrip("-").isdigit():
                    out[name + "_W"] = int(txt) / 1e6
    except Exception as e:  # noqa: BLE001 - reporting only
        out["error"] = str(e)[:200]
    return out


class PowerSampler:
    """Samples the board power and shader clock from sysfs in a thread of
    this process while timed GPU work runs (every ``period`` seconds)."""

    def __init__(self, period=0.05):
        import threading
        self.period, self.samples, self.clk = period, [], []
        self._stop = threading.Event()
        self._t = threading.Thread(target=self._run, daemon=True)
        try:
            self.base = _sysfs_dir()
        except Exception:  # noqa: BLE001
            self.base = None

    def _run(self):
        import glob
        files = []
        if self.base:
            for hw in sorted(glob.glob(os.path.join(self.base, "hwmon", "hwmon*"))):
                for name in ("power1_average", "power1_input"):
                    if os.path.exists(os.path.join(hw, name)):
                        files.append(os.path.join(hw, name))
        while not self._stop.is_set():
            for f in files[:1]:
                txt = _read(f)
                if txt and txt.strip().isdigit():
                    self.samples.append(int(txt) / 1e6)
            if self.base:
                txt = _read(os.path.join(self.base, "pp_dpm_sclk"))
                if txt:
                    cur = [ln for ln in txt.splitlines() if ln.strip().endswith("*")]
                    if cur:
                        try:
                            self.clk.append(float(cur[0].split(":")[1].strip().rstrip("*").strip().lower()
                                                  .replace("mhz", "")))
                        except (IndexError, ValueError):
                            pass
            self._stop.wait(self.period)

    def __enter__(self):
        self._t.start()
        return self

    def __exit__(self, *exc):
        self._stop.set()
        self._t.join()

    def summary(self):
        out = {"samples": len(self.samples)}
        if self.samples:
            out.update(power_W_mean=round(sum(self.samples) / len(self.samples), 1),
                       power_W_max=round(max(self.samples), 1))
        if self.clk:
            out.update(sclk_MHz_mean=round(sum(self.clk) / len(self.clk), 1), sclk_MHz_min=min(self.clk))
        return out


def cpu_baseline(wl, lines, cond, n_sample=40000):
    """The oracle (FP64, OpenMP) on this host: sigma at a random sample of grid
    points of the same workload, all lines; evaluations counted exactly as
    the (line, bin) pairs inside the cut-off."""
    import numpy as np
    import oracle
    import synth
    bins = synth.sample_bins(wl.grid.n_bins, n_sample, 4242)
    Q, _ = oracle.partition(wl.states, wl.population, cond.T)
    nu, S, keep = oracle.intensities(wl.states, lines, wl.mode, wl.population, cond.T, Q)
    alpha, gamma = oracle.widths(nu, lines, wl.profile, cond.T, cond.P, wl.mass_amu)
    snu = np.sort(nu[nu > 0])
    nuk = wl.grid.nu0 + bins * wl.grid.dnu
    evals = int(np.sum(np.searchsorted(snu, nuk + cond.cutoff, side="right")
                       - np.searchsorted(snu, nuk - cond.cutoff, side="left")))
    t0 = time.perf_counter()
    oracle.sigma(nu, S, alpha, gamma, wl.profile, wl.grid, cond.cutoff, bins)
    dt = time.perf_counter() - t0
    cores = oracle.threads()
    # the per-core rate: one thread on the first 1,000 of the sampled points
    b1 = bins[:1000]
    nuk1 = wl.grid.nu0 + b1 * wl.grid.dnu
    evals1 = int(np.sum(np.searchsorted(snu, nuk1 + cond.cutoff, side="right")
                        - np.searchsorted(snu, nuk1 - cond.cutoff, side="left")))
    oracle.set_threads(1)
    t0 = time.perf_counter()
    oracle.sigma(nu, S, alpha, gamma, wl.profile, wl.grid, cond.cutoff, b1)
    dt1 = time.perf_counter() - t0
    oracle.set_threads(cores)
    return {"value": evals / dt, "unit": "profile evals/s", "cores": cores, "kind": "oracle",
            "sample": (f"sigma at {n_sample} random grid points of the 2,000,001-point grid over all "
                       f"1e7 lines ({evals:.3e} evaluations, {dt:.1f} s including the oracle's sort of "
                       f"the lines by wavenumber)"),
            "one_thread": {"value": evals1 / dt1, "unit": "profile evals/s",
                           "sample": f"the first 1000 of those points ({evals1:.3e} evaluations, {dt1:.1f} s)"}}


def pseudo_voigt(X, wl, ds, dl, n_lines, cfg, sampled_ms):
    """The Olivero and Thompson pseudo-Voigts on the same 1e7 lines and
    condition: profile pass alone, FP32 form, main-step kernel configuration."""
    import torch
    out = {"lines": n_lines}
    for kind, name in ((X.XS_PV_OLIVERO, "olivero_f32"), (X.XS_PV_THOMPSON, "thompson_f32")):
        p = X.Plan(kind, X.XS_ABSORPTION, X.XS_LTE, X.XS_FP32, wl.grid, wl.conditions, n_lines,
                   mass_amu=wl.mass_amu)
        p.set_config(**cfg)
        sig = torch.empty((1, wl.grid.n_bins), dtype=torch.float64, device="cuda")
        p.prepare(ds, dl)
        p.profile(out=sig)
        pairs = p.stats()["window_pairs"]
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(3):
            p.profile(out=sig)
        e1.record()
        torch.cuda.synchronize()
        ms = e0.elapsed_time(e1) / 3
        out[name] = {"profile_pass_ms": round(ms, 3), "evals_per_s": pairs / (ms / 1e3),
                     "over_sampled_voigt_f32": round(ms / sampled_ms, 3),
                     "roofline": issue_roofline(f"{name}_1e7", ms, f"k_gather<float,{name.split('_')[0]}>")}
        log(f"pseudo-Voigt {name}: {ms:.2f} ms")
        p.close()
        del sig
    return out


def binned_voigt(X, wl, ds, dl, n_lines, cfg, sampled_ms):
    """The binned Voigt profile (bin means, Table tab:profile) on the same 1e7
    lines and condition: the profile pass alone (after one prepare), FP32 and
    FP64 forms, in the kernel configuration of the main step, and its cost
    relative to the sampled Voigt profile pass of the main step."""
    import torch
    out = {"lines": n_lines}
    for prec, name in ((X.XS_FP32, "f32"), (X.XS_FP64, "f64")):
        p = X.Plan(X.XS_BIN_VOIGT, X.XS_ABSORPTION, X.XS_LTE, prec, wl.grid, wl.conditions, n_lines,
                   mass_amu=wl.mass_amu)
        p.set_config(**cfg)
        sig = torch.empty((1, wl.grid.n_bins), dtype=torch.float64, device="cuda")
        p.prepare(ds, dl)
        p.profile(out=sig)
        pairs = p.stats()["window_pairs"]
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        reps = 3
        e0.record()
        for _ in range(reps):
            p.profile(out=sig)
        e1.record()
        torch.cuda.synchronize()
        ms = e0.elapsed_time(e1) / reps
        out[name] = {"profile_pass_ms": round(ms, 3), "evals_per_s": pairs / (ms / 1e3), "window_pairs": pairs,
                     "roofline": issue_roofline(f"binned_voigt1e7_{name}", ms,
                                                f"profile pass ({'float' if name == 'f32' else 'double'}, BinVoigt)")}
        log(f"binned voigt {name}: {ms:.2f} ms")
        p.close()
        del sig
    out["f32_over_sampled_f32"] = round(out["f32"]["profile_pass_ms"] / sampled_ms, 3)
    out["fp32_over_fp64_speedup"] = round(out["f64"]["profile_pass_ms"] / out["f32"]["profile_pass_ms"], 3)
    return out


# Cooling-function reduction: FP64 operations per (state, temperature) term in
# k_cf_sum: the exponent product, a rounding argument reduction, a degree-11
# polynomial, ldexp, and the accumulating FMAs of Q and W.  Peak issue: 256 CU x 64
# lanes x 2.4 GHz = 39.3e12 lane-instructions/s (FP64 FMA issues at full rate on this
# chip).
CF_INSTR_PER_TERM = 18
PEAK_LANE_INSTR = 256 * 64 * 2.4e9


def cooling_function(X, wl, ds, dl, lines):
    """Cooling function W(T), Eq. (cf), of the same 1e6 states and 1e7 lines
    on the 1-5000 K grid (1 K steps), FP64."""
    import numpy as np
    import torch
    T = np.arange(1.0, 5001.0)
    p = X.Plan(X.XS_VOIGT, X.XS_EMISSION, X.XS_LTE, X.XS_FP64, wl.grid, wl.conditions, lines.n,
               mass_amu=wl.mass_amu)
    p.cooling_function(ds, dl, T)
    torch.cuda.synchronize()
    reps, ms = 3, 0.0
    for _ in range(reps):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        p.cooling_function(ds, dl, T)
        e1.record()
        torch.cuda.synchronize()
        ms += e0.elapsed_time(e1) / reps
    p.close()
    E = wl.states.energy
    nu = E[lines.upper] - E[lines.lower]
    runs = int(np.unique(lines.upper[nu > 0]).size)
    terms = wl.states.n * T.size
    ach = terms * CF_INSTR_PER_TERM / (ms / 1e3)
    log(f"cooling function: {ms:.2f} ms, {terms:.3e} terms")
    return {"temperatures": int(T.size), "lines": lines.n, "states": wl.states.n, "upper_state_runs": runs,
            "ms": round(ms, 3), "terms": terms, "terms_per_s": terms / (ms / 1e3),
            "line_temperature_pairs_per_s": lines.n * T.size / (ms / 1e3),
            "roofline": {"bound": "alu", "achieved": round(ach / 1e12, 3), "peak": round(PEAK_LANE_INSTR / 1e12, 3),
                         "unit": "T VALU lane-instructions/s", "frac": round(ach / PEAK_LANE_INSTR, 4),
                         "instr_per_term": CF_INSTR_PER_TERM}}


def lifetime_voigt(X, wl, ds_plain, dl, n_lines, cfg, sampled_ms):
    """The Voigt profile pass of the same 1e7 lines with predissociation
    widths on a third of the states (lifetimes 10^U(-13,-10) s), FP32."""
    import torch
    import synth
    synth.with_lifetimes(wl, frac=0.33, seed=5)
    ds = X.DeviceStates.from_numpy(wl.states)
    wl.states.lifetime = None
    p = X.Plan(X.XS_VOIGT, X.XS_ABSORPTION, X.XS_LTE, X.XS_FP32, wl.grid, wl.conditions, n_lines,
               mass_amu=wl.mass_amu)
    p.set_config(**cfg)
    sig = torch.empty((1, wl.grid.n_bins), dtype=torch.float64, device="cuda")
    p.prepare(ds, dl)
    p.profile(out=sig)
    pairs = p.stats()["window_pairs"]
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(3):
        p.profile(out=sig)
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / 3
    p.close()
    log(f"lifetime Voigt f32: {ms:.2f} ms")
    return {"lines": n_lines, "states_with_lifetimes": 0.33, "profile_pass_ms": round(ms, 3),
            "evals_per_s": pairs / (ms / 1e3), "over_no_lifetimes": round(ms / sampled_ms, 3)}


def copy_bandwidth():
    """HBM bandwidth a plain device copy reaches on this GPU: a 1 GiB copy
    (1 GiB read + 1 GiB written) timed with events, best of 5."""
    import torch
    a = torch.ones(1 << 28, dtype=torch.float32, device="cuda")
    b = torch.empty_like(a)
    b.copy_(a)
    best = 1e30
    for _ in range(5):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        b.copy_(a)
        e1.record()
        torch.cuda.synchronize()
        best = min(best, e0.elapsed_time(e1))
    del a, b
    torch.cuda.empty_cache()
    return {"GB_per_s": round(2 * (1 << 30) / (best / 1e3) / 1e9, 1), "bytes_moved": 2 * (1 << 30),
            "ms": round(best, 4)}


def hbm_roofline(bytes_per_line, n_lines, ms, copy_gbs):
    ach = bytes_per_line * n_lines / (ms / 1e3) / 1e9
    return {"bound": "hbm", "bytes_per_line": bytes_per_line, "achieved": round(ach, 1), "peak": 8000.0,
            "unit": "GB/s", "frac": round(ach / 8000.0, 4), "measured_copy_GB_per_s": copy_gbs,
            "frac_of_copy": round(ach / copy_gbs, 4) if copy_gbs else None}


def alu_roofline(fpe, pairs, ms, prec, kernel, **extra):
    ach = fpe * pairs / (ms / 1e3) / 1e12
    out = {"bound": "alu", "achieved": round(ach, 3), "peak": PEAK_TFLOPS[prec], "unit": "TFLOP/s",
           "frac": round(ach / PEAK_TFLOPS[prec], 4), "kernel": kernel, "avg_launch_ms": round(ms, 3),
           "flops_per_eval": round(fpe, 3), "evals_per_launch": pairs, "note": EXPANSION_NOTE}
    out.update(extra)
    return out


def timed_replays(p, reps, warm=1):
    """Per-replay device times (ms) of the plan's captured graph, on its stream."""
    import torch
    for _ in range(warm):
        p.replay()
    torch.cuda.synchronize()
    ms = []
    for _ in range(reps):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        p.replay()
        e1.record()
        torch.cuda.synchronize()
        ms.append(e0.elapsed_time(e1))
    return ms


def _spread(ms):
    m = sorted(ms)
    return {"median": round(m[len(m) // 2], 2), "min": round(m[0], 2), "max": round(m[-1], 2), "n": len(m)}


def batched_48_full(X, copy_gbs, reps=3, tune_every=50):
    """The 48-condition opacity grid at its full size: the 1e8-line list of
    the benchmark's generator, T in 8 values x P in 6 values (cut-off 100
    cm^-1 at P >= 10 bar), grid 0-20000 cm^-1 step 0.01, all 48 conditions
    in one captured graph (intensities for the 8 distinct temperatures,
    bucketing, one persistent profile launch).  The kernel configuration is
    autotuned on every ``tune_every``-th line of the list (the full list
    would take minutes per candidate set) and then used for the full list;
    one warm-up and ``reps`` timed replays per form, FP32 and FP64."""
    import numpy as np
    import torch
    import synth
    wl = synth.workload("voigt_grid48_1e8")
    t0 = time.perf_counter()
    ln = wl.lines()
    log(f"batched 48: generated {ln.n} lines in {time.perf_counter() - t0:.1f} s")
    ds = X.DeviceStates.from_numpy(wl.states)
    dl = X.DeviceLines.from_numpy(ln)
    sub = ln.take(np.arange(0, ln.n, tune_every))
    dsub = X.DeviceLines.from_numpy(sub)
    # Voigt region split of the evaluations per condition, from a 1e6-line
    # sample, weighted by each condition's share of the window evaluations
    samp = ln.take(np.arange(0, ln.n, 100))
    wsum, fr = 0.0, {k: np.zeros(len(v)) for k, v in FLOP_REGIONS.items()}
    for c in wl.conditions:
        f = region_fractions(wl, samp, c)
        for k in fr:
            fr[k] += c.cutoff * np.asarray(f[k])
        wsum += c.cutoff
    fracs = {k: list(v / wsum) for k, v in fr.items()}
    del ln, samp
    out = {"lines": wl.n_lines, "conditions": len(wl.conditions), "reps": reps,
           "autotune_sample_lines": sub.n}
    cfg = None
    for prec, name in ((X.XS_FP32, "f32"), (X.XS_FP64, "f64")):
        p = X.Plan(X.XS_VOIGT, X.XS_ABSORPTION, X.XS_LTE, prec, wl.grid, wl.conditions, wl.n_lines,
                   mass_amu=wl.mass_amu)
        sig = torch.empty((len(wl.conditions), wl.grid.n_bins), dtype=torch.float64, device="cuda")
        if cfg is None:
            t0 = time.perf_counter()
            cfg = p.autotune(ds, dsub, sig, cache_path=os.path.join("/tmp", "xsec_autotune_48.json"))
            out["kernel_config"] = cfg
            out["autotune_s"] = round(time.perf_counter() - t0, 1)
            log(f"batched 48: autotuned {cfg} in {out['autotune_s']} s")
        else:
            p.set_config(**cfg)
        p.capture(ds, dl, sig)
        with PowerSampler(period=0.2) as pw:
            ms = timed_replays(p, reps)
        pairs = p.stats()["window_pairs"]
        med = sorted(ms)[len(ms) // 2]
        fpe = flops_per_eval(fracs, ("fwd", name))
        out[name] = {"ms": _spread(ms), "window_pairs": pairs, "evals_per_s": pairs / (med / 1e3),
                     "line_conditions_per_s": wl.n_lines * len(wl.conditions) / (med / 1e3),
                     "power": pw.summary(),
                     "roofline": alu_roofline(fpe, pairs, med, name, "graph: prepare + " + FWD_KERNELS % name,
                                              note="whole graph time (prepare of the 8 intensity slots included)",
                                              region_fractions=[round(x, 5) for x in fracs[("fwd", name)]])}
        log(f"batched 48 {name}: {_spread(ms)} ms, {pairs:.3e} pairs")
        p.close()
        del sig
    out["fp32_over_fp64_speedup"] = round(out["f64"]["ms"]["median"] / out["f32"]["ms"]["median"], 3)
    del dl, ds, dsub
    torch.cuda.empty_cache()
    return out


# Algorithmic HBM bytes per line of the prepare step (intensities,
# bucketing, records) of the two-temperature emission workload, FP32 form:
# reads u, l, A (12) + key written (4) + two radix passes, keys and values
# read and written (2 x 16) + sorted records written (nu 8, gamma_ref 4,
# n_exp 4, index 4, home bin 4, offset 4, window 8) + S~ of the 4
# intensity slots (16) = 100 B.  FP64 form: S of the 4 slots in FP64 (32):
# 116 B.
PREP_BYTES_2T = {"f32": 100, "f64": 116}


def stream_2t_full(X, copy_gbs, gen_threads=16):
    """The two-temperature emission workload at its full size: 1e9 lines in
    10 chunks of 1e8 (generated into host memory first, chunks in parallel
    threads), 4 (T_vib, T_rot) pairs, Doppler at T_rot, grid 0-30000 cm^-1
    step 0.05, streamed from host memory (uploads on a copy stream while the
    previous chunk runs), FP32 and FP64.  Also one 1e8-line chunk resident on
    the device: prepare and profile pass timed apart (the prepare's HBM
    roofline), and the same chunk with custom vibronic densities and with the
    binned Doppler profile."""
    import torch
    from concurrent.futures import ThreadPoolExecutor
    import synth
    wl = synth.workload("twotemp_1e9")
    sizes = wl.chunk_sizes()
    t0 = time.perf_counter()
    with ThreadPoolExecutor(max_workers=max(1, min(gen_threads, wl.n_chunks))) as ex:
        chunks = list(ex.map(wl.chunk, range(wl.n_chunks)))
    log(f"stream 1e9: {wl.n_chunks} chunks generated in {time.perf_counter() - t0:.1f} s")
    ds = X.DeviceStates.from_numpy(wl.states)
    out = {"lines": sum(sizes), "chunks": wl.n_chunks, "conditions": len(wl.conditions)}
    sig = torch.zeros((len(wl.conditions), wl.grid.n_bins), dtype=torch.float64, device="cuda")
    for prec, name in ((X.XS_FP32, "f32"), (X.XS_FP64, "f64")):
        plan = X.Plan(wl.profile, wl.mode, wl.population, prec, wl.grid, wl.conditions, max(sizes),
                      mass_amu=wl.mass_amu)
        st = X.ChunkStreamer(plan, max(sizes))
        st.run(ds, chunks[:1], sig)
        torch.cuda.synchronize()
        with PowerSampler(period=0.05) as pw:
            t0 = time.perf_counter()
            n = st.run(ds, chunks, sig)
            torch.cuda.synchronize()
            ms = (time.perf_counter() - t0) * 1e3
        out[f"streamed_{name}"] = {"ms": round(ms, 1), "line_conditions_per_s": n * len(wl.conditions) / (ms / 1e3),
                                   "upload_GB": round(n * 12 / 1e9, 2), "power": pw.summary()}
        log(f"stream 1e9 {name}: {ms:.0f} ms")
        st.close()
        del st
        # one chunk resident: prepare and profile pass apart
        dl = X.DeviceLines.from_numpy(chunks[0])
        plan.prepare(ds, dl)
        plan.profile(out=sig)
        torch.cuda.synchronize()
        pairs = plan.stats()["window_pairs"]
        tp, tf = [], []
        for _ in range(3):
            ev = [torch.cuda.Event(enable_timing=True) for _ in range(3)]
            ev[0].record()
            plan.prepare(ds, dl)
            ev[1].record()
            plan.profile(out=sig)
            ev[2].record()
            torch.cuda.synchronize()
            tp.append(ev[0].elapsed_time(ev[1]))
            tf.append(ev[1].elapsed_time(ev[2]))
        mp, mf = sorted(tp)[1], sorted(tf)[1]
        out[f"resident_chunk_{name}"] = {"lines": dl.n, "prepare_ms": round(mp, 3), "profile_ms": round(mf, 3),
                                         "window_pairs": pairs, "profile_evals_per_s": pairs / (mf / 1e3),
                                         "prepare_hbm": hbm_roofline(PREP_BYTES_2T[name], dl.n, mp, copy_gbs)}
        log(f"stream 1e9 {name}: resident 1e8 chunk prepare {mp:.2f} ms, profile {mf:.2f} ms")
        plan.close()
        del dl
    out["fp32_over_fp64_speedup_streamed"] = round(out["streamed_f64"]["ms"] / out["streamed_f32"]["ms"], 3)
    # the same 1e8-line chunk with custom vibronic densities, and with the
    # binned Doppler profile (resident; prepare + profile)
    dl = X.DeviceLines.from_numpy(chunks[0])
    del chunks
    variants = {}
    wd = synth.with_vib_densities(synth.workload("twotemp_1e9"))
    dsd = X.DeviceStates.from_numpy(wd.states)
    for key, w_, dss, prof, prec in (("density_f32", wd, dsd, wl.profile, X.XS_FP32),
                                     ("binned_doppler_f32", wl, ds, synth.BIN_DOPPLER, X.XS_FP32),
                                     ("binned_doppler_f64", wl, ds, synth.BIN_DOPPLER, X.XS_FP64)):
        plan = X.Plan(prof, w_.mode, w_.population, prec, w_.grid, w_.conditions, dl.n, mass_amu=w_.mass_amu)
        plan.cross_section(dss, dl, out=sig)
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        plan.cross_section(dss, dl, out=sig)
        e1.record()
        torch.cuda.synchronize()
        ms = e0.elapsed_time(e1)
        variants[key] = {"ms": round(ms, 3), "line_conditions_per_s": dl.n * len(w_.conditions) / (ms / 1e3)}
        log(f"1e8 chunk {key}: {ms:.2f} ms")
        plan.close()
    out["resident_chunk_variants"] = variants
    del dl, ds, dsd, sig
    torch.cuda.empty_cache()
    return out

def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-extras", action="store_true",
                    help="skip the FP64 step, scatter, binned, pseudo-Voigt, lifetime and cooling-function extras")
    ap.add_argument("--no-full", action="store_true",
                    help="skip the 48-condition grid at 1e8 lines and the 1e9-line two-temperature stream")
    ap.add_argument("--full-only", choices=["grid48", "twotemp"], default=None,
                    help="run only the 48-condition grid at 1e8 lines (grid48) or the 1e9-line stream (twotemp) and "
                         "print its JSON (for profiler runs)")
    ap.add_argument("--n-lines", type=int, default=None, help="(testing) fewer lines")
    ap.add_argument("--calib-copy", action="store_true", help="run only a 1 GiB device copy (PMC calibration)")
    args = ap.parse_args()
    world = int(os.environ.get("WORLD_SIZE", "1"))
    if args.gpus != 1 or world != 1:
        print("bench.py runs on one GPU only: the library has no multi-GPU path "
              "(sharding is described in the design notes); run with --gpus 1.", file=sys.stderr)
        sys.exit(2)

    if not args.no_cpu_baseline and not args.calib_copy and not args.full_only:
        # the cpu_baseline leg's oracle is compiled (if stale) now, before
        # this process touches the GPU: afterwards it starts no child process
        import oracle
        oracle.build()

    import torch

    torch.cuda.set_device(0)
    if args.calib_copy:
        a = torch.ones(1 << 28, dtype=torch.float32, device="cuda")
        b = torch.empty_like(a)
        for _ in range(5):
            b.copy_(a)
        torch.cuda.synchronize()
        log("copied 1 GiB x 5")
        return

    import synth
    import paper_2609_17273_amd as X

    copy = copy_bandwidth()
    log(f"device copy: {copy['GB_per_s']} GB/s")
    if args.full_only:
        leg = batched_48_full if args.full_only == "grid48" else stream_2t_full
        print(json.dumps({args.full_only: leg(X, copy["GB_per_s"]), "device_copy": copy}), flush=True)
        return
    t_gen = time.perf_counter()
    wl = synth.workload("voigt_1e7", n_lines=args.n_lines)
    lines = wl.lines()
    cond = wl.conditions[0]
    log(f"generated {lines.n} lines, {wl.states.n} states in {time.perf_counter() - t_gen:.1f} s")
    ds = X.DeviceStates.from_numpy(wl.states)
    dl = X.DeviceLines.from_numpy(lines)
    w = torch.as_tensor(wl.bin_weights(), device="cuda")
    sig = torch.empty((1, wl.grid.n_bins), dtype=torch.float64, device="cuda")

    def plan_for(prec, algo=X.XS_GATHER, conds=None):
        return X.Plan(X.XS_VOIGT, X.XS_ABSORPTION, X.XS_LTE, prec, wl.grid,
                      conds or wl.conditions, lines.n, mass_amu=wl.mass_amu, algo=algo)

    # target spectrum at 1700 K, 0.8 bar (FP64 form), before timing
    tp = plan_for(X.XS_FP64, conds=[synth.Condition(1700.0, 0.8, 25.0)])
    target = tp.cross_section(ds, dl)[0].clone().reshape(1, -1)
    tp.close()
    del tp

    p32 = plan_for(X.XS_FP32)
    cfg = p32.autotune(ds, dl, sig, cache_path=os.path.join("/tmp", "xsec_autotune.json"))
    log(f"autotuned: {cfg}")
    with PowerSampler() as ps32:
        ms32, per32, dist32 = time_steps(p32, ds, dl, sig, w, target, args.steps, args.warmup)
    dev_state = device_state()
    dev_state["during_timed_steps"] = ps32.summary()
    st = p32.stats()
    pairs = st["window_pairs"]
    log(f"fp32 step {ms32:.2f} ms {per32} pairs {pairs:.3e}")

    fracs = region_fractions(wl, lines, cond)
    shares = {prec: adj_block_shares(wl, lines, cond, prec) for prec in ("f32", "f64")}
    rl = {}
    for kind, ms in (("fwd", per32["forward"]), ("adj", per32["adjoint"])):
        fpe = flops_per_eval(fracs, (kind, "f32"), shares["f32"])
        key = "gather_voigt1e7_f32" if kind == "fwd" else "adjoint_voigt1e7_f32"
        extra = {"traffic": traffic_from_profiles(key),
                 "valu": valu_from_profiles(key, ms, ps32.summary().get("sclk_MHz_mean")),
                 "region_fractions": [round(f, 5) for f in fracs[(kind, "f32")]],
                 "peak_note": "78.6 TFLOP/s: FP32 FMA without packed math (256 CU x 4 SIMD x 16 lanes x 2 x "
                              "2.4 GHz), the rate this code can issue; the published 157.3 needs packed FP32"}
        if kind == "adj":
            extra["block_summed_wave_share"] = [round(x, 4) for x in shares["f32"]]
        rl[kind] = alu_roofline(fpe, pairs, ms, "f32",
                                (FWD_KERNELS if kind == "fwd" else ADJ_KERNELS) % "float", **extra)
        rl[kind]["frac_of_published_157"] = round(rl[kind]["achieved"] / 157.3, 4)
    dom = "adj" if per32["adjoint"] >= per32["forward"] else "fwd"
    other = "fwd" if dom == "adj" else "adj"

    extras = {}
    if not args.no_extras:
        p64 = plan_for(X.XS_FP64)
        cfg64 = p64.autotune(ds, dl, sig, cache_path=os.path.join("/tmp", "xsec_autotune.json"))
        log(f"autotuned fp64: {cfg64}")
        with PowerSampler() as ps64:
            ms64, per64, dist64 = time_steps(p64, ds, dl, sig, w, target, max(3, args.steps // 2), 2)
        log(f"fp64 step {ms64:.2f} ms {per64}")
        rl64 = {}
        for kind, ms in (("fwd", per64["forward"]), ("adj", per64["adjoint"])):
            fpe = flops_per_eval(fracs, (kind, "f64"), shares["f64"])
            key = "gather_voigt1e7_f64" if kind == "fwd" else "adjoint_voigt1e7_f64"
            rl64[kind] = alu_roofline(fpe, pairs, ms, "f64",
                                      (FWD_KERNELS if kind == "fwd" else ADJ_KERNELS) % "double",
                                      traffic=traffic_from_profiles(key),
                                      valu=valu_from_profiles(key, ms, ps64.summary().get("sclk_MHz_mean")),
                                      region_fractions=[round(f, 5) for f in fracs[(kind, "f64")]])
        extras["fp64"] = {"ms_per_step": round(ms64, 3), "kernel_config": cfg64,
                          "stage_ms": {k: round(v, 3) for k, v in per64.items()},
                          "step_ms_device": dist64, "evals_per_s": 2 * pairs / (ms64 / 1e3),
                          "roofline_gather": rl64["fwd"], "roofline_adjoint": rl64["adj"],
                          "prepare_hbm": hbm_roofline(100, lines.n, per64["prepare"], copy["GB_per_s"])}
        extras["fp32_over_fp64_speedup"] = {"step": round(ms64 / ms32, 3),
                                            "profile_pass": round(per64["forward"] / per32["forward"], 3),
                                            "adjoint": round(per64["adjoint"] / per32["adjoint"], 3)}
        p64.close()
        for prec, name in ((X.XS_FP32, "f32"), (X.XS_FP64, "f64")):
            ps = plan_for(prec, algo=X.XS_SCATTER)
            ps.prepare(ds, dl)
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            ps.profile(out=sig)
            e0.record()
            ps.profile(out=sig)
            e1.record()
            torch.cuda.synchronize()
            ms = e0.elapsed_time(e1)
            extras[f"scatter_{name}"] = {"profile_pass_ms": round(ms, 3), "evals_per_s": pairs / (ms / 1e3)}
            log(f"scatter {name}: {ms:.2f} ms")
            ps.close()
        extras["gather_over_scatter_speedup_f32"] = round(extras["scatter_f32"]["profile_pass_ms"] / per32["forward"], 2)
        extras["binned_voigt"] = binned_voigt(X, wl, ds, dl, lines.n, cfg, per32["forward"])
        extras["pseudo_voigt"] = pseudo_voigt(X, wl, ds, dl, lines.n, cfg, per32["forward"])
        extras["lifetime_voigt"] = lifetime_voigt(X, wl, ds, dl, lines.n, cfg, per32["forward"])
        extras["cooling_function"] = cooling_function(X, wl, ds, dl, lines)
    p32.close()
    del ds, dl, w, sig, target
    torch.cuda.empty_cache()
    if not args.no_full:
        extras["batched_48_full"] = batched_48_full(X, copy["GB_per_s"])
        extras["stream_2t_full"] = stream_2t_full(X, copy["GB_per_s"])

    evals_step = 2 * pairs
    value = evals_step / (ms32 / 1e3)
    out = {
        "metric": "profile evals/s & lines/s for sigma(nu) at 1e7 lines; batched FP32 vs FP64; adj/fwd",
        "value": value,
        "unit": "profile evals/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms32, 3),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic (seeded generator of the 1e7-line Voigt workload; no dataset)",
        "config": {"workload": "LTE Voigt absorption, 1e6 states, 1e7 lines, T 2000 K, P 1 bar, "
                               "grid 0-20000 cm^-1 step 0.01 (2,000,001 points), cut-off 25 cm^-1; step = "
                               "prepare + sigma + dL/dsigma + adjoint, FP32 log-scaled form",
                   "lines": lines.n, "states": wl.states.n, "grid_points": wl.grid.n_bins,
                   "lines_kept": st["lines_kept"], "window_pairs": pairs, "kernel_config": cfg},
        "stage_ms": {k: round(v, 3) for k, v in per32.items()},
        "step_ms_device": dist32,
        "device_state": dev_state,
        "device_copy": copy,
        "forward_evals_per_s": pairs / (per32["forward"] / 1e3),
        "lines_per_s": lines.n / (ms32 / 1e3),
        "adj_over_fwd": round(per32["adjoint"] / per32["forward"], 3),
        # intensity pass and bucketing (HBM-bound): algorithmic bytes per line =
        # reads u, l, A, gamma_ref, n_exp (20) + key write (4) + two radix
        # passes (2 x 16) + sorted records written (nu 8, gamma_ref 4, n_exp 4,
        # index 4, home bin 4, offset 4, window 8, S~ 4 = 40) = 96 B; the
        # FP64 form writes S in 8 bytes: 100 B
        "prepare_hbm": hbm_roofline(96, lines.n, per32["prepare"], copy["GB_per_s"]),
        "roofline": rl[dom],
        "roofline_other": rl[other],
        **extras,
    }
    if not args.no_cpu_baseline:
        t = time.perf_counter()
        out["cpu_baseline"] = cpu_baseline(wl, lines, cond)
        log(f"cpu baseline {out['cpu_baseline']['value']:.3e} evals/s in {time.perf_counter() - t:.1f} s")
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
