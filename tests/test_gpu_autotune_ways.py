"""The autotuner's file keeps the ways of a profile pass apart: two plans of one profile,
window, line count and table whose passes go through the expansions and through the gather
have entries of their own, and the gather's is tuned whichever came first.  A line of an earlier
file, which names no way, serves the gather."""
import json

import pytest

import synth
from test_gpu_far import FP32, C, _Grid
from xs_helpers import X, gpu_inputs, workload

pytestmark = pytest.mark.gpu


def _tune(n_bins, path, profile=synth.VOIGT):
    import torch
    P = X()
    wl = workload("voigt_1e7", n_states=20000, n_lines=30011, nu_hi=600.0, seed=4242)
    ln = wl.lines()
    ds, dl = gpu_inputs(wl, ln)
    plan = P.Plan(profile, 0, 0, FP32, _Grid(0.0, 0.01, n_bins), [C(900.0, 1.0, 25.0)], ln.n, mass_amu=wl.mass_amu)
    cfg = plan.autotune(ds, dl, torch.empty((1, n_bins), dtype=torch.float64, device="cuda"), cache_path=str(path))
    plan.close()
    return cfg


def _entries(path):
    return [json.loads(q) for q in path.read_text().splitlines()]


@pytest.mark.parametrize("first, second", [(60001, 2000001), (2000001, 60001)])
def test_ways_apart(tmp_path, first, second):
    path = tmp_path / "tune.json"
    _tune(first, path)
    assert len(_entries(path)) == 1
    _tune(second, path)
    e = _entries(path)
    assert len(e) == 2 and e[0]["key"] != e[1]["key"]
    far = [q for q in e if "|far" in q["key"]]
    assert len(far) == 1  # 30011 lines: expansions on 60001 points, the gather on 2000001
    _tune(first, path)
    _tune(second, path)
    assert _entries(path) == e  # both are found again


def test_earlier_line(tmp_path):
    path = tmp_path / "tune.json"
    _tune(2000001, path)
    (q,) = _entries(path)
    assert "far" not in q["key"] and "near" not in q["key"]
    q.update(tile_bins=1024, bucket_bins=64, persistent=0, waves_per_cu=16, chunk_lines=0, adj_blocks=4096)
    path.write_text(json.dumps(q) + "\n")
    cfg = _tune(2000001, path)
    assert cfg["tile_bins"] == 1024 and cfg["bucket_bins"] == 64 and cfg["adj_blocks"] == 4096
    assert _tune(60001, path)["tile_bins"] == 256
