"""What the tuning cache (CIS_TUNE_CACHE) keeps (GPU): choices that were timed without a
schedule bit that narrows them, one entry per terrain of a topology.
"""
import json

import numpy as np
import pytest

from paper_2604_09993_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _traj(api, model, N=12, K=4, seed=710):
    d = synth.gen_nodes(model, N, np.random.default_rng(seed), T=0.02 * N)
    return dict(cm=api.CisModel(model), K=K, X=api.to_device_soa(d["X"]),
                U=api.to_device_soa(d["U"]), s=torch.tensor(d["s"], device="cuda"),
                params=torch.tensor(d["p"], device="cuda"))


def _groups(api, trajs, ops, **kw):
    plan = api.BatchPlan(trajs, ops, sched="tune", graph=False, **kw)
    g = plan.groups()
    plan.close()
    return g


def _entries(path):
    return json.loads(path.read_text())["entries"] if path.exists() else {}


@pytest.mark.parametrize("kind,ops,forced", [
    ("legs", ("discretize",), dict(form="split")),
    ("legs", ("discretize",), dict(form="fused", waves_per_simd=1)),
    ("legs", ("adjoint",), {}),                      # the packed sweep: nothing to time
    ("point", ("adjoint",), dict(adjoint_waves=1, defects_waves=2)),
])
def test_forced_choices_are_not_recorded(tmp_path, monkeypatch, kind, ops, forced):
    from paper_2604_09993_amd import api
    print(f"[gpu] tune cache forced {kind} {ops} {forced}", flush=True)
    path = tmp_path / "tune.json"
    monkeypatch.setenv("CIS_TUNE_CACHE", str(path))
    rng = np.random.default_rng(711)
    model = (synth.legged_model("t22", 2, 2, rng) if kind == "legs"
             else synth.make_point_contact(rng))
    trajs = [_traj(api, model)]
    g = _groups(api, trajs, ops, **forced)
    assert g[0]["from_cache"] == 0 and not _entries(path)
    g = _groups(api, trajs, ops)     # times its candidates, where it has any
    assert g[0]["from_cache"] == 0
    assert bool(_entries(path)) == (ops == ("discretize",) or kind == "point")


def test_a_forced_part_leaves_the_rest(tmp_path, monkeypatch):
    """A forced sweep does not keep the timed defects form out, nor do later plans lose it."""
    from paper_2604_09993_amd import api
    print("[gpu] tune cache, forced part", flush=True)
    path = tmp_path / "tune.json"
    monkeypatch.setenv("CIS_TUNE_CACHE", str(path))
    trajs = [_traj(api, synth.make_point_contact(np.random.default_rng(712)))]
    _groups(api, trajs, ("adjoint",), adjoint_waves=2)
    (e,) = _entries(path).values()
    assert e.get("def_lane", -1) >= 0 and e.get("adj_waves", -1) < 0
    _groups(api, trajs, ("adjoint",))
    (f,) = _entries(path).values()
    assert f["def_lane"] == e["def_lane"] and f["adj_waves"] >= 1
    assert _groups(api, trajs, ("adjoint",))[0]["from_cache"] == 1


def test_entries_by_terrain(tmp_path, monkeypatch):
    """A flat and a sinusoidal model of one topology, in one plan and for the
    single-trajectory tuner, have an entry each."""
    from paper_2604_09993_amd import api
    print("[gpu] tune cache by terrain", flush=True)
    path = tmp_path / "tune.json"
    monkeypatch.setenv("CIS_TUNE_CACHE", str(path))
    trajs = [_traj(api, synth.legged_model("t22", 2, 2, np.random.default_rng(713),
                                           terrain=terrain)) for terrain in ("flat", "sinusoid")]
    g = _groups(api, trajs, ("discretize",))
    assert [x["from_cache"] for x in g] == [0, 0] and len(_entries(path)) == 2
    assert [x["from_cache"] for x in _groups(api, trajs, ("discretize",))] == [1, 1]
    for i, t in enumerate(trajs):
        args = (t["cm"], t["X"], t["U"], t["s"], t["params"], t["K"])
        assert not api.single_tune(*args)[1]["from_cache"]
        assert len(_entries(path)) == 3 + i
        assert api.single_tune(*args)[1]["from_cache"]
