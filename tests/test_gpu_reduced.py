"""Reduced columns of the two-launch form (packed record launch, coupled columns,
closed-form entries) vs the oracle at the edges of their tiles (GPU).

Four intervals share a workgroup and 64 a block of closed-form stores, so the
interval counts sit around 4 and 64; a batch puts intervals of different substep
counts into one workgroup.  Flat and sinusoidal terrain take different column
sets, so every topology runs on both.  Bars as everywhere (tests/parity.py).
A non-finite input has to reach the entries that have a closed form.
"""
import numpy as np
import pytest

import oracle
from paper_2604_09993_amd import synth
from parity import PHI32, PHI64, TOL32, TOL64, compare_outputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TOPOLOGIES = [(1, 1), (1, 2), (2, 1), (2, 2), (2, 3), (4, 3)]


def _case(legs, depth, terrain, N, seed=600):
    rng = np.random.default_rng([seed, legs, depth, N])
    model = synth.legged_model(f"t{legs}{depth}", legs, depth, rng, terrain=terrain,
                               torso="horizontal")
    return model, synth.gen_nodes(model, N, rng, T=0.02 * N)


def _dev(model, d, dtype):
    from paper_2604_09993_amd import api
    return (api.CisModel(model), api.to_device_soa(d["X"], dtype=dtype),
            api.to_device_soa(d["U"], dtype=dtype),
            torch.tensor(d["s"], device="cuda", dtype=dtype),
            torch.tensor(d["p"], device="cuda", dtype=dtype))


def _check(model, d, K, out, dtype):
    from paper_2604_09993_amd import api
    got = {k: v.double().cpu().numpy() for k, v in api.as_interval_major(out).items()}
    fp32 = dtype == torch.float32
    r = [np.float32(d[k]).astype(np.float64) if fp32 else d[k] for k in ("X", "U", "s", "p")]
    ref = oracle.discretize(model, r[0], r[1], r[2], r[3], K)
    errs = compare_outputs(got, ref, phi=PHI32 if fp32 else PHI64)
    bad = {k: e for k, e in errs.items() if not e <= (TOL32 if fp32 else TOL64)}
    assert not bad, bad


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("terrain", ["flat", "sinusoid"])
@pytest.mark.parametrize("legs,depth", TOPOLOGIES)
def test_tile_edges(legs, depth, terrain, dtype):
    from paper_2604_09993_amd import api
    for N, K in ((1, 1), (3, 2), (4, 3), (5, 2), (63, 1), (64, 2), (65, 1)):
        print(f"[gpu] reduced {legs}x{depth} {terrain} {dtype} N={N} K={K}", flush=True)
        model, d = _case(legs, depth, terrain, N)
        cm, X, U, s, p = _dev(model, d, dtype)
        out = api.discretize_split(cm, X, U, s, p, K)
        torch.cuda.synchronize()
        _check(model, d, K, out, dtype)


@pytest.mark.parametrize("terrain", ["flat", "sinusoid"])
@pytest.mark.parametrize("legs,depth", [(1, 1), (2, 2), (2, 3), (4, 3)])
def test_rkf_tile_edges(legs, depth, terrain):
    """Odd and even step counts (the coefficient slots alternate over five stages)."""
    from paper_2604_09993_amd import api
    for N, K in ((1, 1), (4, 2), (5, 3), (65, 1)):
        print(f"[gpu] reduced rkf {legs}x{depth} {terrain} N={N} K={K}", flush=True)
        model, d = _case(legs, depth, terrain, N)
        cm, X, U, s, p = _dev(model, d, torch.float64)
        out = api.discretize_rkf(cm, X, U, s, p, K)
        torch.cuda.synchronize()
        got = {k: v.cpu().numpy() for k, v in api.as_interval_major(out).items()}
        ref = oracle.discretize_rkf(model, d["X"], d["U"], d["s"], d["p"], K)
        errs = compare_outputs(got, ref)
        bad = {k: e for k, e in errs.items() if not e <= TOL64}
        assert not bad, bad
        assert np.all(np.abs(got["err"] - ref["err"]) <= 1e-9 * np.abs(ref["err"]) + 1e-13)


@pytest.mark.parametrize("legs,depth,terrain", [(1, 1, "flat"), (2, 2, "sinusoid"), (4, 3, "flat")])
def test_batch_mixes_substep_counts_in_a_workgroup(legs, depth, terrain):
    from paper_2604_09993_amd import api
    print(f"[gpu] reduced batch {legs}x{depth} {terrain}", flush=True)
    cases, trajs = [], []
    rng = np.random.default_rng(610)
    model, _ = _case(legs, depth, terrain, 2)
    for N, K in ((3, 1), (2, 5), (70, 2), (1, 9)):
        d = synth.gen_nodes(model, N, rng, T=0.02 * N)
        cases.append((d, K))
    cm = None
    for d, K in cases:
        c, X, U, s, p = _dev(model, d, torch.float64)
        cm = cm or c
        trajs.append(dict(cm=cm, X=X, U=U, s=s, params=p, K=K))
    plan = api.BatchPlan(trajs, sched="grid", form="split", graph=True)
    for replay in range(2):
        for o in plan.out:
            for k in ("A", "Bm", "Bp", "S", "d", "xprop"):
                o[k].fill_(float("nan"))
        plan.run("discretize", graph=bool(replay))
        torch.cuda.synchronize()
        for (d, K), o in zip(cases, plan.out):
            _check(model, d, K, {k: o[k] for k in ("A", "Bm", "Bp", "S", "d", "xprop")},
                   torch.float64)
    plan.close()


@pytest.mark.parametrize("terrain", ["flat", "sinusoid"])
def test_non_finite_inputs_reach_the_closed_forms(terrain):
    """A NaN angle of interval 5's start node leaves no finite entry in the angle
    rows of its A, nor in the feet's translation rows (whose contact force turns
    with the angle); the other intervals stay finite.  A NaN dilation reaches
    every pose row."""
    from paper_2604_09993_amd import api
    print(f"[gpu] reduced non-finite {terrain}", flush=True)
    N, K = 9, 2
    model, d = _case(2, 2, terrain, N)
    n, nq, nx = model.n, model.n // 2, model.nx
    feet = [int(b) for b in model.contact_body]
    for what in ("angle", "dilation"):
        e = {k: v.copy() for k, v in d.items()}
        if what == "angle":
            e["X"][5, 2] = np.nan
        else:
            e["s"][5] = np.nan
        cm, X, U, s, p = _dev(model, e, torch.float64)
        out = api.as_interval_major(api.discretize_split(cm, X, U, s, p, K))
        torch.cuda.synchronize()
        A = out["A"].cpu().numpy()
        bad = ~np.isfinite(A[5])
        assert np.isfinite(np.delete(A, 5, axis=0)).all()
        assert np.all(A[5][:, n:] == np.eye(nx)[:, n:])   # structural columns
        if what == "angle":
            rows = [3 * b + 2 for b in range(model.nb)] + [3 * b for b in feet]
            rows += [nq + r for r in rows]
        else:
            rows = list(range(nq))
        assert bad[rows][:, :n].all()


@pytest.mark.parametrize("legs,depth", [(1, 1), (2, 2)])
def test_record_budget_line(legs, depth):
    """FP64 on the sinusoid: the record launch's register budget changes at six
    intervals per CU."""
    from paper_2604_09993_amd import api
    line = 6 * torch.cuda.get_device_properties(0).multi_processor_count
    for N in (line, line + 1):
        print(f"[gpu] reduced {legs}x{depth} sinusoid budget line N={N}", flush=True)
        model, d = _case(legs, depth, "sinusoid", N)
        cm, X, U, s, p = _dev(model, d, torch.float64)
        out = api.discretize_split(cm, X, U, s, p, 1)
        torch.cuda.synchronize()
        _check(model, d, 1, out, torch.float64)
