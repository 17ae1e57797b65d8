"""Masses at the line between the leg elimination and the joint rows' system (GPU).

A link of 16 times the lightest of the torso and the links before it takes the joint
rows' system (1/m): just below and above it, for an inner link and a tip, the impact map
and the paper-faithful dynamics against the oracle.  A fixed body (infinite mass, of
either sign: 1/m = 0) against the oracle with a mass of 1e30.  Bars as everywhere
(tests/parity.py).
"""
import numpy as np
import pytest

from paper_2604_09993_amd import synth
from parity import PHI64, TOL64, block_err
from test_gpu_impact import check as check_impact, oracle_ref, run_gpu
from test_gpu_paper import check as check_paper, run_paper

pytestmark = pytest.mark.gpu
pytest.importorskip("torch")

CASES = [(2, 2, "sinusoid"), (4, 3, "flat")]


def _model(legs, depth, terrain):
    rng = np.random.default_rng([980, legs, depth])
    return synth.legged_model(f"h{legs}{depth}", legs, depth, rng, terrain=terrain,
                              torso="horizontal"), rng


def _finite(res):   # (block_err passes over a NaN)
    assert all(np.isfinite(v).all() for v in res.values())


def _weigh(model, p, depth, body, ratio):
    """p with the mass of `body` (a link of the first leg, from 1) at the ratio."""
    p = p.copy()
    m = p[2:]
    m[body] = ratio * m[:body].min()
    return p


@pytest.mark.parametrize("ratio", [15.9, 16.1])
@pytest.mark.parametrize("tip", [False, True])
@pytest.mark.parametrize("legs,depth,terrain", CASES)
def test_ratio(legs, depth, terrain, tip, ratio):
    print(f"[gpu] heavy {legs}x{depth} {terrain} tip={tip} ratio={ratio}", flush=True)
    model, rng = _model(legs, depth, terrain)
    body = depth if tip else 1
    d = synth.gen_impact_nodes(model, 3, rng)
    d["p"] = _weigh(model, d["p"], depth, body, ratio)
    res = run_gpu(model, d)
    _finite(res)
    check_impact(model, d, res)
    data = synth.gen_paper_nodes(model, 2, rng, T=0.04)
    data["p"] = _weigh(model, data["p"], depth, body, ratio)
    res = run_paper(model, data, 2)
    _finite(res)
    check_paper(model, data, 2, res)


@pytest.mark.parametrize("sign", [1, -1])
@pytest.mark.parametrize("body", [0, 1, 2, -1])
@pytest.mark.parametrize("legs,depth,terrain", CASES)
def test_fixed_body_impact(legs, depth, terrain, body, sign):
    print(f"[gpu] fixed body {body} {legs}x{depth} {terrain} sign {sign}", flush=True)
    model, rng = _model(legs, depth, terrain)
    d = synth.gen_impact_nodes(model, 3, rng)
    d["p"] = d["p"].copy()
    d["p"][2:][body] = sign * np.inf
    res = run_gpu(model, d)
    _finite(res)
    d["p"][2:][body] = 1e30
    ref = oracle_ref(model, d, [0, 1, 2])
    errs = {k: block_err(res[k], ref[k], PHI64) for k in ref}
    assert all(e <= TOL64 for e in errs.values()), errs


@pytest.mark.parametrize("ratio", [1.0, 100.0])
@pytest.mark.parametrize("legs,depth,terrain", [(1, 2, "sinusoid"), (2, 3, "flat")])
def test_paper_record_launches(legs, depth, terrain, ratio):
    """One launch holds both forms' records up to an interval per SIMD, two beyond."""
    import torch
    line = 4 * torch.cuda.get_device_properties(0).multi_processor_count
    model, rng = _model(legs, depth, terrain)
    for N in (line, line + 1):
        print(f"[gpu] paper records {legs}x{depth} N={N} ratio={ratio}", flush=True)
        data = synth.gen_paper_nodes(model, N, rng, T=0.02 * N)
        data["p"] = _weigh(model, data["p"], depth, depth, ratio)
        res = run_paper(model, data, 1)
        _finite(res)
        check_paper(model, data, 1, res, ks=[0, 1, N // 3, N - 2, N - 1])
