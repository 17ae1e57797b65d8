"""Impact map solved leg by leg vs the oracle (GPU): every topology on flat ground and
on a sinusoid, and masses on either side of the ratio beyond which (and for a fixed
body of infinite mass) the joint rows are solved with 1/m instead.  Bars as everywhere
(tests/parity.py).
"""
import numpy as np
import pytest

from paper_2604_09993_amd import synth
from test_gpu_impact import check, run_gpu

pytestmark = pytest.mark.gpu
pytest.importorskip("torch")

TOPOLOGIES = [(1, 1), (1, 2), (2, 1), (2, 2), (2, 3), (4, 3)]


def _case(legs, depth, terrain, n):
    rng = np.random.default_rng([950, legs, depth])
    model = synth.legged_model(f"i{legs}{depth}", legs, depth, rng, terrain=terrain,
                               torso="horizontal")
    return model, synth.gen_impact_nodes(model, n, rng)


@pytest.mark.parametrize("terrain", ["flat", "sinusoid"])
@pytest.mark.parametrize("legs,depth", TOPOLOGIES)
def test_topologies(legs, depth, terrain):
    print(f"[gpu] impact {legs}x{depth} {terrain}", flush=True)
    model, d = _case(legs, depth, terrain, 3)
    check(model, d, run_gpu(model, d))


@pytest.mark.parametrize("mass", [1e2, 1e6, np.inf])
@pytest.mark.parametrize("body", [0, 1, -1])
def test_heavy_bodies(body, mass):
    print(f"[gpu] impact 2x2 body {body} of mass {mass}", flush=True)
    model, d = _case(2, 2, "sinusoid", 3)
    d["p"] = d["p"].copy()
    d["p"][2:][body] = mass
    res = run_gpu(model, d)
    if np.isfinite(mass):
        check(model, d, res)
    else:   # (the oracle's mass columns divide by the mass)
        assert all(np.isfinite(res[k]).all() for k in ("G", "Theta", "JGv", "JTc"))
