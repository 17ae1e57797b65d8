"""Paper-faithful dynamics solved leg by leg, four intervals per record wave, vs the
oracle at the edges of its tiles (GPU): interval counts around 4, every topology on
flat ground and on a sinusoid; and masses on either side of the ratio beyond which
the joint rows are solved with 1/m instead.  Bars as everywhere (tests/parity.py).
"""
import numpy as np
import pytest

from paper_2604_09993_amd import synth
from test_gpu_paper import check, run_paper

pytestmark = pytest.mark.gpu
pytest.importorskip("torch")

TOPOLOGIES = [(1, 1), (1, 2), (2, 1), (2, 2), (2, 3), (4, 3)]


@pytest.mark.parametrize("terrain", ["flat", "sinusoid"])
@pytest.mark.parametrize("legs,depth", TOPOLOGIES)
def test_tile_edges(legs, depth, terrain):
    for N, K in ((1, 1), (3, 2), (4, 1), (5, 2)):
        print(f"[gpu] paper {legs}x{depth} {terrain} N={N} K={K}", flush=True)
        rng = np.random.default_rng([800, legs, depth, N])
        model = synth.legged_model(f"p{legs}{depth}", legs, depth, rng, terrain=terrain,
                                   torso="horizontal")
        data = synth.gen_paper_nodes(model, N, rng, T=0.02 * N)
        check(model, data, K, run_paper(model, data, K))


@pytest.mark.parametrize("mass", [1.0, 1e2, 1e6])
@pytest.mark.parametrize("body", [0, 1, -1])
def test_heavy_bodies(body, mass):
    print(f"[gpu] paper 2x2 body {body} of mass {mass}", flush=True)
    rng = np.random.default_rng(801)
    model = synth.legged_model("p22", 2, 2, rng, terrain="sinusoid", torso="horizontal")
    data = synth.gen_paper_nodes(model, 2, rng, T=0.04)
    data["p"] = data["p"].copy()
    data["p"][2:][body] = mass
    check(model, data, 3, run_paper(model, data, 3))
