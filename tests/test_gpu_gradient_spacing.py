"""Checkpoint spacing that a batch plan chooses (GPU): by the sizes, one spacing per model
where checkpoints of every substep would take more than 4 GiB, so that the packed sweep
runs there too; and gradients that do not depend on the spacing.
"""
import numpy as np
import pytest

from paper_2604_09993_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

KEYS = ("d", "gX", "gU", "gs", "gp")


def _rows(api, model, sizes, rng):
    cm, rows, seeds = api.CisModel(model), [], []
    for N, K in sizes:
        d = synth.gen_nodes(model, N, rng, T=0.02 * N)
        rows.append(dict(cm=cm, K=K, X=api.to_device_soa(d["X"]), U=api.to_device_soa(d["U"]),
                         s=torch.tensor(d["s"], device="cuda"),
                         params=torch.tensor(d["p"], device="cuda")))
        seeds.append(torch.tensor(rng.normal(size=(model.nx, N)), device="cuda"))
    return rows, seeds


def _run(api, rows, seeds, ckpt):
    before = torch.cuda.mem_get_info()[0]
    plan = api.BatchPlan(rows, ("adjoint",), sched="grid", ckpt_every=ckpt, graph=False)
    taken = before - torch.cuda.mem_get_info()[0]
    waves = plan.groups()[0]["adjoint_waves"]
    for o, w in zip(plan.out, seeds):
        o["seed"].copy_(w)
    plan.run("adjoint")
    torch.cuda.synchronize()
    out = [{k: o[k].clone() for k in KEYS} for o in plan.out]
    plan.close()
    return out, waves, taken


@pytest.mark.parametrize("terrain", ["flat", "sinusoid"])
def test_spacings_agree(terrain):
    """The substep starts integrated again are the ones of the defects pass."""
    from paper_2604_09993_amd import api
    print(f"[gpu] gradient spacings {terrain}", flush=True)
    rng = np.random.default_rng(720)
    model = synth.legged_model("s22", 2, 2, rng, terrain=terrain, torso="horizontal")
    rows, seeds = _rows(api, model, ((5, 16), (70, 32)), rng)
    ref = _run(api, rows, seeds, 0)[0]
    for ckpt in (1, 2, 8, 16):
        for a, b in zip(ref, _run(api, rows, seeds, ckpt)[0]):
            assert all(torch.equal(a[k], b[k]) for k in KEYS), ckpt


def test_dense_checkpoints_beyond_the_limit():
    """Unequal substep counts (the largest divisors not above 8 are 8 and 6) with 4.3 GB
    of checkpoints: one spacing of 4 and the packed sweep."""
    from paper_2604_09993_amd import api
    print("[gpu] gradient spacing beyond 4 GiB", flush=True)
    rng = np.random.default_rng(721)
    model = synth.MODEL_MAKERS["quad13"](rng)
    rows, seeds = _rows(api, model, ((900, 4096), (800, 4092)), rng)
    got, waves, taken = _run(api, rows, seeds, 0)
    ref, want, _ = _run(api, rows, seeds, 4)
    assert waves == want == 4 and taken < 2 << 30
    for a, b in zip(got, ref):
        assert all(torch.equal(a[k], b[k]) for k in KEYS)
        assert all(torch.isfinite(a[k]).all() for k in ("gs", "gp"))
