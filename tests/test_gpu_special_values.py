"""Very large and non-finite inputs (GPU): what does not depend on them stays as it is.

Arguments whose squares overflow: a root is infinite and a quotient by it zero, as in
the oracle's formulas.  A NaN reaches what has it in its formula, not what has a zero
coefficient by it for the lack of a contact, nor other intervals.
"""
import numpy as np
import pytest

from paper_2604_09993_amd import synth
from test_gpu_impact import DELTA, run_gpu
from test_gpu_paper import run_paper

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

BIG = 1e200


def _legs(terrain, legs=2, depth=2):
    rng = np.random.default_rng([970, legs, depth])
    return synth.legged_model(f"v{legs}{depth}", legs, depth, rng, terrain=terrain,
                              torso="horizontal"), rng


@pytest.mark.parametrize("terrain", ["flat", "sinusoid"])
def test_impact_arguments_whose_squares_overflow(terrain):
    """FB(a, b) = a + b - sqrt(a^2 + b^2 + delta) is -inf with slope 1 in the other
    argument; phi_t / sqrt(phi_t^2 + 1) is 0."""
    print(f"[gpu] impact overflow {terrain}", flush=True)
    model, rng = _legs(terrain)
    d = synth.gen_impact_nodes(model, 3, rng)
    tip = int(model.contact_body[0])
    plain = run_gpu(model, d)
    other = np.arange(plain["Theta"].shape[1]) >= 10
    for what in ("velocity", "normal", "tangent"):
        e = {k: v.copy() for k, v in d.items()}
        if what == "velocity":
            e["Xp"][1, 3 * model.nb + 3 * tip + 1] = BIG
            lost = [1]
        elif what == "normal":
            e["Phi"][1, 1] = BIG
            lost = [0, 1]
        else:
            e["Phi"][1, 0] = BIG
            lost = []
        r = run_gpu(model, e)
        T, J = r["Theta"][1], r["JTc"][1]
        assert np.all(T[lost] == -np.inf), (what, T[:10])
        for k in ("Theta", "JTc"):   # the other contact, the other nodes
            assert np.array_equal(r[k][1][other], plain[k][1][other])
            assert np.array_equal(r[k][::2], plain[k][::2])
        if what == "velocity":
            # row 1 by everything but Phi_n and the infinite root: w; row 7: -w
            # (2 w dw, the root's argument's derivative, is finite for dw < 1e100)
            keep = [c for c in range(14) if c != 10 and abs(J[7][c]) < 1e100]
            assert len(keep) >= 10
            assert np.array_equal(J[1][keep], -J[7][keep]) and J[1][10] == 1.0
            assert np.isfinite(np.delete(T, lost)).all()
        elif what == "tangent":
            # lam is the tangential velocity: the difference of rows 2 and 3 over 2 Phi_n
            pn = e["Phi"][1, 1]
            e["Gamma"][1, 0] = 0.0
            free = run_gpu(model, e)["Theta"][1]
            assert np.array_equal(T[2:4], free[2:4]) and np.isfinite(T[2:4]).all()
            assert abs(0.5 * (T[2] + T[3]) + DELTA) <= 1e-14 * max(1.0, abs(pn))
            assert np.isfinite(J[2:4]).all()


@pytest.mark.parametrize("terrain", ["flat", "sinusoid"])
def test_paper_friction_whose_square_overflows(terrain):
    """mu enters the friction-cone row and the violation row alone, and both stay finite
    where (mu phi_n)^2 overflows."""
    print(f"[gpu] paper overflow {terrain}", flush=True)
    model, rng = _legs(terrain)
    data = synth.gen_paper_nodes(model, 3, rng, T=0.06)
    plain = run_paper(model, data, 2)
    data["p"] = data["p"].copy()
    data["p"][0] = BIG
    res = run_paper(model, data, 2)
    n, nc = model.n, model.nc
    rows = [r for r in range(n + 4 * nc) if r < n or (r - n) % 4 != 3]
    for k in ("A", "Bm", "Bp"):
        assert np.isfinite(res[k]).all(), k
        assert np.array_equal(res[k][:, rows], plain[k][:, rows]), k


def _nan_run(kind, model, d, K, where):
    """The outputs of intervals with a NaN at `where` of X's node 2, and of plain ones."""
    from paper_2604_09993_amd import api
    cm = api.CisModel(model)
    out = []
    for value in (None, float("nan")):
        X = d["X"].copy()
        if value is not None:
            X[2, where] = value
        args = (cm, api.to_device_soa(X), api.to_device_soa(d["U"]),
                torch.tensor(d["s"], device="cuda"), torch.tensor(d["p"], device="cuda"), K)
        r = (api.discretize_split if kind == "split" else api.discretize_rkf)(*args)
        torch.cuda.synchronize()
        out.append({k: v.cpu().numpy() for k, v in api.as_interval_major(
            {k: v for k, v in r.items() if k != "err"}).items()})
    return out


@pytest.mark.parametrize("kind", ["split", "rkf"])
@pytest.mark.parametrize("terrain", ["flat", "sinusoid"])
def test_nan_torso_velocity(terrain, kind):
    """The torso's x rate enters its x row and the violation row alone."""
    print(f"[gpu] NaN torso velocity {kind} {terrain}", flush=True)
    model, rng = _legs(terrain)
    d = synth.gen_nodes(model, 6, rng, T=0.12)
    nq, n, nx = 3 * model.nb, model.n, model.nx
    plain, res = _nan_run(kind, model, d, 2, nq)
    rows = [r for r in range(nx - 1) if r not in (0, nq)]
    for k in ("A", "Bm", "Bp", "S"):
        assert np.array_equal(np.delete(res[k], 2, 0), np.delete(plain[k], 2, 0)), k
        assert np.array_equal(res[k][2][rows], plain[k][2][rows]), k


@pytest.mark.parametrize("kind", ["split", "rkf"])
def test_nan_foot_height(kind):
    """On flat ground a foot's height enters the value of its integral row, not the
    row's coefficients, and the violation row."""
    print(f"[gpu] NaN foot height {kind}", flush=True)
    model, rng = _legs("flat")
    d = synth.gen_nodes(model, 6, rng, T=0.12)
    plain, res = _nan_run(kind, model, d, 2, 3 * int(model.contact_body[0]) + 1)
    for k in ("A", "Bm", "Bp"):
        assert np.array_equal(np.delete(res[k], 2, 0), np.delete(plain[k], 2, 0)), k
    assert np.array_equal(res["A"][2][:model.nx - 1], plain["A"][2][:model.nx - 1])


@pytest.mark.parametrize("terrain", ["flat", "sinusoid"])
def test_nan_torso_position_gradient(terrain):
    """The torso's x enters the joint rows of the violation by x and y: its own y row of
    gX, which has the joints' y distances alone, stays as it is."""
    from paper_2604_09993_amd import api
    print(f"[gpu] NaN torso position, gradient {terrain}", flush=True)
    model, rng = _legs(terrain)
    d = synth.gen_nodes(model, 6, rng, T=0.12)
    cm = api.CisModel(model)
    seed = torch.tensor(rng.normal(size=(model.nx, 6)), device="cuda")
    s, p = torch.tensor(d["s"], device="cuda"), torch.tensor(d["p"], device="cuda")
    U, res = api.to_device_soa(d["U"]), []
    for value in (None, float("nan")):
        X = d["X"].copy()
        if value is not None:
            X[2, 0] = value
        Xd = api.to_device_soa(X)
        f = api.defects(cm, Xd, U, s, p, 2, ckpt_every=1)
        g = api.adjoint(cm, Xd, U, s, p, 2, f["ckpt"], 1, seed)
        torch.cuda.synchronize()
        res.append({k: v.cpu().numpy() for k, v in g.items()})
    rows = [1, 3 * model.nb + 1]
    for k in ("gX", "gs"):   # other intervals
        assert np.array_equal(np.delete(res[0][k], 2, -1), np.delete(res[1][k], 2, -1)), k
    assert np.array_equal(res[0]["gX"][rows, 2], res[1]["gX"][rows, 2])
