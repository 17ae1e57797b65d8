"""Performance cases of the interval linearize-and-discretize framework.

Each case is one call that a program using this framework makes in its loop: the
discretization of one trajectory (what an SCP iteration does), a batch plan over
several trajectories (one model or a mix of models), the gradient step (defects
and reverse sweep), the Fehlberg and paper-faithful transcriptions, and the
impact-map linearization.  Sizes are those of the repository's workloads
(hopper N=20 K=10, cheetah7 N=50 K=20, quad13 N=200 K=20, 12,800 quad13
intervals, 12,864 impact nodes) and generic ragged ones.

``exact`` restates the maps in plain torch, FP64: the right-hand side batched
over intervals, its dense Jacobian by forward-mode differentiation, and the
Runge-Kutta recursion of the state and of every sensitivity column.
"""
from __future__ import annotations

import numpy as np
import torch

from paper_2604_09993_amd import api, synth

DT = 0.02           # mean interval length (s): cheetah7 N = 50 over one second
TYPES = {"f64": torch.float64, "f32": torch.float32}
MIX = ("hopper", "cheetah7", "hopper", "biped5", "cheetah7", "hopper", "biped5", "hopper",
       "cheetah7", "hopper")


# --------------------------------------------------------------------------- cases
def listed():
    return [
        # the smallest call: one SCP iterate of the monoped-like hopper
        dict(name="hopper_N20_K10", kind="discretize", model="hopper", N=20, K=10, type="f64"),
        # one SCP iterate of the HalfCheetah-shaped chain
        dict(name="cheetah7_N50_K20", kind="discretize", model="cheetah7", N=50, K=20, type="f64"),
        # a long biped trajectory on the sinusoid, sizes that divide nothing
        dict(name="biped5_N333_K17", kind="discretize", model="biped5", N=333, K=17, type="f64"),
        # the quadruped-shaped chain, one trajectory in the two-launch form with a kept workspace
        dict(name="quad13_N200_K20_split", kind="split", model="quad13", N=200, K=20, type="f64"),
        # gradient of a merit through autograd (defects, checkpoints, reverse sweep)
        dict(name="cheetah7_N50_K20_grad", kind="gradient", model="cheetah7", N=50, K=20, C=5,
             type="f64"),
        # multiple shooting over ten uneven trajectories of three models, one graph replay
        dict(name="mixed10", kind="batch", model="mixed", T=10, Nlo=60, Nhi=300, K=20, type="f64"),
        # 12,800 quad13 intervals: the throughput workload, both precisions
        dict(name="quad13_12800", kind="batch", model="quad13", T=10, Nlo=1280, Nhi=1280, K=20,
             type="f64"),
        dict(name="quad13_12800_f32", kind="batch", model="quad13", T=10, Nlo=1280, Nhi=1280, K=20,
             type="f32"),
        # the gradient step of a large batch
        dict(name="quad13_12800_grad", kind="batch_grad", model="quad13", T=10, Nlo=1280, Nhi=1280,
             K=20, type="f64"),
        # Fehlberg 4(5) transcription of a large set of intervals
        dict(name="rkf_quad13_N3201_K20", kind="rkf", model="quad13", N=3201, K=20, type="f64"),
        # paper-faithful dynamics (joint forces eliminated)
        dict(name="paper_quad13_N1603_K20", kind="paper", model="quad13", N=1603, K=20, type="f64"),
        # node constraints of every node of the quad13 batch
        dict(name="impact_quad13_12864", kind="impact", model="quad13", N=12864, type="f64"),
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(lo * (hi / lo) ** rng.random()))

    kind = rng.choice(("discretize", "discretize", "split", "gradient", "batch", "batch_grad",
                       "rkf", "paper", "impact"))
    model = rng.choice(("hopper", "biped5", "cheetah7", "quad13"))
    if kind == "impact":
        return dict(kind=kind, model=model, N=size(64, 12800), type="f64")
    if kind in ("batch", "batch_grad"):
        lo = size(20, 1000)
        return dict(kind=kind, model=rng.choice((model, "mixed")), T=rng.randint(2, 10), Nlo=lo,
                    Nhi=rng.randint(lo, min(2 * lo, 1280)), K=rng.randint(8, 20),
                    type="f64" if kind == "batch_grad" else rng.choice(("f64", "f64", "f32")))
    K = rng.randint(4, 30)
    if kind == "gradient":
        C = rng.choice([c for c in range(1, 9) if K % c == 0])
        return dict(kind=kind, model=model, N=size(8, 1000), K=K, C=C, type="f64")
    top = dict(discretize=2000, split=4000, rkf=2500, paper=1000)[kind]
    return dict(kind=kind, model=model, N=size(8, top), K=K,
                type="f64" if kind == "paper" else rng.choice(("f64", "f64", "f32")))


# -------------------------------------------------------------------------- inputs
def _model(name):
    return synth.MODEL_MAKERS[name](np.random.default_rng(11))


def _poses(model, n, r):
    """Joint-closed poses [n, nb, 3], the lowest foot U(-0.02, 0.10) m above the terrain."""
    q = np.zeros((n, model.nb, 3))
    q[:, 0, 0] = r.uniform(-0.5, 0.5, n)
    q[:, 0, 2] = r.uniform(-0.2, 0.2, n)

    def at(b, a):
        c, s = np.cos(q[:, b, 2]), np.sin(q[:, b, 2])
        return np.stack([c * a[0] - s * a[1], s * a[0] + c * a[1]], axis=1)

    for j in range(model.nj):
        p, c = int(model.joint_parent[j]), int(model.joint_child[j])
        q[:, c, 2] = q[:, p, 2] + r.uniform(-0.5, 0.5, n)
        q[:, c, :2] = q[:, p, :2] + at(p, model.anchor_parent[j]) - at(c, model.anchor_child[j])
    gap = np.full(n, np.inf)
    for i in range(model.nc):
        b = int(model.contact_body[i])
        P = q[:, b, :2] + at(b, model.contact_point[i])
        gap = np.minimum(gap, P[:, 1] - model.terrain_amplitude
                         * np.sin(model.terrain_wavenumber * P[:, 0]))
    q[:, :, 1] += (r.uniform(-0.02, 0.10, n) - gap)[:, None]
    return q.reshape(n, -1)


def _nodes(model, N, r, paper=False, dt=DT):
    """Node data of one trajectory, rows first ([rows, N+1]), FP64."""
    nb, nj, nc = model.nb, model.nj, model.nc
    n, ny = 6 * nb, 4 * nc + 1 if paper else nc + 1
    X = np.zeros((N + 1, n + ny))
    X[:, :3 * nb] = _poses(model, N + 1, r)
    X[:, 3 * nb:n] = r.normal(0.0, 0.5, (N + 1, 3 * nb))
    if paper:
        U = np.zeros((N + 1, nj + 3 * nc))
        U[:, :nj] = r.normal(0.0, model.torque_sigma, (N + 1, nj))
        pn = r.uniform(0.0, 30.0, (N + 1, nc))
        U[:, nj::3] = r.uniform(-0.8, 0.8, (N + 1, nc)) * pn
        U[:, nj + 1::3] = pn
        U[:, nj + 2::3] = r.uniform(0.0, 1.0, (N + 1, nc))
    else:
        U = np.zeros((N + 1, 3 * nj + 3 * nc))
        U[:, :nj] = r.normal(0.0, model.torque_sigma, (N + 1, nj))
        U[:, nj:3 * nj] = r.normal(0.0, 10.0, (N + 1, 2 * nj))
        U[:, 3 * nj:] = r.uniform(0.0, 30.0, (N + 1, 3 * nc))
    s = r.uniform(0.5, 2.0, N) * dt
    return dict(X=np.ascontiguousarray(X.T), U=np.ascontiguousarray(U.T), s=s, p=model.params())


def _trajectories(case, seed):
    """[(model, K, node data)] of a case."""
    r = np.random.default_rng([7, seed])
    dt = 0.5 * DT if case["model"] == "quad13" else DT
    if case["kind"] in ("batch", "batch_grad"):
        sizes = np.random.default_rng([5, case["T"], case["Nlo"]])   # the same for every seed
        out = []
        for t in range(case["T"]):
            name = MIX[t] if case["model"] == "mixed" else case["model"]
            N = int(sizes.integers(case["Nlo"], case["Nhi"] + 1))
            K = case["K"] + int(sizes.integers(-4, 11)) if case["model"] == "mixed" else case["K"]
            m = _model(name)
            out.append((m, K, _nodes(m, N, r, dt=dt)))
        return out
    m = _model(case["model"])
    return [(m, case["K"], _nodes(m, case["N"], r, paper=case["kind"] == "paper", dt=dt))]


def _seeds(trajs, seed):
    """Cotangents dJ/dF~ [nx, N] of every trajectory."""
    r = np.random.default_rng([13, seed])
    return [r.normal(0.0, 1.0, (d["X"].shape[0], d["s"].shape[0])) for _, _, d in trajs]


def _impact_nodes(case, seed):
    m = _model(case["model"])
    r = np.random.default_rng([17, seed])
    n, nb, nc = case["N"], m.nb, m.nc
    Xm = np.zeros((n, m.nx))
    Xm[:, :3 * nb] = _poses(m, n, r)
    Xm[:, 3 * nb:6 * nb] = r.normal(0.0, 0.5, (n, 3 * nb))
    Xm[:, 6 * nb:] = r.uniform(0.0, 0.1, (n, m.ny))
    Xp = Xm.copy()
    Xp[:, :3 * nb] += r.normal(0.0, 1e-3, (n, 3 * nb))
    Xp[:, 3 * nb:6 * nb] += r.normal(0.0, 0.5, (n, 3 * nb))
    Xp[:, 6 * nb:] += r.uniform(0.0, 0.1, (n, m.ny))
    pn = r.uniform(0.0, 5.0, (n, nc))
    pt = r.uniform(-0.8, 0.8, (n, nc)) * pn
    Phi = np.stack([pt, pn], axis=2).reshape(n, 2 * nc)
    return m, dict(Xp=Xp, Xm=Xm, Phi=Phi, Gamma=r.uniform(0.0, 1.0, (n, nc)), p=m.params())


IMPACT_DELTA, IMPACT_EPS = 0.05, 1e-4


def prepare(case, seed):
    dt = TYPES[case["type"]]

    def dev(a):
        return torch.from_numpy(np.array(a, order="C")).to("cuda").to(dt)

    if case["kind"] == "impact":
        m, d = _impact_nodes(case, seed)
        return dict(case=case, cm=api.CisModel(m), p=dev(d["p"]),
                    **{k: dev(d[k].T) for k in ("Xp", "Xm", "Phi", "Gamma")})
    trajs = _trajectories(case, seed)
    seeds = _seeds(trajs, seed) if "grad" in case["kind"] else None
    if case["kind"] in ("batch", "batch_grad"):
        models = {}
        rows = []
        for m, K, d in trajs:
            cm = models.setdefault(m.name, api.CisModel(m))
            rows.append(dict(cm=cm, X=dev(d["X"]), U=dev(d["U"]), s=dev(d["s"]), params=dev(d["p"]),
                             K=K))
        op = "discretize" if case["kind"] == "batch" else "adjoint"
        plan = api.BatchPlan(rows, (op,))
        if op == "adjoint":
            for o, w in zip(plan.out, seeds):
                o["seed"].copy_(dev(w))
        return dict(case=case, plan=plan, op=op)
    m, K, d = trajs[0]
    st = dict(case=case, cm=api.CisModel(m), K=K, X=dev(d["X"]), U=dev(d["U"]), s=dev(d["s"]),
              p=dev(d["p"]))
    if case["kind"] == "gradient":
        st["seed"] = dev(seeds[0])
        for k in ("X", "U", "s", "p"):
            st[k].requires_grad_(True)
    elif case["kind"] == "split":
        st["ws"] = torch.empty(api.split_workspace_bytes(st["cm"], case["N"], K, dt),
                               device="cuda", dtype=torch.uint8)
    elif case["kind"] == "rkf":
        st["ws"] = torch.empty(api.rkf_workspace_bytes(st["cm"], case["N"], K, dt),
                               device="cuda", dtype=torch.uint8)
    return st


# ---------------------------------------------------------------------------- pass
def run(st):
    kind = st["case"]["kind"]
    if kind in ("batch", "batch_grad"):
        st["plan"].run(st["op"], graph=True)
        keys = (("A", "Bm", "Bp", "S", "d", "xprop") if kind == "batch"
                else ("d", "xprop", "gX", "gU", "gs", "gp"))
        return [{k: o[k] for k in keys} for o in st["plan"].out]
    cm = st["cm"]
    if kind == "impact":
        return api.impact_linearize(cm, st["Xp"], st["Xm"], st["Phi"], st["Gamma"], st["p"],
                                    IMPACT_DELTA, IMPACT_EPS)
    X, U, s, p, K = st["X"], st["U"], st["s"], st["p"], st["K"]
    if kind == "discretize":
        return api.discretize(cm, X, U, s, p, K)
    if kind == "split":
        return api.discretize_split(cm, X, U, s, p, K, waves=2, ws=st["ws"])
    if kind == "rkf":
        return api.discretize_rkf(cm, X, U, s, p, K, ws=st["ws"])
    if kind == "paper":
        return api.discretize_paper(cm, X, U, s, p, K)
    F = api.CisDefects.apply(X, U, s, p, cm, K, st["case"]["C"])
    g = torch.autograd.grad(F, (X, U, s, p), st["seed"])
    return dict(F=F.detach(), gX=g[0], gU=g[1], gs=g[2], gp=g[3])


# ---------------------------------------------------------------------------- work
def _phi_flops(model):
    # operations of one nominal stage (right-hand side and Jacobian nonzeros)
    return {"hopper": 300, "biped5": 700, "cheetah7": 1000, "quad13": 2000}[model.name]


def _forward_work(case, model, N, K, paper=False, rkf=False):
    """Bytes in and out once; operations of the sparse method on dense columns."""
    n = 6 * model.nb
    nx = n + (4 * model.nc + 1 if paper else model.nc + 1)
    m = model.nj + 3 * model.nc if paper else model.m
    size = 8 if case["type"] == "f64" else 4
    by = size * N * (nx * nx + 2 * nx * m + 3 * nx + nx + m + 1)
    c = n + 2 * m + 1
    nnz = 6 * model.nb + 2 * model.nb + 4 * model.nj + 4 * model.nc
    fl = K * (8 * nnz * c + 14 * nx * c + 4 * _phi_flops(model)) * N
    if rkf:
        fl = K * (10 * nnz * c + 28 * nx * c + 6 * _phi_flops(model)) * N
    return by, fl


def work(case):
    if case["kind"] == "impact":
        m = _model(case["model"])
        per = (2 * m.nx + 3 * m.nc + m.nx + 10 * m.nc + m.ny
               + 3 * m.nb * (7 * m.nb + 2 * m.nc) + 140 * m.nc)
        return dict(bytes=8.0 * per * case["N"], flops=2.0 * case["N"] * 3 * m.nb * (2 * m.nj) * 4)
    by = fl = 0.0
    if case["kind"] in ("batch", "batch_grad"):
        sizes = np.random.default_rng([5, case["T"], case["Nlo"]])
        rows = []
        for t in range(case["T"]):
            name = MIX[t] if case["model"] == "mixed" else case["model"]
            N = int(sizes.integers(case["Nlo"], case["Nhi"] + 1))
            K = case["K"] + int(sizes.integers(-4, 11)) if case["model"] == "mixed" else case["K"]
            rows.append((_model(name), N, K))
    else:
        rows = [(_model(case["model"]), case["N"], case["K"])]
    for m, N, K in rows:
        if "grad" in case["kind"]:
            by += 8.0 * N * (2 * (m.nx + m.m + 1) + 3 * m.nx)
            nnz = 8 * m.nb + 4 * m.nj + 4 * m.nc
            fl += N * K * (12.0 * _phi_flops(m) + 8 * (nnz + 2 * m.m) + 28 * m.nx)
        else:
            b, f = _forward_work(case, m, N, K, case["kind"] == "paper", case["kind"] == "rkf")
            by += b
            fl += f
    return dict(bytes=by, flops=fl)


# --------------------------------------------------------------------------- exact
def _sabs(a):
    return a * a / (torch.sqrt(a * a + 1) + 1)


def _ramp(a):
    return torch.where(a > 0, _sabs(a), torch.zeros_like(a))


class _Maps:
    """Right-hand sides of one interval (unbatched; vmap and jacfwd go over them)."""

    def __init__(self, model, dev):
        def t(a):
            return torch.tensor(np.asarray(a, dtype=np.float64), device=dev)

        self.nb, self.nj, self.nc = model.nb, model.nj, model.nc
        self.par = torch.tensor(model.joint_parent, dtype=torch.long, device=dev)
        self.chi = torch.tensor(model.joint_child, dtype=torch.long, device=dev)
        self.cb = torch.tensor(model.contact_body, dtype=torch.long, device=dev)
        eye = torch.eye(self.nb, dtype=torch.float64, device=dev)
        self.EP, self.EC, self.EB = eye[self.par], eye[self.chi], eye[self.cb]
        self.rp, self.rc, self.cr = t(model.anchor_parent), t(model.anchor_child), t(model.contact_point)
        self.k, self.d = t(model.stiffness), t(model.damping)
        self.ipm = t(model.link_length) ** 2 / 12.0
        self.g, self.A, self.kap = model.gravity, model.terrain_amplitude, model.terrain_wavenumber
        # grad h: rows (joint, axis), columns (body, x y theta); the theta entries are filled per pose
        H = torch.zeros(self.nj, 2, self.nb, 3, dtype=torch.float64, device=dev)
        for ax in range(2):
            H[:, ax, :, ax] = self.EP - self.EC
        self.H0 = H

    @staticmethod
    def turn(th, r):
        c, s = torch.cos(th), torch.sin(th)
        return torch.stack([c * r[:, 0] - s * r[:, 1], s * r[:, 0] + c * r[:, 1]], -1)

    def geometry(self, q):
        th = q[:, 2]
        ap, ac = self.turn(th[self.par], self.rp), self.turn(th[self.chi], self.rc)
        a = self.turn(th[self.cb], self.cr)
        P = q[self.cb, :2] + a
        w = self.kap * P[:, 0]
        Hx = -self.A * self.kap * torch.cos(w)
        rG = 1.0 / torch.sqrt(1 + Hx * Hx)
        sd = (P[:, 1] - self.A * torch.sin(w)) * rG
        nn = torch.stack([Hx * rG, rG], -1)
        tt = torch.stack([rG, -Hx * rG], -1)
        return ap, ac, a, sd, nn, tt

    @staticmethod
    def cross(a, f):
        return a[:, 0] * f[:, 1] - a[:, 1] * f[:, 0]

    def speed(self, v, a):
        om = v[self.cb, 2]
        return torch.stack([v[self.cb, 0] - om * a[:, 1], v[self.cb, 1] + om * a[:, 0]], -1)

    def spring(self, q, v):
        return (-self.k * (q[self.chi, 2] - q[self.par, 2])
                - self.d * (v[self.chi, 2] - v[self.par, 2]))

    def base(self, x, u, ub, p):
        nb, nj, nc = self.nb, self.nj, self.nc
        q, v = x[:3 * nb].reshape(nb, 3), x[3 * nb:6 * nb].reshape(nb, 3)
        mu, mass = p[0], p[2:]
        ap, ac, a, sd, nn, tt = self.geometry(q)
        lam = u[nj:3 * nj].reshape(nj, 2)
        tq = u[:nj] + self.spring(q, v)
        L = u[3 * nj:].reshape(nc, 3)
        F = tt * (L[:, 1] - L[:, 2])[:, None] + nn * L[:, 0][:, None]
        force = self.EP.T @ lam - self.EC.T @ lam + self.EB.T @ F
        torque = (self.EP.T @ (self.cross(ap, lam) - tq) + self.EC.T @ (tq - self.cross(ac, lam))
                  + self.EB.T @ self.cross(a, F))
        acc = torch.cat([force / mass[:, None], (torque / (mass * self.ipm))[:, None]], 1)
        acc = acc - torch.tensor([0.0, self.g, 0.0], dtype=x.dtype, device=x.device)
        B = ub[3 * nj:].reshape(nc, 3)
        vt = (tt * self.speed(v, a)).sum(1)
        av = _sabs(vt)
        cc = (B[:, 0] * sd + B[:, 1] * _ramp(vt) + B[:, 2] * _ramp(-vt)
              + (mu * B[:, 0] - B[:, 1] - B[:, 2]) * av)
        h = q[self.par, :2] + ap - q[self.chi, :2] - ac
        ct = _sabs(h).sum() + _ramp(-sd).sum()
        return torch.cat([v.reshape(-1), acc.reshape(-1), cc, ct[None]])

    def grad_h(self, ap, ac):
        th = torch.stack([
            -ap[:, 1][:, None] * self.EP + ac[:, 1][:, None] * self.EC,
            ap[:, 0][:, None] * self.EP - ac[:, 0][:, None] * self.EC], 1)      # [nj, 2, nb]
        full = torch.cat([self.H0[..., :2], th[..., None]], -1)
        return full.reshape(2 * self.nj, 3 * self.nb)

    def minv(self, mass):
        return torch.stack([1 / mass, 1 / mass, 1 / (mass * self.ipm)], 1).reshape(-1)

    def wrench(self, a, F):
        """Generalized forces [3 nb] of contact forces F [nc, 2]."""
        return torch.cat([self.EB.T @ F, (self.EB.T @ self.cross(a, F))[:, None]], 1).reshape(-1)

    def paper(self, x, u, ub, p):
        nb, nj, nc = self.nb, self.nj, self.nc
        q, v = x[:3 * nb].reshape(nb, 3), x[3 * nb:6 * nb].reshape(nb, 3)
        mu, mass = p[0], p[2:]
        ap, ac, a, sd, nn, tt = self.geometry(q)
        tq = u[:nj] + self.spring(q, v)
        c = u[nj:].reshape(nc, 3)
        pt, pn, gm = c[:, 0], c[:, 1], c[:, 2]
        W = self.wrench(a, tt * pt[:, None] + nn * pn[:, None])
        own = torch.stack([torch.zeros_like(mass), -mass * self.g,
                           self.EC.T @ tq - self.EP.T @ tq], 1).reshape(-1)
        W = W + own
        mi = self.minv(mass)
        G = self.grad_h(ap, ac)
        wp, wc = v[self.par, 2], v[self.chi, 2]
        cv = (-(wp * wp)[:, None] * ap + (wc * wc)[:, None] * ac).reshape(-1)
        lam = -(torch.linalg.inv((G * mi) @ G.T) @ (G @ (mi * W) + cv))
        acc = mi * (W + G.T @ lam)
        lc = (tt * self.speed(v, a)).sum(1) + gm * pt / torch.sqrt(pt * pt + 1)
        rc = _sabs(mu * pn) - _sabs(pt)
        ct = (_ramp(-pn) + _ramp(-sd) + _ramp(-gm) + _ramp(-rc)).sum()
        return torch.cat([v.reshape(-1), acc, torch.stack([pn, lc, gm, rc], 1).reshape(-1), ct[None]])

    def impact(self, z, nx, delta):
        """(v+ - v*, Theta) as a function of (x~+, x~-, Phi, Gamma, p)."""
        nb, nc = self.nb, self.nc
        xp, xm = z[:nx], z[nx:2 * nx]
        Phi = z[2 * nx:2 * nx + 2 * nc].reshape(nc, 2)
        Gam = z[2 * nx + 2 * nc:2 * nx + 3 * nc]
        p = z[2 * nx + 3 * nc:]
        mu, e, mass = p[0], p[1], p[2:]
        q = xp[:3 * nb].reshape(nb, 3)
        vp, vm = xp[3 * nb:6 * nb], xm[3 * nb:6 * nb]
        ap, ac, a, sd, nn, tt = self.geometry(q)
        mi = self.minv(mass)
        u = vm + mi * self.wrench(a, tt * Phi[:, :1] + nn * Phi[:, 1:])
        G = self.grad_h(ap, ac)
        vs = u - mi * (G.T @ (torch.linalg.inv((G * mi) @ G.T) @ (G @ u)))
        Pt, Pn = Phi[:, 0], Phi[:, 1]
        w = (nn * self.speed((vp + e * vm).reshape(nb, 3), a)).sum(1)
        lam = (tt * self.speed(vp.reshape(nb, 3), a)).sum(1) + Gam * Pt / torch.sqrt(Pt * Pt + 1)
        rho = _sabs(mu * Pn) - _sabs(Pt)

        def fb(x, y):
            return x + y - torch.sqrt(x * x + y * y + delta)

        th = torch.stack([fb(Pn, sd), fb(Pn, w), Pn * lam - delta, -Pn * lam - delta, fb(Gam, rho),
                          -Pn, -sd, -w, -Gam, -rho], 1)
        return torch.cat([vp - vs, th.reshape(-1)])


# classical RK4, and Fehlberg's 4(5) pair (fourth-order weights, fifth-order weights)
RK4 = dict(c=(0.0, 0.5, 0.5, 1.0), a=((), (0.5,), (0.0, 0.5), (0.0, 0.0, 1.0)),
           b=(1 / 6, 1 / 3, 1 / 3, 1 / 6))
RKF = dict(c=(0.0, 1 / 4, 3 / 8, 12 / 13, 1.0, 1 / 2),
           a=((), (1 / 4,), (3 / 32, 9 / 32), (1932 / 2197, -7200 / 2197, 7296 / 2197),
              (439 / 216, -8.0, 3680 / 513, -845 / 4104),
              (-8 / 27, 2.0, -3544 / 2565, 1859 / 4104, -11 / 40)),
           b=(25 / 216, 0.0, 1408 / 2565, 2197 / 4104, -1 / 5, 0.0),
           b5=(16 / 135, 0.0, 6656 / 12825, 28561 / 56430, -9 / 50, 2 / 55))


def _integrate(f, x0, u0, u1, s, p, K, tab, sens=True):
    """F~ [N, nx], its derivative by (x, U_k, U_k+1, s, p) [N, nx, cols] and the
    embedded estimate [N], each interval with its own substep count K [N]."""
    N, nx = x0.shape
    m, P = u0.shape[1], p.shape[1]
    ub = 0.5 * (u0 + u1)
    h = 1.0 / K
    x, err = x0, torch.zeros_like(s)
    Z = None
    if sens:
        Z = torch.zeros(N, nx, nx + 2 * m + 1 + P, dtype=x0.dtype, device=x0.device)
        Z[:, :, :nx] = torch.eye(nx, dtype=x0.dtype, device=x0.device)
    jac = torch.func.vmap(torch.func.jacfwd(lambda z: f(z[:nx], z[nx:nx + m], z[nx + m:nx + 2 * m],
                                                        z[nx + 2 * m:])))
    val = torch.func.vmap(f)
    stages = len(tab["c"])
    for j in range(int(K.max())):
        live = (K > j).to(x0.dtype)
        ks, kz = [], []
        for i in range(stages):
            tau = ((j + tab["c"][i]) * h)[:, None]
            u = (1 - tau) * u0 + tau * u1
            xi = x + sum((h[:, None] * a) * k for a, k in zip(tab["a"][i], ks) if a != 0.0)
            F = val(xi, u, ub, p)
            ks.append(s[:, None] * F)
            if sens and (i < 5):
                zi = Z + sum((h[:, None, None] * a) * k for a, k in zip(tab["a"][i], kz) if a != 0.0)
                J = jac(torch.cat([xi, u, ub, p], 1))
                d = torch.bmm(J[:, :, :nx].contiguous(), zi)
                Ju, Jb = J[:, :, nx:nx + m], J[:, :, nx + m:nx + 2 * m]
                d[:, :, nx:nx + m] += (1 - tau)[:, :, None] * Ju + 0.5 * Jb
                d[:, :, nx + m:nx + 2 * m] += tau[:, :, None] * Ju + 0.5 * Jb
                d *= s[:, None, None]
                d[:, :, nx + 2 * m] += F
                d[:, :, nx + 2 * m + 1:] += s[:, None, None] * J[:, :, nx + 2 * m:]
                kz.append(d)
        hl = (h * live)[:, None]
        x = x + sum((hl * b) * k for b, k in zip(tab["b"], ks) if b != 0.0)
        if "b5" in tab:
            e = sum((hl * (b5 - b)) * k for b, b5, k in zip(tab["b"], tab["b5"], ks))
            err = torch.maximum(err, e.abs().amax(1))
        if sens:
            Z = Z + sum((hl[:, :, None] * b) * k for b, k in zip(tab["b"], kz) if b != 0.0)
    return x, Z, err


def _exact_trajs(case, seed):
    """Per trajectory: X_k, X_k+1 (rows last), F~, Z, err, in FP64 on the rounded inputs."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    rnd = np.float32 if case["type"] == "f32" else np.float64
    trajs = _trajectories(case, seed)
    out = [None] * len(trajs)
    for name in sorted({m.name for m, _, _ in trajs}):
        ids = [i for i, (m, _, _) in enumerate(trajs) if m.name == name]
        maps = _Maps(trajs[ids[0]][0], dev)

        def cat(pick):
            a = np.concatenate([np.asarray(pick(trajs[i])) for i in ids], 0)
            return torch.from_numpy(a.astype(rnd).astype(np.float64)).to(dev)

        n_of = [trajs[i][2]["s"].shape[0] for i in ids]
        x0, x1 = cat(lambda t: t[2]["X"].T[:-1]), cat(lambda t: t[2]["X"].T[1:])
        u0, u1 = cat(lambda t: t[2]["U"].T[:-1]), cat(lambda t: t[2]["U"].T[1:])
        s = cat(lambda t: t[2]["s"])
        p = cat(lambda t: np.tile(t[2]["p"], (t[2]["s"].shape[0], 1)))
        K = torch.cat([torch.full((n,), float(trajs[i][1]), dtype=torch.float64, device=dev)
                       for i, n in zip(ids, n_of)])
        f = maps.paper if case["kind"] == "paper" else maps.base
        tab = RKF if case["kind"] == "rkf" else RK4
        parts = []
        for at in range(0, x0.shape[0], 1024):
            sl = slice(at, at + 1024)
            parts.append(_integrate(f, x0[sl], u0[sl], u1[sl], s[sl], p[sl], K[sl], tab))
        F, Z, err = (torch.cat([q[e] for q in parts]) for e in range(3))
        at = 0
        for i, n in zip(ids, n_of):
            sl = slice(at, at + n)
            out[i] = (x1[sl], F[sl], Z[sl], err[sl])
            at += n
    return trajs, out


def exact(case, seed):
    if case["kind"] == "impact":
        return _exact_impact(case, seed)
    trajs, res = _exact_trajs(case, seed)
    out = []
    for (m, K, d), (x1, F, Z, err), w in zip(trajs, res, _seeds(trajs, seed)):
        nx, mu = d["X"].shape[0], d["U"].shape[0]
        A, Bm, Bp = Z[:, :, :nx], Z[:, :, nx:nx + mu], Z[:, :, nx + mu:nx + 2 * mu]
        S, Pi = Z[:, :, nx + 2 * mu], Z[:, :, nx + 2 * mu + 1:]
        soa = {"d": (F - x1).T, "xprop": F.T}
        if "grad" in case["kind"]:
            lam = torch.from_numpy(w.T.copy()).to(F.device)[:, :, None]
            N = lam.shape[0]
            gX = torch.zeros(nx, N + 1, dtype=F.dtype, device=F.device)
            gX[:, :N] = (A * lam).sum(1).T
            gU = torch.zeros(mu, N + 1, dtype=F.dtype, device=F.device)
            gU[:, :N] += (Bm * lam).sum(1).T
            gU[:, 1:] += (Bp * lam).sum(1).T
            soa.update(gX=gX, gU=gU, gs=(S * lam[:, :, 0]).sum(1),
                       gp=(Pi * lam).sum(1).sum(0))
            if case["kind"] == "gradient":
                soa["F"] = soa.pop("xprop")
                del soa["d"]
        else:
            soa.update(A=A.permute(1, 2, 0), Bm=Bm.permute(1, 2, 0), Bp=Bp.permute(1, 2, 0), S=S.T)
            if case["kind"] == "rkf":
                soa["err"] = err
        out.append({k: v.contiguous() for k, v in soa.items()})
    return out if case["kind"] in ("batch", "batch_grad") else out[0]


def _exact_impact(case, seed):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    m, d = _impact_nodes(case, seed)
    maps = _Maps(m, dev)
    nb, nc, nx, nq = m.nb, m.nc, m.nx, 3 * m.nb
    n = case["N"]

    def t(a):
        return torch.from_numpy(np.ascontiguousarray(a)).to(dev)

    z = torch.cat([t(d["Xp"]), t(d["Xm"]), t(d["Phi"]), t(d["Gamma"]), t(np.tile(d["p"], (n, 1)))], 1)

    def f(v):
        return maps.impact(v, nx, IMPACT_DELTA)

    fv, jv = torch.func.vmap(f), torch.func.vmap(torch.func.jacfwd(f))
    val = torch.cat([fv(z[a:a + 1024]) for a in range(0, n, 1024)])
    J = torch.cat([jv(z[a:a + 1024]) for a in range(0, n, 1024)])
    phi0, gam0, p0 = 2 * nx, 2 * nx + 2 * nc, 2 * nx + 3 * nc
    cols = (list(range(nq)) + list(range(nx + nq, nx + 2 * nq)) + list(range(phi0, phi0 + 2 * nc))
            + list(range(p0 + 2, p0 + 2 + nb)))
    G = t(d["Xp"]) - t(d["Xm"])
    G[:, nq:2 * nq] = val[:, :nq]
    JTc = torch.empty(n, 10 * nc, 14, dtype=torch.float64, device=dev)
    for i in range(nc):
        b = int(m.contact_body[i])
        c = ([3 * b + e for e in range(3)] + [nq + 3 * b + e for e in range(3)]
             + [nx + nq + 3 * b + e for e in range(3)]
             + [phi0 + 2 * i, phi0 + 2 * i + 1, gam0 + i, p0, p0 + 1])
        JTc[:, 10 * i:10 * i + 10] = J[:, nq + 10 * i:nq + 10 * i + 10][:, :, c]
    relax = torch.full((m.ny,), IMPACT_DELTA, dtype=torch.float64, device=dev)
    relax[-1] = IMPACT_EPS
    Psi = t(d["Xm"][1:, 2 * nq:]) - t(d["Xp"][:-1, 2 * nq:]) - relax
    return dict(G=G, Theta=val[:, nq:].contiguous(), JGv=J[:, :nq][:, :, cols].contiguous(), JTc=JTc,
                Psi=Psi)
