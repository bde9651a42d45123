"""The workloads that the library's speed is measured on.

Every case is one call that a program makes through the public entry points
(``binding.Engine`` / ``binding.FbEngine`` / ``autograd.jd_cost``): one Monte
Carlo cost and gradient, one differentiated cost, or one run of the Armijo
gradient iteration.  ``listed()`` names twelve of them, from the smallest
problems (where latency and launches count) to the largest; ``draw`` gives more
from the same ranges:

  open-loop model  d = 1..8, 2^11..2^20 paths, 50..2000 steps, FP32 and FP64
                   paths, stored trajectory or checkpoints every 16, 32 or 64
                   steps, linear and cubic drift; the gradient iteration with
                   1000..65536 paths and 50..300 steps
  particle model   500..2^20 particles, 50..500 steps, FP32 and FP64 paths,
                   fixed and jump-adapted grid, rings of 2..2048 particles,
                   exact and surrogate gradient, mostly the 10 x 10 grid of
                   shape functions; the gradient iteration with 500..16384
                   particles

``exact`` evaluates the same definitions (the draws, the Euler steps, the cost,
the discrete adjoint) in 64 bits with plain torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2505_04328_amd import autograd as jd_autograd
from paper_2505_04328_amd import binding as jdb
from paper_2505_04328_amd import workloads as wl

OPEN = dict(model="open", call="grad", d=1, N=1000, M=1 << 20, T=1.0, lam=5.0, cubic=0.0,
            jump_mean=0.0, jump_std=0.2, precision="fp32", mode="store", K=0, iters=0)
FB = dict(model="fb", call="grad", N=50, M=2000, T=5.0, np=1, grid="fixed", init="gauss",
          mode="store", svar="given", nx=10, nv=10, precision="fp32", iters=0)


def listed():
    return [
        # The published experiments' size: 2000 particles, 50 steps of 0.1, 10 x 10 shape
        # functions; one gradient.
        dict(FB, name="paper_cloud_grad"),
        # One ring of 2000 coupled particles at the published step count, FP64 paths.
        dict(FB, name="paper_ring_grad_fp64", M=1, np=2000, init="ellipse", precision="fp64"),
        # The whole gradient iteration on the jump-adapted grid at the published size.
        dict(FB, name="paper_adapted_descent", grid="adapted", call="optimize", iters=10),
        # The 1-D problem solved to the end: 20 FP64 gradient iterations of 10^4 paths.
        dict(OPEN, name="ou_descent_fp64", call="optimize", N=100, M=10_000, lam=2.0,
             precision="fp64", iters=20),
        # One gradient of a request in the middle of the serving mix, ragged path count.
        dict(OPEN, name="request_grad_d4", d=4, N=777, M=150_001, lam=6.0),
        # The headline gradient: 2^20 paths x 1000 steps, 1-D, FP32 paths.
        dict(OPEN, name="ou_grad_1m", jump_mean=-0.1, jump_std=0.3),
        # The same with FP64 paths.
        dict(OPEN, name="ou_grad_1m_fp64", jump_mean=-0.1, jump_std=0.3, precision="fp64"),
        # Eight coupled components, stored trajectory (16.8 GB).
        dict(OPEN, name="linear8_grad_1m", d=8, N=500, T=2.0, lam=3.0),
        # Differentiating the cost with checkpoints instead of the trajectory, cubic drift.
        dict(OPEN, name="cubic8_autograd", call="autograd", d=8, N=2000, M=1 << 18, T=2.0,
             lam=3.0, cubic=0.1, mode="recompute", K=64),
        # The particle model at scale: independent particles, rings, jump-adapted grid.
        dict(FB, name="cloud_grad_1m", N=500, M=1 << 20),
        dict(FB, name="ring_grad_512x2000", N=500, M=512, np=2000, init="ellipse"),
        dict(FB, name="adapted_grad_1m", N=500, M=1 << 20, grid="adapted"),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        c = _draw_one(rng)
        if _milliseconds(c) <= 20.0:
            return c


def _draw_one(rng):
    kind = rng.choices(["grad", "autograd", "optimize", "cloud", "ring", "adapted", "surrogate",
                        "fb_optimize"], [6, 2, 3, 4, 2, 2, 1, 2])[0]
    if kind in ("grad", "autograd", "optimize"):
        c = dict(OPEN, d=rng.choice([1, 1, 2, 3, 4, 6, 8]), N=_logint(rng, 50, 2000),
                 M=_logint(rng, 1 << 11, 1 << 20), T=rng.choice([1.0, 2.0]),
                 lam=round(rng.uniform(0.0, 10.0), 3), cubic=rng.choice([0.0, 0.0, 0.1]),
                 precision=rng.choice(["fp32", "fp32", "fp64"]), call=kind)
        if kind == "optimize":
            c.update(M=_logint(rng, 1000, 65536), N=_logint(rng, 50, 300),
                     iters=rng.randint(5, 30))
        if kind == "autograd" or rng.random() < 0.25:
            c.update(mode="recompute", K=min(c["N"], rng.choice([16, 32, 64])))
        return c
    c = dict(FB, N=_logint(rng, 50, 500), precision=rng.choice(["fp32", "fp32", "fp64"]),
             init=rng.choice(["gauss", "uniform"]), M=_logint(rng, 500, 1 << 20))
    if rng.random() < 0.25:
        c.update(nx=rng.randint(4, 16), nv=rng.randint(4, 16))
    if kind == "ring":
        npr = rng.choice([_logint(rng, 2, 256), rng.randint(257, 2048), 2000])
        c.update(np=npr, M=max(1, c["M"] // npr), init="ellipse")
    elif kind == "adapted":
        c["grid"] = "adapted"
    elif kind == "surrogate":
        c.update(mode="surrogate", svar=rng.choice(["given", "fit"]))
    elif kind == "fb_optimize":
        c.update(call="optimize", iters=rng.randint(3, 12), N=_logint(rng, 50, 150),
                 M=_logint(rng, 500, 16384), grid=rng.choice(["fixed", "adapted"]))
    return c


def _milliseconds(c):
    """A pass's time, roughly, so that a drawn case costs no more than the largest listed one."""
    units = float(c["M"]) * c["N"] * c.get("np", 1)
    sweeps = 2.0 * c["iters"] if c["call"] == "optimize" else 1.0
    if c["model"] == "open":
        ns = 1e-3 * (1.0 + 2.0 * c["d"]) * (1.8 if c["mode"] == "recompute" else 1.0)
    else:
        ns = 25e-3 * (1.9 if c["grid"] == "adapted" else 1.3 if c["mode"] == "surrogate" else 1.0)
        ns *= max(1.0, c["nx"] * c["nv"] / 100.0)
    if c["precision"] == "fp64":
        ns *= 3.3
    return sweeps * units * ns * 1e-6


# ---------------------------------------------------------------------------
# Inputs.

def _open_data(case, seed):
    """The open-loop problem's arrays: the 1-D Ornstein-Uhlenbeck model, or for
    d > 1 a stable symmetric drift with random diffusion scales."""
    d, N, T = case["d"], case["N"], case["T"]
    rng = np.random.default_rng(seed)
    t = np.arange(N) * (T / N)
    if d == 1:
        A, s = np.array([[-1.0]]), np.array([0.3])
    else:
        q, r = np.linalg.qr(rng.standard_normal((d, d)))
        q = q * np.sign(np.diag(r))
        A = (q * rng.uniform(-2.0, -0.2, d)) @ q.T
        s = rng.uniform(0.1, 0.5, d)
    u = 0.5 * np.sin(2.0 * math.pi * t[:, None] / T + rng.uniform(0, 2 * math.pi, d))
    u = u + 0.05 * rng.standard_normal((N, d))
    if case["call"] == "optimize":
        u = np.zeros((N, d))
    return dict(A=A, B=np.eye(d), s=s, x0=np.zeros(d), xT=np.ones(d), u=u, nu=1e-3,
                jm=np.full(d, case["jump_mean"]), js=np.full(d, case["jump_std"]),
                xd=np.repeat(np.sin(2.0 * math.pi * t)[:, None], d, axis=1), key=1 + seed)


def _fb_data(case, seed):
    """The particle model's numbers: the settings of workloads.feedback_problem."""
    N, T = case["N"], case["T"]
    rng = np.random.default_rng(seed)
    L = case["nx"] * case["nv"]
    mu = np.zeros((N, L)) if case["call"] == "optimize" else rng.normal(0.0, 0.5, (N, L))
    zd = np.zeros((N + 1, 2))
    ring = case["init"] == "ellipse"
    z0, s0 = {"gauss": ((0.75, 0.75), (0.1, 0.1)), "uniform": ((0.0, 0.0), (1.0, 1.0)),
              "ellipse": ((0.0, 0.0), (0.0, 0.0))}[case["init"]]
    rate = math.sqrt(10.0 / math.pi)
    v0 = np.array(s0) ** 2 / (1.0 if case["init"] == "gauss" else 3.0)
    return dict(mu=mu, zd=zd, z0=z0, s0=s0, ring=ring, eta=1.0, b1=0.05, b2=0.1, gamma=0.9,
                beta=10.0, rate=rate, xmax=2.0, vmax=2.0, eps=0.5, alpha=1e-2, sigJ=0.5,
                omega=0.5 if ring else 0.0, ax=1.5, av=1.7071067811865475, svar0=v0,
                svar1=np.array([0.05 ** 2, 0.1 ** 2 + rate / 20.0]), key=1 + seed)


ZETA0 = {"open": 1.0, "fb": 10.0}


def prepare(case, seed):
    dev = "cuda:0"
    if case["model"] == "open":
        q = _open_data(case, seed)
        p = wl.Problem(d=case["d"], N=case["N"], T=case["T"], lam=case["lam"],
                       cubic=case["cubic"], nu=q["nu"], x0=q["x0"], A=q["A"], B=q["B"], s=q["s"],
                       jump_mean=q["jm"], jump_std=q["js"], xT=q["xT"], xd=q["xd"])
        eng = jdb.Engine(p, M=case["M"], seed=q["key"], precision=case["precision"],
                         mode=case["mode"], K=case["K"], device=dev)
        u = torch.from_numpy(np.ascontiguousarray(q["u"])).to(dev)
        if case["call"] == "autograd":
            u.requires_grad_(True)
    else:
        q = _fb_data(case, seed)
        p = wl.feedback_problem(
            N=case["N"], T=case["T"], init=case["init"], zd=q["zd"], eta=q["eta"], b1=q["b1"],
            b2=q["b2"], gamma=q["gamma"], beta=q["beta"], nx=case["nx"], nv=case["nv"],
            xmax=q["xmax"], vmax=q["vmax"], eps=q["eps"], alpha=q["alpha"], sigJ=q["sigJ"],
            z0=q["z0"], s0=q["s0"], svar0=q["svar0"], svar1=q["svar1"], np_=case["np"],
            omega=q["omega"], cost="ellipse" if q["ring"] else "track", ax=q["ax"], av=q["av"],
            grid=case["grid"], svar=case["svar"])
        eng = jdb.FbEngine(p, M=case["M"], seed=q["key"], precision=case["precision"], device=dev,
                           mode=case["mode"])
        u = torch.from_numpy(q["mu"]).to(dev)
    return dict(case=case, eng=eng, u=u)


def run(state):
    case, eng, u = state["case"], state["eng"], state["u"]
    if case["call"] == "grad":
        J, g = eng.cost_grad(u)
        return {"J": J, "g": g}
    if case["call"] == "autograd":
        u.grad = None
        J = jd_autograd.jd_cost(u, eng)
        J.backward()
        return {"J": J.detach(), "u_grad": u.grad}
    u, log = eng.optimize(u.clone(), n_max=case["iters"], zeta0=ZETA0[case["model"]])
    return {"u": u, "backtracks": np.array([e["backtracks"] for e in log], np.int64),
            **{k: np.array([e[k] for e in log]) for k in ("J", "gnorm", "zeta", "J_new")}}


def work(case):
    """The control and the target read, the cost and gradient (or the control)
    written; and the arithmetic of the method per path and step, a fused
    multiply-add as two: the Philox blocks (60 each), the Box-Muller pairs, the
    Euler step, the cost and the adjoint step.  The gradient iteration counts one
    trial per iteration."""
    N = case["N"]
    if case["model"] == "open":
        d = case["d"]
        fwd = 60 * ((d + 1) // 2) + 8 * d + 2 * d * d + 6 * d + 3 * d + (4 * d if case["cubic"] else 0)
        adj = 2 * d * d + 4 * d + (5 * d if case["cubic"] else 0)
        units, nbytes = float(case["M"]) * N, 8.0 * (3 * N * d + 1)
    else:
        nx, nv = case["nx"], case["nv"]
        fwd = 6 * (nx + nv) + 2 * nx * nv + 3 * nx + 60 + 40
        adj = 9 * (nx + nv) + 4 * nx * nv + 6 * nx + 2 * nx * nv + 40
        if case["grid"] == "adapted":
            more = 1.0 + math.sqrt(10.0 / math.pi) * case["T"] / N  # sub-steps per interval
            fwd, adj = fwd * more, adj * more
        units = float(case["M"]) * case["np"] * N
        nbytes = 8.0 * (2 * N * nx * nv + 2 * (N + 1) + 1)
    if case["call"] == "optimize":
        return {"bytes": nbytes * case["iters"], "flops": units * (2 * fwd + adj) * case["iters"]}
    return {"bytes": nbytes, "flops": units * (fwd + adj)}


# ---------------------------------------------------------------------------
# The same values in 64 bits with plain torch.

_F = torch.float64
_MASK = 0xFFFFFFFF


def _device():
    return "cuda:0" if torch.cuda.is_available() else "cpu"


def _philox(m, k, it, blk, key):
    """Philox4x32-10 words of the counters (m, k, it, blk) under the 64-bit key."""
    k0, k1 = key & _MASK, key >> 32
    c = [m, k, torch.as_tensor(it, device=m.device), torch.as_tensor(blk, device=m.device)]
    for _ in range(10):
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
        c = [((p1 >> 32) & _MASK) ^ c[1] ^ k0, p1 & _MASK, ((p0 >> 32) & _MASK) ^ c[3] ^ k1,
             p0 & _MASK]
        k0, k1 = (k0 + 0x9E3779B9) & _MASK, (k1 + 0xBB67AE85) & _MASK
    return torch.broadcast_tensors(*c)


def _unit(w):
    return ((w >> 8) | 1).to(_F) * 2.0 ** -24


def _pair(wa, wb):
    r, th = torch.sqrt(-2.0 * torch.log(_unit(wa))), 2.0 * math.pi * _unit(wb)
    return r * torch.cos(th), r * torch.sin(th)


def _counts(w, thr):
    return torch.bucketize((w[0] & 255) | (w[1] & 255) << 8 | (w[2] & 255) << 16 | (w[3] & 255) << 24,
                           thr, right=True)


def _thresholds(mean, dev):
    p = F = math.exp(-mean)
    out = []
    for j in range(31):
        if j:
            p = p * mean / j
            F = F + p
        out.append(min(1 << 32, math.floor(math.ldexp(F, 32))))
    return torch.tensor(out, dtype=torch.int64, device=dev)


class _Open:
    """J and g of the open-loop model."""

    def __init__(self, case, seed):
        self.c, self.dev = case, _device()
        q = _open_data(case, seed)
        self.key, self.nu = q["key"], q["nu"]
        self.t = {k: torch.from_numpy(np.ascontiguousarray(q[k])).to(self.dev, _F)
                  for k in ("A", "B", "s", "x0", "xT", "u", "jm", "js", "xd")}
        self.dt = case["T"] / case["N"]
        self.thr = _thresholds(case["lam"] * self.dt, self.dev)
        self.m = torch.arange(case["M"], dtype=torch.int64, device=self.dev)
        self.kept = {}

    def noise(self, it, k):
        """The Brownian term and jump increment (d, M) of step k; a few steps at a time."""
        per = max(1, (1 << 22) // self.c["M"])
        at = (it, k // per)
        if at not in self.kept:
            if self.c["call"] != "optimize" or (self.kept and next(iter(self.kept))[0] != it):
                self.kept.clear()
            k0 = k // per * per
            ks = torch.arange(k0, min(k0 + per, self.c["N"]), dtype=torch.int64, device=self.dev)
            d, zw, zj, n = self.c["d"], [], [], None
            for b in range((d + 1) // 2):
                w = _philox(self.m[None, :], ks[:, None], it, b, self.key)
                n = _counts(w, self.thr) if b == 0 else n
                for i in range(2 * b, min(2 * b + 2, d)):
                    x, y = _pair(w[2 * (i % 2)], w[2 * (i % 2) + 1])
                    zw.append(x)
                    zj.append(y)
            n = n.to(_F)[:, None, :]
            zw, zj = torch.stack(zw, 1), torch.stack(zj, 1)
            bw = math.sqrt(self.dt) * self.t["s"][None, :, None] * zw
            dj = n * self.t["jm"][None, :, None] + self.t["js"][None, :, None] * torch.sqrt(n) * zj
            self.kept[at] = bw + dj
        return self.kept[at][k % per]

    def forward(self, u, it, keep):
        t, dt, c3 = self.t, self.dt, self.c["cubic"]
        X = t["x0"][:, None].expand(-1, self.c["M"]).contiguous()
        acc, path = torch.zeros(self.c["M"], dtype=_F, device=self.dev), []
        bu = u @ t["B"].T
        for k in range(self.c["N"]):
            if keep:
                path.append(X)
            acc += (X - t["xd"][k][:, None]).square().sum(0)
            f = t["A"] @ X + bu[k][:, None]
            if c3:
                f = f - c3 * X * X * X
            X = X + dt * f + self.noise(it, k)
        C = 0.5 * dt * acc + 0.5 * (X - t["xT"][:, None]).square().sum(0)
        return C.mean() + 0.5 * self.nu * dt * u.square().sum(), X, path

    def grad(self, u, it):
        t, dt, c3 = self.t, self.dt, self.c["cubic"]
        J, X, path = self.forward(u, it, True)
        lam = X - t["xT"][:, None]
        g = torch.empty_like(u)
        for k in range(self.c["N"] - 1, -1, -1):
            g[k] = self.nu * u[k] + t["B"].T @ lam.mean(1)
            X = path.pop()
            a = t["A"].T @ lam + (X - t["xd"][k][:, None])
            if c3:
                a = a - 3.0 * c3 * X * X * lam
            lam = lam + dt * a
        return J, g


class _Particles:
    """J and g of the particle model: fixed grid (independent particles and
    rings), jump-adapted grid, surrogate gradient."""

    def __init__(self, case, seed):
        self.c, self.dev = case, _device()
        self.q = q = _fb_data(case, seed)
        self.key, self.dt = q["key"], case["T"] / case["N"]
        self.P = case["M"] * case["np"]
        self.m = torch.arange(self.P, dtype=torch.int64, device=self.dev)
        self.u = torch.from_numpy(q["mu"]).to(self.dev)
        self.zd = q["zd"]
        self.thr = _thresholds(q["rate"] * self.dt, self.dev)
        dx, dv = 2 * q["xmax"] / case["nx"], 2 * q["vmax"] / case["nv"]
        self.xc = (torch.arange(case["nx"], device=self.dev, dtype=_F) + 0.5) * dx - q["xmax"]
        self.vc = (torch.arange(case["nv"], device=self.dev, dtype=_F) + 0.5) * dv - q["vmax"]
        self.kept = {}

    def start(self, it):
        q = self.q
        w = _philox(self.m, torch.as_tensor(_MASK, device=self.dev), it, 0, self.key)
        if self.c["init"] == "uniform":
            return (q["z0"][0] + q["s0"][0] * (2 * _unit(w[0]) - 1),
                    q["z0"][1] + q["s0"][1] * (2 * _unit(w[1]) - 1))
        a, b = _pair(w[0], w[1])
        if self.c["init"] == "gauss":
            return q["z0"][0] + q["s0"][0] * a, q["z0"][1] + q["s0"][1] * b
        th = 2.0 * math.pi * (self.m % self.c["np"]).to(_F) / self.c["np"]
        return q["ax"] * torch.cos(th) + q["s0"][0] * a, q["av"] * torch.sin(th) + q["s0"][1] * b

    def step_draws(self, it, k):
        """(Zx, Zv, ZJ, n) of step k; a few steps at a time."""
        per = max(1, (1 << 22) // self.P)
        at = (it, k // per)
        if at not in self.kept:
            if self.c["call"] != "optimize" or (self.kept and next(iter(self.kept))[0] != it):
                self.kept.clear()
            k0 = k // per * per
            ks = torch.arange(k0, min(k0 + per, self.c["N"]), dtype=torch.int64, device=self.dev)
            w = _philox(self.m[None, :], ks[:, None], it, 0, self.key)
            self.kept[at] = (*_pair(w[0], w[1]), _pair(w[2], w[3])[0], _counts(w, self.thr))
        return tuple(x[k % per] for x in self.kept[at])

    def bumps(self, z, c0, deriv=False):
        """b(z - c_i) (centres x particles) and, if asked, its derivative."""
        eps = self.q["eps"]
        r = z[None, :] - c0[:, None]
        s = 1.0 - (eps * r).square()
        inside = s > 0
        s = torch.where(inside, s, torch.ones_like(s))
        b = torch.where(inside, torch.exp(-1.0 / s), torch.zeros_like(s))
        return (b, b * (-2.0 * eps * eps) * r / (s * s)) if deriv else b

    def control(self, mu_k, x, v):
        px, pv = self.bumps(x, self.xc), self.bumps(v, self.vc)
        return (px * (mu_k.view(self.c["nx"], self.c["nv"]) @ pv)).sum(0)

    def control_d(self, mu_k, x, v):
        (px, dx), (pv, dv) = self.bumps(x, self.xc, True), self.bumps(v, self.vc, True)
        mu = mu_k.view(self.c["nx"], self.c["nv"])
        t = mu @ pv
        return (px * t).sum(0), (dx * t).sum(0), (px * (mu @ dv)).sum(0), px, pv

    def project(self, px, pv, w):
        """sum_p px[i, p] pv[l, p] w[p], the particles in chunks."""
        n = w.shape[0]
        ch = 4096
        if n <= ch:
            return (px @ (pv * w).T).reshape(-1)
        body = n // ch * ch
        a = px[:, :body].reshape(px.shape[0], -1, ch).transpose(0, 1).contiguous()
        b = (pv * w)[:, :body].reshape(pv.shape[0], -1, ch).permute(1, 2, 0).contiguous()
        out = torch.bmm(a, b).sum(0)
        if body < n:
            out = out + px[:, body:] @ (pv[:, body:] * w[body:]).T
        return out.reshape(-1)

    def track(self, x, v, zd, grad=False):
        q = self.q
        s2 = q["sigJ"] ** 2
        if q["ring"]:
            e = (x / q["ax"]).square() + (v / q["av"]).square() - 1.0
            J = -torch.exp(-e * e / (2 * s2))
            return (-J * e / s2 * 2 * x / q["ax"] ** 2, -J * e / s2 * 2 * v / q["av"] ** 2) if grad else J
        rx, rv = x - zd[0], v - zd[1]
        J = -torch.exp(-(rx * rx + rv * rv) / (2 * s2))
        return (-J * rx / s2, -J * rv / s2) if grad else J

    def sides(self, x):
        r = x.view(self.c["M"], self.c["np"])
        return (torch.roll(r, 1, 1) + torch.roll(r, -1, 1)).reshape(-1)

    def factors(self, n):
        """gamma^n and sqrt(V_n)."""
        q = self.q
        g = q["gamma"] ** n.to(_F)
        V = (1.0 - g * g) / (1.0 - q["gamma"] ** 2) / (2.0 * q["beta"])
        return g, torch.sqrt(V)

    def forward(self, mu, it, keep):
        if self.c["grid"] == "adapted":
            return self.forward_adapted(mu, it, keep)
        q, dt, sq = self.q, self.dt, math.sqrt(self.dt)
        x, v = self.start(it)
        acc, path = torch.zeros(self.P, dtype=_F, device=self.dev), []
        for k in range(self.c["N"]):
            zx, zv, zj, n = self.step_draws(it, k)
            gn, sv = self.factors(n)
            u = self.control(mu[k], x, v)
            if keep:
                path.append((x, v, gn))
            f = u - q["eta"] * x
            if q["ring"]:
                f = f - q["omega"] * (2.0 * x - self.sides(x))
            x, v = x + dt * v + q["b1"] * sq * zx, gn * (v + dt * f + q["b2"] * sq * zv) + sv * zj
            acc += 0.5 * dt * q["alpha"] * u * u + dt * self.track(x, v, self.zd[k + 1])
        return acc.mean(), (x, v), path

    def grad(self, mu, it):
        if self.c["mode"] == "surrogate":
            return self.grad_surrogate(mu, it)
        J, end, path = self.forward(mu, it, True)
        if self.c["grid"] == "adapted":
            return J, self.adjoint_adapted(mu, path)
        q, dt, N = self.q, self.dt, self.c["N"]
        gx, gv = self.track(*end, self.zd[N], True)
        lx, lv = dt * gx, dt * gv
        g = torch.empty_like(mu)
        for k in range(N - 1, -1, -1):
            x, v, gn = path.pop()
            u, ux, uv, px, pv = self.control_d(mu[k], x, v)
            w = gn * lv
            g[k] = self.project(px, pv, q["alpha"] * u + w) / self.P
            gx, gv = self.track(x, v, self.zd[k], True)
            nlx = lx + dt * (ux - q["eta"]) * w + dt * gx + dt * q["alpha"] * u * ux
            if q["ring"]:
                nlx = nlx + dt * q["omega"] * (self.sides(w) - 2.0 * w)
            lx, lv = nlx, dt * lx + (1.0 + dt * uv) * w + dt * gv + dt * q["alpha"] * u * uv
        return J, g

    def grad_surrogate(self, mu, it):
        q, dt, N = self.q, self.dt, self.c["N"]
        J, end, path = self.forward(mu, it, True)
        g = torch.empty_like(mu)
        var = torch.zeros(N + 1, 2, dtype=_F, device=self.dev)
        gns = []
        for k in range(N + 1):
            x, v = path[k][:2] if k < N else end
            var[k, 0], var[k, 1] = x.var(correction=0), v.var(correction=0)
            if k < N:
                u = self.control(mu[k], x, v)
                g[k] = self.project(self.bumps(x, self.xc), self.bumps(v, self.vc), q["alpha"] * u)
                gns.append(path[k][2])
        t = torch.arange(N + 1, dtype=_F, device=self.dev)[:, None] * dt
        if self.c["svar"] == "fit":
            tc = t - t.mean()
            b = (tc * (var - var.mean(0))).sum(0) / tc.square().sum()
            a = var.mean(0) - b * t.mean()
        else:
            a, b = (torch.as_tensor(z, dtype=_F, device=self.dev) for z in (q["svar0"], q["svar1"]))
        sd = torch.sqrt(torch.clamp(a + b * t, min=0.0))
        w = _philox(self.m, torch.as_tensor(0xFFFFFFFE, device=self.dev), it, 1, self.key)
        sx, sv = _pair(w[0], w[1])
        state = lambda k: (self.zd[k][0] + sd[k, 0] * sx, self.zd[k][1] + sd[k, 1] * sv)  # noqa: E731
        gx, gv = self.track(*state(N), self.zd[N], True)
        lx, lv = dt * gx, dt * gv
        for k in range(N - 1, -1, -1):
            x, v = state(k)
            u, ux, uv, px, pv = self.control_d(mu[k], x, v)
            w = gns[k] * lv
            g[k] = (g[k] + self.project(px, pv, w)) / self.P
            gx, gv = self.track(x, v, self.zd[k], True)
            lx, lv = (lx + dt * (ux - q["eta"]) * w + dt * gx + dt * q["alpha"] * u * ux,
                      dt * lx + (1.0 + dt * uv) * w + dt * gv + dt * q["alpha"] * u * uv)
        return J, g

    def target(self, k, a):
        z0, z1 = self.zd[k], self.zd[k + 1]
        return (1.0 - a) * z0[0] + a * z1[0], (1.0 - a) * z0[1] + a * z1[1]

    def forward_adapted(self, mu, it, keep):
        """Per interval, sub-step r of the particles with at least r jumps in it."""
        q, dt = self.q, self.dt
        x, v = self.start(it)
        acc, path = torch.zeros(self.P, dtype=_F, device=self.dev), []
        for k in range(self.c["N"]):
            zx, zv, _, n = self.step_draws(it, k)
            x, v = x.clone(), v.clone()
            idx, a0, zx, zv = self.m, torch.zeros(self.P, dtype=_F, device=self.dev), zx, zv
            subs = []
            for r in range(32):
                ni = n[idx]
                more = ni > r
                a1 = torch.ones_like(a0)
                mi = idx[more]
                if mi.numel():
                    kk = torch.as_tensor(k, device=self.dev)
                    V = _unit(_philox(mi, kk, it, 64 + r // 4, self.key)[r % 4])
                    a1[more] = a0[more] + (1 - a0[more]) * (1 - V ** (1.0 / (ni[more] - r).to(_F)))
                d = (a1 - a0) * dt
                xi, vi = x[idx], v[idx]
                u = self.control(mu[k], xi, vi)
                xn = xi + d * vi + q["b1"] * torch.sqrt(d) * zx
                vn = vi + d * (u - q["eta"] * xi) + q["b2"] * torch.sqrt(d) * zv
                if mi.numel():
                    w = _philox(mi, kk, it, r + 1, self.key)
                    S = _pair(w[2], w[3])[0]
                    vn[more] = q["gamma"] * vn[more] + S / math.sqrt(2.0 * q["beta"])
                    zx, zv = _pair(w[0], w[1])
                if keep:
                    subs.append((idx, xi, vi, xn, vn, a0, a1, more))
                acc[idx] += d * (0.5 * q["alpha"] * u * u + self.track(xn, vn, self.target(k, a1)))
                x[idx], v[idx] = xn, vn
                idx, a0 = mi, a1[more]
                if not mi.numel():
                    break
            if keep:
                path.append(subs)
        return acc.mean(), (x, v), path

    def adjoint_adapted(self, mu, path):
        q, dt = self.q, self.dt
        lx = torch.zeros(self.P, dtype=_F, device=self.dev)
        lv = torch.zeros_like(lx)
        g = torch.zeros_like(mu)
        for k in range(self.c["N"] - 1, -1, -1):
            for idx, x, v, xe, ve, a0, a1, jump in reversed(path.pop()):
                d = (a1 - a0) * dt
                gx, gv = self.track(xe, ve, self.target(k, a1), True)
                ex, ev = lx[idx] + d * gx, lv[idx] + d * gv
                ev = torch.where(jump, q["gamma"] * ev, ev)
                u, ux, uv, px, pv = self.control_d(mu[k], x, v)
                g[k] += self.project(px, pv, d / dt * (q["alpha"] * u + ev)) / self.P
                lx[idx] = ex + d * ((ux - q["eta"]) * ev + q["alpha"] * u * ux)
                lv[idx] = ev + d * (uv * ev + ex + q["alpha"] * u * uv)
        return g


def _descend(model, c):
    """The Armijo gradient iteration (c = 1e-4, halving from the first step)."""
    u, logs = (model.t["u"] if c["model"] == "open" else model.u), []
    for it in range(c["iters"]):
        J, g = model.grad(u, it)
        g2 = model.dt * float(g.square().sum())
        zeta = ZETA0[c["model"]]
        for _ in range(30):
            ut = u - zeta * g
            Jt = model.forward(ut, it, False)[0]
            if float(Jt) <= float(J) - 1e-4 * zeta * g2:
                break
            zeta *= 0.5
        u = ut
        logs.append((float(J), math.sqrt(g2), zeta, float(Jt)))
    return {"u": u, "backtracks": None,
            **{k: np.array(v) for k, v in zip(("J", "gnorm", "zeta", "J_new"), zip(*logs))}}


def exact(case, seed):
    model = (_Open if case["model"] == "open" else _Particles)(case, seed)
    if case["call"] == "optimize":
        return _descend(model, case)
    u = model.t["u"] if case["model"] == "open" else model.u
    J, g = model.grad(u, 0)
    return {"J": J, "u_grad": g * model.dt} if case["call"] == "autograd" else {"J": J, "g": g}
