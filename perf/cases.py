"""Performance cases: the calls a program makes of this library, over the sizes it serves.

Every case is one pass through the public entry points (paper_2605_02744_amd) on
seeded synthetic star clusters in Henon units (G = M = 1): Plummer spheres, or a
two-component model (dense core, wide halo, unequal masses).  The listed cases
are the workloads the library is used for, at their own sizes and at ragged
ones; draw() spreads the same kinds of calls over their whole size ranges.

A case's "kind" is the call:
  accel      nbody_accel, one force evaluation
  kdk        nbody_step, `steps` kick-drift-kick steps of a run under way
  ensemble   nbody_step_batched, `steps` steps of independent clusters
  vjp        nbody_accel_vjp, the force's vector-Jacobian product
  grad       trajectory() and its gradient with respect to x0, v0 and m
  jerk       nbody_accel_jerk, acceleration + jerk
  hermite4   nbody_step_hermite, `steps` steps of a run under way
  hermite6   nbody_step_hermite6, `steps` steps of a run under way
  energy     nbody_energy and nbody_potential, the diagnostics of a snapshot
"""
import math

import numpy as np
import torch

import paper_2605_02744_amd as nb

HENON_A = 3.0 * math.pi / 16.0  # Plummer scale radius of a cluster with G = M = 1, E = -1/4

# flops of one ordered interaction, by the formula of each evaluation
FLOPS = {"accel": 20, "kdk": 20, "ensemble": 20, "vjp": 48, "jerk": 42, "hermite4": 42, "hermite6": 80, "energy": 12}


def listed():
    return [
        # one force evaluation of a small cluster, as an outer loop or a test calls it: launches and latency
        dict(name="accel_1000_fp32c", kind="accel", n=1000, eps=0.01, precision="fp32c", model="plummer"),
        # a small cluster integrated in double precision, ten steps a call
        dict(name="kdk_1024_fp64", kind="kdk", n=1024, eps=0.01, dt=1.0 / 128, steps=10, precision="fp64",
             model="plummer"),
        # a mid-size cluster of unequal masses at a ragged size, the double-precision reference force
        dict(name="accel_30011_fp64", kind="accel", n=30011, eps=0.005, precision="fp64", model="twocomp"),
        # the 65536-body cluster run in the fast precision, a few steps between outputs
        dict(name="kdk_65536_fp32c", kind="kdk", n=65536, eps=0.005, dt=1.0 / 256, steps=4, precision="fp32c",
             model="plummer"),
        # the large single evaluation: two-component model of 2^20 particles
        dict(name="accel_1m_fp32c", kind="accel", n=1 << 20, eps=0.001, precision="fp32c", model="twocomp"),
        # 512 independent clusters of 64 to 4096 particles stepped together
        dict(name="ensemble_512_fp32c", kind="ensemble", ncl=512, nmin=64, nmax=4096, dt=1.0 / 512, steps=5,
             precision="fp32c"),
        # a smaller ensemble in double precision
        dict(name="ensemble_100_fp64", kind="ensemble", ncl=100, nmin=64, nmax=2000, dt=1.0 / 512, steps=10,
             precision="fp64"),
        # forward and backward: the gradient of a 16384-body trajectory, checkpoints every 20 steps
        dict(name="grad_16384_fp32c", kind="grad", n=16384, eps=0.01, dt=1.0 / 256, steps=60, every=20,
             precision="fp32c"),
        # backward alone, in double precision at a ragged size: one adjoint step of a user's own integrator
        dict(name="vjp_9973_fp64", kind="vjp", n=9973, eps=0.01, precision="fp64", model="plummer"),
        # a fourth-order Hermite run of a small collisional system in double precision
        dict(name="hermite4_5000_fp64", kind="hermite4", n=5000, eps=0.002, dt=1.0 / 512, steps=5, precision="fp64",
             model="plummer"),
        # one sixth-order Hermite step of a large run with nearly no softening
        dict(name="hermite6_204800_fp32c", kind="hermite6", n=204800, eps=1e-7, dt=1.0 / 1024, steps=1,
             precision="fp32c", model="plummer"),
        # the diagnostics a run writes with each snapshot: energies, momenta and every particle's potential
        dict(name="energy_65536_fp64", kind="energy", n=65536, eps=0.005, precision="fp64", model="plummer"),
    ]


def _size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["accel", "accel", "kdk", "kdk", "ensemble", "vjp", "grad", "jerk", "hermite4", "hermite6",
                       "energy"])
    precision = rng.choice(["fp32c", "fp32c", "fp32c", "fp64", "fp64", "fp32"])
    c = dict(kind=kind, precision=precision)
    if kind == "ensemble":
        nmax = _size(rng, 100, 4096)
        c.update(ncl=_size(rng, 8, 512), nmin=max(1, nmax // rng.choice([1, 4, 64])), nmax=nmax, dt=1.0 / 512,
                 steps=rng.randint(1, 10))
        return c
    if kind == "grad":
        c.update(n=_size(rng, 300, 16384), eps=0.01, dt=1.0 / 256, steps=rng.randint(3, 40), every=rng.randint(5, 20))
        return c
    top = {"accel": 500000, "kdk": 65536, "vjp": 150000, "jerk": 150000, "hermite4": 65536, "hermite6": 65536,
           "energy": 200000}[kind]
    n = _size(rng, 100, top)
    c.update(n=n, eps=rng.choice([0.01, 0.005, 0.002]), model=rng.choice(["plummer", "twocomp"]))
    if kind in ("kdk", "hermite4", "hermite6"):
        c.update(dt=1.0 / 512, steps=rng.randint(1, 10 if n < 20000 else 4))
    if kind == "energy":
        c["precision"] = "fp64"
    return c


# ------------------------------------------------------------------ inputs
def _plummer_radii(rng, n, a):
    x = rng.uniform(1e-6, 0.999, n)
    return a / np.sqrt(x ** (-2.0 / 3.0) - 1.0)


def _isotropic(rng, mag):
    z = rng.uniform(-1.0, 1.0, mag.size)
    phi = rng.uniform(0.0, 2.0 * math.pi, mag.size)
    rho = np.sqrt(1.0 - z * z)
    return np.stack([rho * np.cos(phi), rho * np.sin(phi), z]) * mag


def _speed_fractions(rng, n):
    """v / v_escape drawn from q^2 (1 - q^2)^(7/2) by rejection."""
    q = np.empty(0)
    while q.size < n:
        u = rng.random((2, 4 * n + 64))
        q = np.concatenate([q, u[0][0.1 * u[1] < u[0] ** 2 * (1.0 - u[0] ** 2) ** 3.5]])
    return q[:n]


def _cluster(rng, n, model):
    """(x, v, m) of one cluster of unit mass."""
    if model == "twocomp":
        nc = int(round(0.9 * n))
        r = np.concatenate([_plummer_radii(rng, nc, 0.5), _plummer_radii(rng, n - nc, 3.0)])
        m = np.exp(rng.uniform(math.log(0.1), math.log(10.0), n))
        m /= m.sum()
    else:
        r = _plummer_radii(rng, n, HENON_A)
        m = np.full(n, 1.0 / n)
    x = _isotropic(rng, r)
    v = _isotropic(rng, _speed_fractions(rng, n) * math.sqrt(2.0) * (r * r + HENON_A * HENON_A) ** -0.25)
    return x, v, m


def _inputs(case, seed):
    """The case's host arrays, from the seed alone."""
    rng = np.random.default_rng(seed)
    if case["kind"] == "ensemble":
        # the layout belongs to the case (a program steps the same clusters again and again), the stars to the seed
        sizes = np.random.default_rng(case["ncl"]).integers(case["nmin"], case["nmax"] + 1, size=case["ncl"])
        off = np.zeros(case["ncl"] + 1, dtype=np.int64)
        np.cumsum(sizes, out=off[1:])
        x, v, _ = _cluster(rng, int(off[-1]), "plummer")
        return dict(x=x, v=v, m=np.repeat(1.0 / sizes, sizes), off=off, eps=0.04 / np.sqrt(sizes))
    x, v, m = _cluster(rng, case["n"], case.get("model", "plummer"))
    h = dict(x=x, v=v, m=m)
    if case["kind"] == "vjp":
        h["w"] = rng.standard_normal(x.shape)
    if case["kind"] == "grad":  # the final state the trajectory is fitted to
        h["target"] = x + 1e-2 * rng.standard_normal(x.shape)
    return h


def prepare(case, seed):
    h = _inputs(case, seed)
    s = {k: torch.from_numpy(a).cuda() if k not in ("off", "eps") else a for k, a in h.items()}
    s["case"] = case
    x, v, m, kind, prec = s["x"], s["v"], s["m"], case["kind"], case["precision"]
    # a run under way holds the evaluation at its current state
    if kind in ("kdk", "ensemble", "hermite4", "hermite6"):
        s["a"] = torch.empty_like(x)
    if kind == "kdk":
        nb.nbody_step(x, v, s["a"], m, case["dt"], 0, eps=case["eps"], precision=prec)
    elif kind == "ensemble":
        nb.nbody_step_batched(s["off"], s["eps"], x, v, s["a"], m, case["dt"], 0, precision=prec)
    elif kind == "hermite4":
        s["jk"] = torch.empty_like(x)
        nb.nbody_step_hermite(x, v, s["a"], s["jk"], m, case["dt"], 0, eps=case["eps"], precision=prec)
    elif kind == "hermite6":
        s["jk"], s["sn"], s["cr"] = (torch.empty_like(x) for _ in range(3))
        nb.nbody_step_hermite6(x, v, s["a"], s["jk"], s["sn"], s["cr"], m, case["dt"], 0, eps=case["eps"],
                               precision=prec)
    elif kind == "grad":
        for t in (x, v, m):
            t.requires_grad_(True)
    return s


# -------------------------------------------------------------------- pass
def run(s):
    c = s["case"]
    x, v, m, kind, prec = s["x"], s["v"], s["m"], c["kind"], c["precision"]
    if kind == "accel":
        return nb.nbody_accel(x, m, eps=c["eps"], precision=prec)
    if kind == "kdk":
        return nb.nbody_step(x, v, s["a"], m, c["dt"], c["steps"], eps=c["eps"], precision=prec, acc_valid=True)
    if kind == "ensemble":
        return nb.nbody_step_batched(s["off"], s["eps"], x, v, s["a"], m, c["dt"], c["steps"], precision=prec,
                                     acc_valid=True)
    if kind == "vjp":
        return nb.nbody_accel_vjp(x, m, s["w"], eps=c["eps"], precision=prec)
    if kind == "jerk":
        return nb.nbody_accel_jerk(x, v, m, eps=c["eps"], precision=prec)
    if kind == "hermite4":
        return nb.nbody_step_hermite(x, v, s["a"], s["jk"], m, c["dt"], c["steps"], eps=c["eps"], precision=prec,
                                     acc_valid=True)
    if kind == "hermite6":
        nb.nbody_step_hermite6(x, v, s["a"], s["jk"], s["sn"], s["cr"], m, c["dt"], c["steps"], eps=c["eps"],
                               precision=prec, acc_valid=True)
        return x, v, s["a"], s["jk"], s["sn"]
    if kind == "energy":
        return nb.nbody_energy(x, v, m, eps=c["eps"]), nb.nbody_potential(x, m, eps=c["eps"])
    if kind == "grad":
        xT, vT = nb.trajectory(x, v, m, c["dt"], c["steps"], every=c["every"], eps=c["eps"], precision=prec)
        loss = 0.5 * ((xT - s["target"]) ** 2).sum()
        return (xT.detach(), vT.detach()) + torch.autograd.grad(loss, (x, v, m))
    raise ValueError(kind)


def _pairs(case):
    """Ordered interactions of one evaluation (an ensemble's sizes taken at their mean)."""
    if case["kind"] == "ensemble":
        lo, hi = case["nmin"], case["nmax"]
        return case["ncl"] * ((lo * lo + lo * hi + hi * hi) / 3.0 - (lo + hi) / 2.0)
    return float(case["n"]) * (case["n"] - 1)


def work(case):
    kind, pairs = case["kind"], _pairs(case)
    n = case["ncl"] * (case["nmin"] + case["nmax"]) / 2.0 if kind == "ensemble" else case["n"]
    # doubles in and out per particle
    words = {"accel": 4 + 3, "kdk": 10 + 9, "ensemble": 10 + 9, "vjp": 7 + 4, "grad": 10 + 13, "jerk": 7 + 6,
             "hermite4": 13 + 12, "hermite6": 19 + 18, "energy": 7 + 1}[kind]
    if kind == "grad":  # a force a step forward, a force and a VJP a step backward
        flops = case["steps"] * (20 + 20 + 48) * pairs
    else:
        flops = case.get("steps", 1) * FLOPS[kind] * pairs
    return {"bytes": 8.0 * words * n, "flops": flops}


# ------------------------------------------------- the same in plain 64 bits
def _blocks(n):
    step = max(1, min(n, (1 << 25) // n))
    return [(i, min(n, i + step)) for i in range(0, n, step)]


def _pair_block(x, eps, i, j):
    """d = x_j - x_i, 1/s and s^-3/2 (zero for the own pair) of rows i..j against all."""
    d = [x[c][None, :] - x[c][i:j, None] for c in range(3)]
    si = 1.0 / (d[0] * d[0] + d[1] * d[1] + d[2] * d[2] + eps * eps)
    w = si * torch.sqrt(si)
    r = torch.arange(i, j, device=x.device)
    w[r - i, r] = 0.0
    return d, si, w


def _rows(x, out, f):
    for i, j in _blocks(x.shape[1]):
        f(out, i, j)
    return out


def _accel64(x, m, eps):
    def f(a, i, j):
        d, _, w = _pair_block(x, eps, i, j)
        w = w * m[None, :]
        for c in range(3):
            a[c, i:j] = (w * d[c]).sum(1)
    return _rows(x, torch.empty_like(x), f)


def _deriv64(x, v, acc, m, eps):
    """(a, jerk, snap) along paths of constant acceleration acc (snap None without acc)."""
    def f(out, i, j):
        d, si, w = _pair_block(x, eps, i, j)
        w = w * m[None, :]
        u = [v[c][None, :] - v[c][i:j, None] for c in range(3)]
        al = (d[0] * u[0] + d[1] * u[1] + d[2] * u[2]) * si
        if acc is not None:
            b = [acc[c][None, :] - acc[c][i:j, None] for c in range(3)]
            be = sum(u[c] * u[c] + d[c] * b[c] for c in range(3)) * si + al * al
        for c in range(3):
            p0 = w * d[c]
            p1 = w * u[c] - 3.0 * al * p0
            out[0][c, i:j] = p0.sum(1)
            out[1][c, i:j] = p1.sum(1)
            if acc is not None:
                out[2][c, i:j] = (w * b[c] - 6.0 * al * p1 - 3.0 * be * p0).sum(1)
    return _rows(x, [torch.empty_like(x) for _ in range(2 if acc is None else 3)], f)


def _vjp64(x, m, w, eps):
    def f(out, i, j):
        d, si, q = _pair_block(x, eps, i, j)
        dw = d[0] * w[0][None, :] + d[1] * w[1][None, :] + d[2] * w[2][None, :]
        out[1][i:j] = -(q * dw).sum(1)
        u = [m[i:j, None] * w[c][None, :] - m[None, :] * w[c][i:j, None] for c in range(3)]
        du = 3.0 * si * (d[0] * u[0] + d[1] * u[1] + d[2] * u[2])
        for c in range(3):
            out[0][c, i:j] = (q * (u[c] - du * d[c])).sum(1)
    return _rows(x, [torch.empty_like(x), torch.empty_like(m)], f)


def _kdk64(x, v, m, eps, dt, steps, keep=None):
    x, v, a = x.clone(), v.clone(), _accel64(x, m, eps)
    for _ in range(steps):
        v = v + 0.5 * dt * a
        x = x + dt * v
        a = _accel64(x, m, eps)
        v = v + 0.5 * dt * a
        if keep is not None:
            keep.append(x)
    return x, v, a


def exact(case, seed):
    kind, steps = case["kind"], case.get("steps", 1)
    evals = {"grad": 7 * steps, "hermite4": 2 * steps + 2, "hermite6": 4 * steps + 6, "vjp": 3, "jerk": 2}.get(kind, steps + 1)
    if evals * _pairs(case) > 1.5e11:
        return None
    h = {k: torch.from_numpy(a).cuda() if k not in ("off", "eps") else a for k, a in _inputs(case, seed).items()}
    x, v, m, eps, dt = h["x"], h["v"], h["m"], case.get("eps"), case.get("dt")
    if kind == "accel":
        return _accel64(x, m, eps)
    if kind == "kdk":
        return _kdk64(x, v, m, eps, dt, steps)
    if kind == "ensemble":
        got = [_kdk64(x[:, p:q], v[:, p:q], m[p:q], float(e), dt, steps)
               for p, q, e in zip(h["off"][:-1].tolist(), h["off"][1:].tolist(), h["eps"])]
        return tuple(torch.cat([g[k] for g in got], 1) for k in range(3))
    if kind == "vjp":
        return tuple(_vjp64(x, m, h["w"], eps))
    if kind == "jerk":
        return tuple(_deriv64(x, v, None, m, eps))
    if kind == "hermite4":
        a, jk = _deriv64(x, v, None, m, eps)
        for _ in range(steps):
            xp = x + v * dt + a * (dt ** 2 / 2) + jk * (dt ** 3 / 6)
            vp = v + a * dt + jk * (dt ** 2 / 2)
            a1, j1 = _deriv64(xp, vp, None, m, eps)
            v1 = v + (a + a1) * (dt / 2) + (jk - j1) * (dt ** 2 / 12)
            x = x + (v + v1) * (dt / 2) + (a - a1) * (dt ** 2 / 12)
            v, a, jk = v1, a1, j1
        return x, v, a, jk
    if kind == "hermite6":
        a = _accel64(x, m, eps)
        a, jk, sn = _deriv64(x, v, a, m, eps)
        cr = torch.zeros_like(a)
        for _ in range(steps):
            xp = x + v * dt + a * (dt ** 2 / 2) + jk * (dt ** 3 / 6) + sn * (dt ** 4 / 24) + cr * (dt ** 5 / 120)
            vp = v + a * dt + jk * (dt ** 2 / 2) + sn * (dt ** 3 / 6) + cr * (dt ** 4 / 24)
            ap = a + jk * dt + sn * (dt ** 2 / 2) + cr * (dt ** 3 / 6)
            a1, j1, s1 = _deriv64(xp, vp, ap, m, eps)
            v1 = v + (a + a1) * (dt / 2) - (j1 - jk) * (dt ** 2 / 10) + (sn + s1) * (dt ** 3 / 120)
            x = x + (v + v1) * (dt / 2) - (a1 - a) * (dt ** 2 / 10) + (jk + j1) * (dt ** 3 / 120)
            A = (a1 - a - jk * dt - sn * (dt ** 2 / 2)) / dt ** 3
            cr = 60.0 * A - 36.0 * (j1 - jk - sn * dt) / dt ** 2 + 9.0 * (s1 - sn) / dt
            v, a, jk, sn = v1, a1, j1, s1
        return x, v, a, jk, sn
    if kind == "energy":
        phi = torch.empty_like(m)
        for i, j in _blocks(m.shape[0]):
            _, si, w = _pair_block(x, eps, i, j)
            phi[i:j] = -((w / si) * m[None, :]).sum(1)
        K, W = 0.5 * (m * (v * v).sum(0)).sum(), 0.5 * (m * phi).sum()
        L = torch.linalg.cross(x, v, dim=0)
        return torch.cat([torch.stack([K, W, K + W]), (m * v).sum(1), (m * L).sum(1)]), phi
    if kind == "grad":
        traj = [x]
        xT, vT, _ = _kdk64(x, v, m, eps, dt, steps, traj)
        lx, lv, gm = xT - h["target"], torch.zeros_like(x), torch.zeros_like(m)
        for k in range(steps, -1, -1):  # the kicks at position k: half ones at the ends
            gx, g = _vjp64(traj[k], m, lv * (0.5 * dt if k in (0, steps) else dt), eps)
            lx, gm = lx + gx, gm + g
            if k:
                lv = lv + dt * lx
        return xT, vT, lx, lv, gm
    return None
