"""Measured work of the library: what its users call, through its public entry points.

A case is a dict of plain values; ``prepare`` makes what a program holds before
the call, ``run`` makes the call, ``exact`` computes the same outputs in 64
bits with plain torch, ``work`` counts the bytes and operations the call cannot
do without. Kinds of case:

  accel      acceleration (and potential) of one particle set on itself
  probe      acceleration and potential at probe points from another set
  step       a leapfrog run in place: updated positions, velocities, accelerations
  rollout    a differentiable leapfrog rollout, forward and backward: the end
             state and the gradients of a loss with respect to x0, v0 and m
  diag       the conserved quantities of a state
  diffusion  one explicit step of the 3-D diffusion equation
"""

import math

import numpy as np
import torch

import paper_2411_18889_amd as nb
from paper_2411_18889_amd import api
from nbody_inputs.configs import perturb_state, random_unit_vectors
from nbody_inputs.plummer import plummer_sphere, plummer_with_subcluster

GRID = dict(dx=0.5, dy=0.25, dz=1.0, dt=0.01, kappa=1.5)


def listed():
    return [
        # The smallest call: a thousand bodies once, with the potential, as an
        # interactive program or a unit of a larger scheme asks for it.
        dict(name="accel-tilec-1000", kind="accel", n=1000, prec="mix_tilec", log2eps=-6,
             potential=True),
        # The fp64-1024 workload: ten FP64 leapfrog steps of a small cluster,
        # where launches and latency count.
        dict(name="step-f64-1024", kind="step", n=1024, prec="f64", log2eps=-6, steps=10,
             graph=False),
        # Fitting initial conditions of a few thousand bodies: a short rollout
        # and its gradient, a checkpoint every step; not a round size.
        dict(name="rollout-tilec-5003", kind="rollout", n=5003, prec="mix_tilec", log2eps=-7,
             steps=10, ckpt_every=0),
        # One checkpoint interval (20 steps) of the adjoint-16384 workload,
        # forward and backward, the walk reconstructing the states between.
        dict(name="rollout-tilec-16384", kind="rollout", n=16384, prec="mix_tilec", log2eps=-7,
             steps=20, ckpt_every=20),
        # The fp32-65536 workload, ten of its steps.
        dict(name="step-f32-65536", kind="step", n=65536, prec="f32", log2eps=-8, steps=10,
             graph=False),
        # A reference gradient in FP64 at a size that is no multiple of a block.
        dict(name="rollout-f64-20011", kind="rollout", n=20011, prec="f64", log2eps=-7, steps=2,
             ckpt_every=1),
        # The subcluster-262144 workload's force evaluation with compensated sums.
        dict(name="accel-kahan-262144", kind="accel", n=262144, prec="mix_kahan", log2eps=-9,
             potential=False, subcluster=True),
        # Field and potential of a large cluster at many probe points.
        dict(name="probe-acc64-16001", kind="probe", ni=16001, nj=100003, prec="mix_acc64",
             log2eps=-9),
        # The scale-2^20 workload: one step of the rollout, forward and backward.
        dict(name="rollout-tilec-2^20", kind="rollout", n=1 << 20, prec="mix_tilec", log2eps=-10,
             steps=1, ckpt_every=0),
        # Energy and momentum of a running simulation, as a monitor asks every
        # few steps.
        dict(name="diag-tilec-16384", kind="diag", n=16384, prec="mix_tilec", log2eps=-7),
        # The paper's diffusion demo at its best-performing size.
        dict(name="diffusion-512", kind="diffusion", nx=512, ny=512, nz=512),
        # A grid whose sides are not round, as a simulation box comes.
        dict(name="diffusion-150x175x201", kind="diffusion", nx=150, ny=175, nz=201),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


PAIRS_MAX = 1.0e11  # pair interactions of a drawn case (the largest listed: 4.4e12)


def draw(rng):
    kind = rng.choice(["accel", "probe", "step", "rollout", "diag", "diffusion", "diffusion"])
    if kind == "diffusion":
        while True:
            s = [_log_int(rng, 16, 700) for _ in range(3)]
            if rng.random() < 0.5:  # sides of whole vectors are as common as odd ones
                s[2] = (s[2] + 3) // 4 * 4
            if s[0] * s[1] * s[2] <= 512 ** 3:
                return dict(kind=kind, nx=s[0], ny=s[1], nz=s[2])
    prec = rng.choice(["mix_tilec", "mix_tilec", "f32", "f64", "mix_acc32", "mix_kahan", "mix_acc64"])
    log2eps = rng.randint(-10, -6)
    if kind == "probe":
        ni, nj = _log_int(rng, 100, 100000), _log_int(rng, 1000, 300000)
        return dict(kind=kind, ni=ni, nj=nj, prec=prec, log2eps=log2eps)
    if kind == "accel":
        return dict(kind=kind, n=_log_int(rng, 500, 300000), prec=prec, log2eps=log2eps,
                    potential=rng.random() < 0.5, subcluster=rng.random() < 0.3)
    if kind == "diag":
        return dict(kind=kind, n=_log_int(rng, 500, 200000), prec=prec, log2eps=log2eps)
    n = _log_int(rng, 500, 100000)
    steps = rng.randint(1, 12)
    while (steps + 1) * (3 if kind == "rollout" else 1) * float(n) * n > PAIRS_MAX and steps > 1:
        steps -= 1
    if kind == "step":
        return dict(kind=kind, n=n, prec=prec, log2eps=log2eps, steps=steps,
                    graph=rng.random() < 0.3)
    return dict(kind=kind, n=n, prec=prec, log2eps=log2eps, steps=steps,
                ckpt_every=rng.choice([0, 1, 4, 20]))


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _cluster(case, n, seed):
    """(x, v, m) of a seeded Plummer sphere (with an offset subcluster where
    the case asks for one); masses equal, or within 0.5 .. 1.5 of the mean
    where n is not a power of two."""
    if case.get("subcluster"):
        x, v, m = plummer_with_subcluster(n, 2 * seed + 3, 2 * seed + 4)
    else:
        x, v, m = plummer_sphere(n, seed)
    if n & (n - 1):
        m = m * np.random.default_rng(seed).uniform(0.5, 1.5, size=n)
    return x, v, m


def _dev(a, dtype):
    return torch.tensor(a, dtype=dtype, device="cuda")


def _grid(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.rand((case["nx"], case["ny"], case["nz"]), dtype=torch.float32, device="cuda",
                      generator=g)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "diffusion":
        f = _grid(case, seed)
        return dict(case=case, f=f, out=torch.empty_like(f))
    prec = case["prec"]
    pdt, mdt = nb.pos_dtype(prec), nb.mass_dtype(prec)
    if kind == "probe":
        x, _, m = _cluster(case, case["nj"], seed)
        # probe points: positions drawn as the cluster's, moved a little
        xi, _, _ = plummer_sphere(case["ni"], seed + 77)
        xi = perturb_state(xi, xi, seed, 1e-2)[0]
        return dict(case=case, xi=_dev(xi, pdt), xj=_dev(x, pdt), m=_dev(m, mdt))
    n = case["n"]
    x, v, m = _cluster(case, n, seed)
    s = dict(case=case, x=_dev(x, pdt), v=_dev(v, pdt), m=_dev(m, mdt))
    if kind == "step":
        s["acc"] = torch.empty_like(s["x"])
        if case["graph"]:  # the cached graph needs the same workspace on every call
            s["ws"] = torch.empty(api.workspace_size(1, n, prec), dtype=torch.uint8, device="cuda")
    if kind == "rollout":
        s["x"].requires_grad_()
        s["v"].requires_grad_()
        s["m"].requires_grad_()
        s["gx"] = _dev(random_unit_vectors((3, n), seed + 1), pdt)
        s["gv"] = _dev(random_unit_vectors((3, n), seed + 2), pdt)
    return s


# ---------------------------------------------------------------------------
# The calls
# ---------------------------------------------------------------------------

def _eps_dt(case):
    eps = 2.0 ** case["log2eps"]
    return eps, 0.5 * eps


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "diffusion":
        return api.diffusion3d_step(state["f"], out=state["out"], **GRID)
    eps, dt = _eps_dt(case)
    prec = case["prec"]
    if kind == "accel":
        return nb.accel(state["x"], state["m"], eps, prec=prec, potential=case["potential"])
    if kind == "probe":
        return nb.accel(state["xi"], state["m"], eps, prec=prec, xj=state["xj"], potential=True)
    if kind == "step":
        nb.step(state["x"], state["v"], state["m"], state["acc"], eps, dt, case["steps"], prec=prec,
                graph=case["graph"], workspace=state.get("ws"))
        return state["x"], state["v"], state["acc"]
    if kind == "diag":
        return nb.diag(state["x"], state["v"], state["m"], eps, prec=prec)
    ins = (state["x"], state["v"], state["m"])
    xs, vs = nb.rollout(*ins, eps, dt, case["steps"], ckpt_every=case["ckpt_every"] or "auto",
                        prec=prec)
    g = torch.autograd.grad((xs, vs), ins, (state["gx"], state["gv"]))
    return xs.detach(), vs.detach(), g[0], g[1], g[2]


# ---------------------------------------------------------------------------
# The same in 64 bits
# ---------------------------------------------------------------------------

def _chunks(ni, nj):
    c = max(1, (1 << 26) // nj)
    return [slice(k, min(ni, k + c)) for k in range(0, ni, c)]


def _field64(xi, xj, m, eps, same):
    """Acceleration and potential at xi from the masses m at xj."""
    a, p = torch.empty_like(xi), torch.empty_like(xi[0])
    for s in _chunks(xi.shape[1], xj.shape[1]):
        d = xj[:, None, :] - xi[:, s, None]
        r = (d.square().sum(0) + eps * eps).rsqrt()
        p[s] = -(r * m).sum(1)
        w = r * r * r * m
        for q in range(3):
            a[q, s] = (d[q] * w).sum(1)
        del d, r, w
    if same:
        p += m / eps
    return a, p


def _vjp64(x, m, lam, eps):
    """J^T lam and G^T lam at x (G the derivative of the force in the masses)."""
    jt, gt = torch.empty_like(x), torch.empty_like(m)
    for s in _chunks(x.shape[1], x.shape[1]):
        d = x[:, None, :] - x[:, s, None]
        r2 = 1.0 / (d.square().sum(0) + eps * eps)
        r3 = r2 * r2.sqrt()
        gt[s] = -(r3 * (d * lam[:, None, :]).sum(0)).sum(1)
        u = m[s, None] * lam[:, None, :] - m * lam[:, s, None]
        e = -3.0 * r2 * (d * u).sum(0)
        for q in range(3):
            jt[q, s] = (r3 * (u[q] + e * d[q])).sum(1)
        del d, r2, r3, u, e
    return jt, gt


def _leapfrog64(x, v, m, eps, dt, steps):
    h = 0.5 * dt
    a, _ = _field64(x, x, m, eps, True)
    path = [x]
    for _ in range(steps):
        v = v + h * a
        x = x + dt * v
        a, _ = _field64(x, x, m, eps, True)
        v = v + h * a
        path.append(x)
    return x, v, a, path


def _gradient64(path, m, gx, gv, eps, dt):
    h = 0.5 * dt
    lx, lv, lm = gx.clone(), gv.clone(), torch.zeros_like(m)
    for k in range(len(path) - 1, -1, -1):
        c = h if k in (0, len(path) - 1) else dt
        jt, gt = _vjp64(path[k], m, lv, eps)
        lx = lx + c * jt
        lm = lm + c * gt
        if k:
            lv = lv + dt * lx
    return lx, lv, lm


def _pairs(case):
    """Pair interactions of a pass (both ends of a pair counted)."""
    if case["kind"] == "probe":
        return float(case["ni"]) * case["nj"]
    return float(case["n"]) ** 2


def exact(case, seed):
    kind = case["kind"]
    if kind == "diffusion":
        f = _grid(case, seed).double()
        cx, cy, cz = (GRID["kappa"] * GRID["dt"] / GRID[k] ** 2 for k in ("dx", "dy", "dz"))
        out = f * (1.0 - 2.0 * (cx + cy + cz))
        for dim, c in ((0, cx), (1, cy), (2, cz)):
            n = f.shape[dim]
            k = torch.arange(n, device=f.device)
            out += c * f.index_select(dim, (k + 1).clamp(max=n - 1))
            out += c * f.index_select(dim, (k - 1).clamp(min=0))
        return out
    passes = {"step": 1 + case.get("steps", 0), "rollout": 4 * (1 + case.get("steps", 0))}
    if _pairs(case) * passes.get(kind, 1) > 1.2e12:
        return None  # minutes in 64 bits
    eps, dt = _eps_dt(case)
    s = prepare(case, seed)
    m = s["m"].detach().double()
    with torch.no_grad():
        if kind == "probe":
            return _field64(s["xi"].double(), s["xj"].double(), m, eps, False)
        x, v = s["x"].detach().double(), s["v"].detach().double()
        if kind == "accel":
            a, p = _field64(x, x, m, eps, True)
            return (a, p) if case["potential"] else a
        if kind == "step":
            return _leapfrog64(x, v, m, eps, dt, case["steps"])[:3]
        if kind == "diag":
            _, p = _field64(x, x, m, eps, True)
            ke, pe = 0.5 * (m * v.square().sum(0)).sum(), 0.5 * (m * p).sum()
            mom = (m * v).sum(1)
            ang = (m * torch.cross(x, v, dim=0)).sum(1)
            com = (m * x).sum(1) / m.sum()
            return torch.cat([torch.stack([ke, pe, ke + pe]), mom, ang, com, m.sum()[None]])
        xs, vs, _, path = _leapfrog64(x, v, m, eps, dt, case["steps"])
        return (xs, vs) + _gradient64(path, m, s["gx"].double(), s["gv"].double(), eps, dt)


# ---------------------------------------------------------------------------
# Bytes and operations that a pass cannot do without
# ---------------------------------------------------------------------------

def work(case):
    """Operations: a fused multiply-add counts 2, a reciprocal square root 2.
    A pair of a set with itself needs one evaluation for both of its ends:
    27 for the force, 31 with the potential, 58 for the adjoint pass (no force
    sums), 13 for the potential energy; a probe and a source 22. Bytes: each
    input read once, each output written once."""
    kind = case["kind"]
    if kind == "diffusion":
        pts = case["nx"] * case["ny"] * case["nz"]
        return {"bytes": 8 * pts, "flops": 13 * pts}
    ps = 4 if case["prec"] == "f32" else 8
    ms = 8 if case["prec"] == "f64" else 4
    if kind == "probe":
        ni, nj = case["ni"], case["nj"]
        return {"bytes": ni * 7 * ps + nj * (3 * ps + ms), "flops": 22 * ni * nj}
    n = case["n"]
    pairs = n * (n - 1) // 2
    if kind == "accel":
        pot = case["potential"]
        return {"bytes": n * ((7 if pot else 6) * ps + ms), "flops": (31 if pot else 27) * pairs}
    if kind == "step":
        return {"bytes": n * (15 * ps + ms), "flops": (case["steps"] + 1) * 27 * pairs}
    if kind == "diag":
        return {"bytes": n * (6 * ps + ms), "flops": 13 * pairs}
    # forward: the end state; backward: cotangents in, gradients out
    return {"bytes": n * (24 * ps + 2 * ms), "flops": (case["steps"] + 1) * (27 + 58) * pairs}
