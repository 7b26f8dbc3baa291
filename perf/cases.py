"""What a user of this framework has it do, as cases that can be timed and compared.

Five kinds of work, each through the public entry points of the package:

  step        time steps of coupled droplets (Solver.step), then the fields and
              the nodes that a program reads after them; 2D and 3D, one droplet
              or a batch of uneven boxes, every storage format, one or two
              viscosities
  monitor     the FP64 diagnostics and the contact radius of a droplet, which a
              program asks for every hundred steps or so of a run
  checkpoint  populations written to and read back from a handle (restart files)
  mlp         the warm-start network's forward pass
  train       optimiser steps of that network

The sizes are those of this repository's workloads and benchmark, or the odd
sizes between them.
"""
import math

import numpy as np
import torch

from paper_2503_20605_amd import MLP, Solver, make_params

DEV = "cuda"
STORE = {"f32": 0, "f16": 1, "bf16": 2}


def listed():
    return [
        # a short look at a small droplet: few cells, few steps, latency counts
        dict(name="small_2d", kind="step", dim=2, nx=128, ny=64, nz=1, R=20.0, nodes=128, tau=1.0, sigma=0.01,
             theta=60.0, xi=2.0, lam=1.0, respace=0.05, storage="f32", steps=20, n=1),
        # a point of the parameter sweep: one droplet on a box that fits the caches
        dict(name="sweep_2d", kind="step", dim=2, nx=1024, ny=512, nz=1, R=120.0, nodes=1024, tau=0.6, sigma=0.005,
             theta=60.0, xi=3.0, lam=1.0, respace=0.0, storage="f32", steps=130, n=1),
        # the batch that makes training data and runs to equilibrium: 256 uneven boxes
        dict(name="batch_2d_f16", kind="step", dim=2, nx=512, ny=256, nz=1, R=100.0, nodes=785, tau=1.0, sigma=0.006,
             theta=90.0, xi=2.0, lam=1.0, respace=0.05, storage="f16", steps=260, n=256),
        # the equilibrium shape study: a small 3D box under a fine mesh
        dict(name="statics_3d", kind="step", dim=3, nx=80, ny=80, nz=60, R=20.0, nodes=45, tau=1.0, sigma=0.01,
             theta=90.0, xi=2.0, lam=1.0, respace=0.0, storage="f32", steps=130, n=1),
        # the benchmark's droplet on a wall, far above the caches
        dict(name="wall_3d", kind="step", dim=3, nx=256, ny=256, nz=128, R=40.0, nodes=45, tau=0.8, sigma=0.005,
             theta=90.0, xi=4.0, lam=1.0, respace=0.0, storage="f32", steps=130, n=1),
        # the same in half-precision storage
        dict(name="wall_3d_f16", kind="step", dim=3, nx=256, ny=256, nz=128, R=40.0, nodes=45, tau=0.8, sigma=0.005,
             theta=90.0, xi=4.0, lam=1.0, respace=0.0, storage="f16", steps=130, n=1),
        # a spreading run: two viscosities, rows that are no multiple of a wavefront
        dict(name="spreading_3d", kind="step", dim=3, nx=240, ny=240, nz=130, R=60.0, nodes=64, tau=0.8, sigma=0.005,
             theta=60.0, xi=2.0, lam=10.0, respace=0.0, storage="f32", steps=66, n=1),
        # the numbers that a run prints
        dict(name="monitor_3d", kind="monitor", dim=3, nx=256, ny=256, nz=128, R=40.0, nodes=45, tau=0.8, sigma=0.005,
             theta=90.0, xi=4.0, lam=1.0, respace=0.0, storage="f32", steps=2, n=1),
        # a restart file out and in
        dict(name="checkpoint_3d", kind="checkpoint", dim=3, nx=240, ny=240, nz=130, storage="f16"),
        # initial states predicted for a few droplets, and for a whole batch
        dict(name="mlp_small", kind="mlp", batch=64, hidden=256, layers=3, out=1280),
        dict(name="mlp_batch", kind="mlp", batch=4096, hidden=256, layers=3, out=1280),
        # full-batch optimiser steps
        dict(name="mlp_train", kind="train", batch=4096, hidden=256, layers=3, out=1280, steps=4),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "monitor", "checkpoint", "mlp", "mlp", "train"])
    if kind in ("mlp", "train"):
        c = dict(kind=kind, batch=_log(rng, 1 if kind == "mlp" else 200, 4096), hidden=rng.choice([64, 100, 128, 200, 256]),
                 layers=rng.choice([2, 3]), out=_log(rng, 100, 1280))
        if kind == "train":
            c["steps"] = rng.randint(1, 4)
        return c
    storage = rng.choice(["f32", "f32", "f16", "bf16"])
    dim = rng.choice([2, 3])
    if kind == "checkpoint":
        nx, ny = _log(rng, 40, 240), _log(rng, 40, 240)
        return dict(kind=kind, dim=dim, nx=nx, ny=ny, nz=_log(rng, 20, 130) if dim == 3 else 1, storage=storage)
    c = dict(kind=kind, dim=dim, xi=2.0, sigma=round(rng.uniform(0.002, 0.01), 4), tau=round(rng.uniform(0.6, 1.5), 3),
             theta=round(rng.uniform(60.0, 120.0), 1), storage=storage, n=1)
    if dim == 2:
        c["n"] = rng.choice([1, 1, _log(rng, 2, 200)]) if kind == "step" else 1
        R = math.exp(rng.uniform(math.log(16.0), math.log(80.0)))
        c.update(nx=int(3.2 * R) + rng.randint(32, 300), ny=int(2.0 * R) + rng.randint(10, 160), nz=1, R=round(R, 2),
                 nodes=int(2 * math.pi * R / 0.8), lam=rng.choice([1.0, 1.0, 4.0]), respace=0.05)
        c["steps"] = rng.randint(2, 150)
    else:
        R = math.exp(rng.uniform(math.log(10.0), math.log(45.0)))
        c.update(nx=int(3.0 * R) + rng.randint(8, 100), ny=int(3.0 * R) + rng.randint(8, 100),
                 nz=int(1.8 * R) + rng.randint(8, 40), R=round(R, 2), nodes=max(10, int(1.1 * R)),
                 lam=rng.choice([1.0, 1.0, 5.0]), respace=0.0)
        c["steps"] = rng.randint(2, 100)
    if kind == "monitor":
        c["steps"] = 2
    return c


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _cap_outline(R, deg, base, n, xc):
    """Closed outline of a circular cap on the line y = base, uniform in arc length."""
    th = math.radians(deg)
    arc, flat = 2 * th * R, 2 * R * math.sin(th)
    s = np.arange(n) * ((arc + flat) / n)
    a = 0.5 * math.pi - th + s / R
    on = s < arc
    x = np.where(on, xc + R * np.cos(a), xc - R * math.sin(th) + (s - arc))
    y = np.where(on, base - R * math.cos(th) + R * np.sin(a), base)
    return np.stack([x, y], axis=1)


_spheres = {}


def _sphere(nu):
    """Geodesic sphere: every icosahedron face split into nu^2 triangles."""
    if nu in _spheres:
        return _spheres[nu]
    p = (1 + math.sqrt(5)) / 2
    B = np.array([[-1, p, 0], [1, p, 0], [-1, -p, 0], [1, -p, 0], [0, -1, p], [0, 1, p], [0, -1, -p], [0, 1, -p],
                  [p, 0, -1], [p, 0, 1], [-p, 0, -1], [-p, 0, 1]])
    d = np.linalg.norm(B[:, None] - B[None], axis=2)
    near = np.isclose(d, 2.0)
    faces = [(a, b, c) for a in range(12) for b in range(a + 1, 12) for c in range(b + 1, 12)
             if near[a, b] and near[b, c] and near[a, c]]
    i, j = np.meshgrid(np.arange(nu + 1), np.arange(nu + 1), indexing="ij")
    ok = i + j <= nu
    at = -np.ones((nu + 1, nu + 1), int)
    at[ok] = np.arange(ok.sum())
    w = np.stack([nu - i - j, i, j], -1)[ok] / nu
    up = i + j < nu
    t1 = np.stack([at[i[up], j[up]], at[i[up] + 1, j[up]], at[i[up], j[up] + 1]], 1)
    dn = i + j < nu - 1
    t2 = np.stack([at[i[dn] + 1, j[dn]], at[i[dn] + 1, j[dn] + 1], at[i[dn], j[dn] + 1]], 1)
    V = np.concatenate([w @ B[list(f)] for f in faces])
    T = np.concatenate([np.concatenate([t1, t2]) + k * ok.sum() for k in range(len(faces))])
    _, first, inv = np.unique(np.round(V, 9), axis=0, return_index=True, return_inverse=True)
    V, T = V[first], inv.reshape(-1)[T]
    V = V / np.linalg.norm(V, axis=1, keepdims=True)
    a, b, c = V[T[:, 0]], V[T[:, 1]], V[T[:, 2]]
    flip = np.einsum("ij,ij->i", np.cross(b - a, c - a), a + b + c) < 0
    T[flip] = T[flip][:, [0, 2, 1]]
    _spheres[nu] = (V, T.astype(np.int32))
    return _spheres[nu]


def _cap_mesh(R, deg, base, nu, xy):
    """Spherical cap on the plane z = base: the geodesic sphere projected onto it from an inner point."""
    U, T = _sphere(nu)
    th = math.radians(deg)
    p0 = np.array([xy[0], xy[1], base + 0.4 * R * (1 - math.cos(th))])
    m = p0 - np.array([xy[0], xy[1], base - R * math.cos(th)])
    b = U @ m
    ts = -b + np.sqrt(b * b - m @ m + R * R)
    tp = np.where(U[:, 2] < 0, (base - p0[2]) / np.where(U[:, 2] < 0, U[:, 2], -1.0), np.inf)
    V = p0 + np.minimum(ts, tp)[:, None] * U
    V[tp <= ts, 2] = base
    return V, T


def _droplets(c, seed):
    """Parameters, nodes and triangles of the case's droplets."""
    rng = np.random.default_rng(seed)
    sizes = np.random.default_rng([c["n"], c["nx"], c["ny"]])  # a batch's boxes belong to the case, their physics to the seed
    P, nodes, tris = [], [], []
    for _ in range(c["n"]):
        nx, ny, R, nn, th, tau, sg = c["nx"], c["ny"], c["R"], c["nodes"], c["theta"], c["tau"], c["sigma"]
        if c["n"] > 1:  # uneven boxes below the largest, as the batch draws have them
            while True:
                R = sizes.uniform(15.0, c["R"])
                nx, ny = (int(sizes.integers(a, max(a + 1, m // 32 + 1))) * 32 for a, m in ((4, c["nx"]), (2, c["ny"])))
                if 2.6 * R <= nx - 16 and R + 10 <= 0.8 * ny:
                    break
                nx, ny = c["nx"], c["ny"]
                if 2.6 * R <= nx - 16 and R + 10 <= 0.8 * ny:
                    break
            th, tau, sg = rng.uniform(60.0, 120.0), rng.uniform(0.6, 1.5), rng.uniform(0.002, 0.01)
            nn = int(round(2 * math.pi * R / 0.8))
        R *= 1 + rng.uniform(-0.01, 0.01)
        deg = 90 + rng.uniform(-5, 5)
        P.append(make_params(dim=c["dim"], nx=nx, ny=ny, nz=c["nz"], tau=tau, sigma=sg, theta_eq_deg=th, xi=c["xi"]))
        off = rng.uniform(-0.5, 0.5, 2)
        if c["dim"] == 2:
            nodes.append(_cap_outline(R, deg, c["xi"], nn, nx / 2 + off[0]))
            tris.append(None)
        else:
            V, T = _cap_mesh(R, deg, c["xi"], nn, (nx / 2 + off[0], ny / 2 + off[1]))
            nodes.append(V)
            tris.append(T)
    return P, nodes, tris


def _solver(c, seed):
    P, nodes, tris = _droplets(c, seed)
    s = Solver(P, nodes, tris if c["dim"] == 3 else None, storage=STORE[c["storage"]], device=DEV)
    # the lattice-kernel variant a tuned program holds for such a box
    s.set_lb_variant(4 if c["dim"] == 2 else (25 if c["nx"] % 64 == 0 else 29))
    for d in range(c["n"]):
        if c["lam"] != 1.0:
            s.set_viscosity_ratio(d, c["lam"])
        if c["respace"]:
            s.set_node_respacing(d, c["respace"])
    return s


def _fields(c, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    sh = (c["nz"], c["ny"], c["nx"])
    rho = 1 + 1e-3 * torch.randn(sh, generator=g, device=DEV)
    U = 1e-2 * torch.randn((c["dim"],) + sh, generator=g, device=DEV)
    return rho, U


def _weights(c, seed):
    rng = np.random.default_rng(seed)
    widths = [4] + [c["hidden"]] * c["layers"] + [c["out"]]
    packed = []
    for a, b in zip(widths[:-1], widths[1:]):
        packed += [rng.standard_normal((a, b)).reshape(-1) / math.sqrt(a), 0.1 * rng.standard_normal(b)]
    return widths, np.concatenate(packed).astype(np.float32)


def _samples(c, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    x = torch.randn((c["batch"], 4), generator=g, device=DEV)
    t = 0.3 * torch.randn((c["batch"], c["out"]), generator=g, device=DEV)
    return x, t


def _populations(c, seed):
    Q = 9 if c["dim"] == 2 else 19
    g = torch.Generator(device=DEV).manual_seed(seed)
    return 1e-3 * torch.randn((Q, c["nz"], c["ny"], c["nx"]), generator=g, device=DEV, dtype=torch.float64)


def prepare(case, seed):
    c, k = case, case["kind"]
    if k in ("mlp", "train"):
        widths, w = _weights(c, seed)
        net = MLP(widths, c["batch"], device=DEV)
        net.set_params(w)
        x, t = _samples(c, seed)
        return dict(c=c, net=net, x=x, t=t)
    if k == "checkpoint":
        p = make_params(dim=c["dim"], nx=c["nx"], ny=c["ny"], nz=c["nz"])
        return dict(c=c, s=Solver([p], None, storage=STORE[c["storage"]], device=DEV), f=_populations(c, seed))
    s = _solver(c, seed)
    if k == "monitor":
        s.step(c["steps"])
    return dict(c=c, s=s)


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def run(state):
    c, k = state["c"], state["c"]["kind"]
    if k == "mlp":
        return state["net"].forward(state["x"])
    if k == "train":
        loss = [state["net"].train_step(state["x"], state["t"], 1e-3) for _ in range(c["steps"])]
        return {"loss": torch.tensor(loss, dtype=torch.float32), "params": state["net"].get_params()}
    s = state["s"]
    if k == "checkpoint":
        s.write_populations(0, state["f"])
        return s.read_populations(0)
    if k == "monitor":
        r1, r2, n = s.contact_radius(0, 1.25 * c["xi"], 0.005 * c["R"])
        return {"diag": _table([s.diagnostics(0)]), "contact": torch.tensor([r1, r2], dtype=torch.float64), "n": n}
    s.step(c["steps"])
    if c["n"] == 1:
        rho, U, F = s.read_fields(0)
        q, v, f = s.read_nodes(0)
        return {"rho": rho, "U": U, "F": F, "q": q, "v": v, "f": f}
    got = [s.read_fields(d) for d in range(c["n"])]
    return {"rho": torch.cat([g[0].reshape(-1) for g in got]), "U": torch.cat([g[1].reshape(-1) for g in got]),
            "F": torch.cat([g[2].reshape(-1) for g in got]), "diag": _table(s.diagnostics(-1))}


_FIELDS = ("mass", "momentum", "sum_phi", "sum_F", "dropped_F", "volume", "area", "contact_radius", "height",
           "theta_meas", "max_normal_speed", "max_speed", "min_h", "edge_min", "edge_max")


def _table(diags):
    rows = []
    for d in diags:
        r = []
        for name in _FIELDS:
            r += d[name] if isinstance(d[name], list) else [d[name]]
        rows.append(r)
    return torch.tensor(rows, dtype=torch.float64)


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------

def work(case):
    c, k = case, case["kind"]
    if k in ("mlp", "train"):
        w = [4] + [c["hidden"]] * c["layers"] + [c["out"]]
        par = sum(a * b + b for a, b in zip(w[:-1], w[1:]))
        mul = 2.0 * c["batch"] * sum(a * b for a, b in zip(w[:-1], w[1:]))
        if k == "mlp":
            return {"bytes": 4.0 * c["batch"] * (4 + c["out"]) + 2.0 * par, "flops": mul}
        return {"bytes": c["steps"] * (4.0 * c["batch"] * (4 + c["out"]) + 24.0 * par), "flops": 3 * mul * c["steps"]}
    Q, b = (9, 4) if c["dim"] == 2 else (19, 4)
    if c["storage"] != "f32":
        b = 2
    cells = c["nx"] * c["ny"] * c["nz"]
    if k == "checkpoint":
        return {"bytes": cells * Q * 2.0 * (8 + b), "flops": 0.0}
    if c["n"] > 1:
        cells = 0.45 * cells * c["n"]  # the boxes are drawn below the largest
    out = 4.0 * (1 + 2 * c["dim"]) * cells
    if k == "monitor":
        return {"bytes": cells * Q * b + out, "flops": cells * 2.0 * Q}
    # the state in and out once, and the fields that are read; the arithmetic of every step
    return {"bytes": cells * 2.0 * Q * b + out, "flops": c["steps"] * cells * (150.0 if c["dim"] == 2 else 330.0)}


# ---------------------------------------------------------------------------
# The same in 64 bits
# ---------------------------------------------------------------------------

C2 = [(0, 0), (1, 0), (-1, 0), (0, 1), (0, -1), (1, 1), (-1, -1), (-1, 1), (1, -1)]
C3 = [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1), (1, 1, 0), (-1, -1, 0), (1, -1, 0),
      (-1, 1, 0), (1, 0, 1), (-1, 0, -1), (1, 0, -1), (-1, 0, 1), (0, 1, 1), (0, -1, -1), (0, 1, -1), (0, -1, 1)]


def _delta(q, n, wall):
    """The four taps of the delta kernel along one axis: cells and weights (zero beyond a wall)."""
    base = torch.floor(q - 0.5) - 1
    i = base[:, None] + torch.arange(4, device=q.device)
    r = (i + 0.5 - q[:, None]).abs()
    w = torch.where(r <= 1, (3 - 2 * r + torch.sqrt((1 + 4 * r - 4 * r * r).clamp(min=0))) / 8,
                    (5 - 2 * r - torch.sqrt((-7 + 12 * r - 4 * r * r).clamp(min=0))) / 8)
    i = i.long()
    if wall:
        return i.clamp(0, n - 1), torch.where((i >= 0) & (i < n), w, torch.zeros_like(w))
    return i % n, w


def _forces(q, T, p):
    """Nodal forces: surface tension and wetting."""
    if T is None:
        e = torch.roll(q, -1, 0) - q
        le = e.norm(dim=1, keepdim=True)
        t = e / le
        f = p.sigma * (t - torch.roll(t, 1, 0))
        n = torch.stack([t[:, 1], -t[:, 0]], 1)
        n = n + torch.roll(n, 1, 0)
        share = 0.5 * (le + torch.roll(le, 1, 0))
    else:
        a, b, c = q[T[:, 0]], q[T[:, 1]], q[T[:, 2]]
        m = torch.linalg.cross(b - a, c - a)
        ln = m.norm(dim=1, keepdim=True)
        m = m / ln
        f, n, share = torch.zeros_like(q), torch.zeros_like(q), torch.zeros_like(q[:, :1])
        for k, (u, v) in enumerate(((b, c), (c, a), (a, b))):
            f.index_add_(0, T[:, k], -0.5 * p.sigma * torch.linalg.cross(m, v - u))
            n.index_add_(0, T[:, k], m)
            share.index_add_(0, T[:, k], ln / 6)
    n = n / n.norm(dim=1, keepdim=True)
    A = p.sigma * (p.m_exp - 1) * (p.n_exp - 1) / ((p.n_exp - p.m_exp) * p.xi) * (1 + math.cos(p.theta_eq))
    s = p.xi / q[:, -1:]
    return f - share * A * (s ** p.n_exp - s ** p.m_exp) * n


def _exact_step(c, seed):
    P, nodes, tris = _droplets(c, seed)
    p, dim = P[0], c["dim"]
    C = C2 if dim == 2 else C3
    W = [(4 / 9, 1 / 9, 1 / 36) if dim == 2 else (1 / 3, 1 / 18, 1 / 36)][0]
    w = [W[sum(abs(x) for x in v)] for v in C]
    n = [c["nx"], c["ny"], c["nz"]][:dim]
    sh = tuple(reversed(n))
    ax = [dim - 1 - a for a in range(dim)]  # tensor axis of each lattice axis
    wall = [False] * (dim - 1) + [True]
    q = torch.tensor(nodes[0], dtype=torch.float64, device=DEV)
    T = None if tris[0] is None else torch.tensor(tris[0], dtype=torch.long, device=DEV)
    f = torch.zeros((len(C),) + sh, dtype=torch.float64, device=DEV)  # deviations from the weights
    om = 1 / p.tau
    for _ in range(c["steps"]):
        ph = _forces(q, T, p)
        taps = [_delta(q[:, a], n[a], wall[a]) for a in range(dim)]
        if dim == 2:
            cell = taps[1][0][:, :, None] * n[0] + taps[0][0][:, None, :]
            wt = taps[1][1][:, :, None] * taps[0][1][:, None, :]
        else:
            cell = (taps[2][0][:, :, None, None] * n[1] + taps[1][0][:, None, :, None]) * n[0] + taps[0][0][:, None, None, :]
            wt = taps[2][1][:, :, None, None] * taps[1][1][:, None, :, None] * taps[0][1][:, None, None, :]
        cell, wt = cell.reshape(len(q), -1), wt.reshape(len(q), -1)
        F = torch.stack([torch.zeros(int(np.prod(sh)), dtype=torch.float64, device=DEV).index_add_(
            0, cell.reshape(-1), (ph[:, a:a + 1] * wt).reshape(-1)).reshape(sh) for a in range(dim)])
        g = torch.empty_like(f)
        for i, v in enumerate(C):
            g[i] = torch.roll(f[i], v, ax)
            if v[-1]:  # the walls of the last axis: half-way bounce-back
                o = i if i == 0 else (i + 1 if i % 2 else i - 1)
                at = 0 if v[-1] > 0 else n[-1] - 1
                g[i][at] = f[o][at]
        drho = g.sum(0)
        rho = 1 + drho
        U = torch.stack([sum(g[i] * v[a] for i, v in enumerate(C) if v[a]) + 0.5 * F[a] for a in range(dim)]) / rho
        usq, uF = (U * U).sum(0), (U * F).sum(0)
        for i, v in enumerate(C):
            cu, cF = sum(U[a] * v[a] for a in range(dim)), sum(F[a] * v[a] for a in range(dim))
            eq = w[i] * (drho + rho * (3 * cu + 4.5 * cu * cu - 1.5 * usq))
            f[i] = g[i] - om * (g[i] - eq) + (1 - 0.5 * om) * w[i] * (3 * (cF - uF) + 9 * cu * cF)
        vel = torch.stack([(U[a].reshape(-1)[cell] * wt).sum(1) for a in range(dim)], 1)
        qn = q + vel
        if c["respace"]:
            a, b = torch.roll(q, 1, 0), torch.roll(q, -1, 0)
            ch = b - a
            qn = qn + 0.5 * c["respace"] * ((b - q).norm(dim=1) - (q - a).norm(dim=1))[:, None] * ch / ch.norm(dim=1, keepdim=True)
        q = qn
    full = (sh[0],) + sh[1:] if dim == 3 else (1,) + sh
    return {"rho": rho.reshape(full), "U": U.reshape((dim,) + full), "F": F.reshape((dim,) + full), "q": q.cpu().numpy(),
            "v": vel.cpu().numpy(), "f": ph.cpu().numpy()}


def _gelu(z):
    return 0.5 * z * (1 + torch.erf(z / math.sqrt(2)))


def _exact_net(c, seed):
    widths, packed = _weights(c, seed)
    par, o = [], 0
    for a, b in zip(widths[:-1], widths[1:]):
        for sh in ((a, b), (b,)):
            k = int(np.prod(sh))
            par.append(torch.tensor(packed[o:o + k].reshape(sh), dtype=torch.float64, device=DEV, requires_grad=True))
            o += k
    x, t = (v.double() for v in _samples(c, seed))

    def forward():
        h = x
        for l in range(0, len(par), 2):
            h = h @ par[l] + par[l + 1]
            h = _gelu(h) if l + 2 < len(par) else h
        return h

    if c["kind"] == "mlp":
        return forward().detach()
    losses = []
    opt = torch.optim.Adam(par, lr=1e-3, betas=(0.9, 0.999), eps=1e-8)
    for _ in range(c["steps"]):
        opt.zero_grad()
        loss = ((forward() - t) ** 2).mean()
        loss.backward()
        opt.step()
        losses.append(loss.detach().cpu())
    return {"loss": torch.stack(losses), "params": None}


def exact(case, seed):
    c, k = case, case["kind"]
    if k in ("mlp", "train"):
        return _exact_net(c, seed)
    if k == "checkpoint":
        return _populations(c, seed)
    if k == "step" and c["n"] == 1 and c["lam"] == 1.0:
        return _exact_step(c, seed)
    return None  # batches, two viscosities and reductions over a state that the steps before made
