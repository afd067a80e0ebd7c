"""The work that users of the planner have it do, as measurable cases.

A case is one pass through the public entry points of the Python binding over
the C ABI: a plan (rollout and selection), a gradient of the candidate costs,
the preparation of a new map, or a burst of requests to the planning server.
Sizes come from the repository's own workloads (``inputs.py``: c1, c2, c3, c4,
c5 and the paper's solver shape; ``bench.py``: its rows) and from ragged sizes
between them; all data are float32, the only type the library takes.

``listed`` names the cases, ``draw`` gives more of the same ranges,
``prepare`` makes the inputs and the planner a program keeps, ``run`` is one
pass, ``work`` what it cannot do without, and ``exact`` the same outputs in 64
bits, written here from the model's equations in plain torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2603_20525_amd import inputs
from paper_2603_20525_amd import plan as P

# Operations of one Euler step of each model (an add, multiply, fused
# multiply-add, compare or transcendental call counts one).
SRB_STEP, SRB_COSTMAP, EST_STEP, RK4_STEP, ADJOINT_STEP = 386, 16, 109, 1576, 1502
LAMBDA = 25.0                      # softmin temperature, cost units
SIGMA_OBSTACLE, EPS_OBSTACLE = 1.0e6, 0.25


# ---------------------------------------------------------------- the cases

def listed():
    return [
        # The smallest plan (c1): a coarse first look, or the local repair of
        # a plan; its time is launches, waiting and one wave's latency.
        _plan("plan-small", K=64, N=50, terrain="bumps", W=128, H=128, res=0.2, v0=8.0),
        # One plan per control period (c2): the ordinary call of an MPC loop.
        _plan("plan-single", K=4096, N=100, terrain="fbm", W=512, H=512, res=0.1, v0=15.0),
        # The stress plan (c5): many candidates over a large fine map.
        _plan("plan-stress", K=65536, N=200, dt=0.01, terrain="slopes", W=2048, H=2048,
              res=0.05, v0=20.0, std0=0.15, std1=0.3),
        # MPPI-style use among obstacles, at a ragged size: costmap, two
        # calls, the weighted mean, the final states.
        _plan("plan-softmin-costmap", K=10007, N=73, terrain="fbm", W=317, H=251, res=0.1,
              v0=10.0, select="softmin", costmap=True, final=True),
        # The paper's solver end to end: uniform steering rates drawn in the
        # kernel, 16 holds of 50 Euler substeps, arg-min.
        _plan("sampled-paper", K=204288, N=16, S=50, dt=0.25, draws="uniform", terrain="fbm",
              W=512, H=512, res=0.1, v0=7.5, vehicle="paper"),
        # Gaussian candidates around the last plan, drawn in the kernel; an
        # odd number of them, between the tuned sizes.
        _plan("sampled-gauss", K=30011, N=60, draws="gauss", terrain="fbm", W=512, H=512,
              res=0.1, v0=12.0),
        # The extended single-track baseline on the paper's shape.
        _plan("est-paper", model="est", K=204288, N=16, S=50, dt=0.25, draws="held",
              terrain="fbm", W=512, H=512, res=0.1, v0=7.5, vehicle="paper", select="none",
              final=True),
        # The Runge-Kutta integrator on the ordinary plan.
        _plan("rk4-single", model="rk4", K=4096, N=100, terrain="fbm", W=512, H=512, res=0.1,
              v0=15.0, select="none", final=True),
        # Gradient refinement (c4): costs and their gradients.
        _grad("grad-refine", K=1024, N=100, every=10, terrain="fbm", W=512, H=512, res=0.1,
              v0=15.0),
        # A new map for the SRB model: smoothed at 0.3 m, 20 obstacles and a
        # path boundary turned into a costmap, packed, and a plan on it.
        _map("map-srb", W=2048, H=2048, res=0.05, sigma=0.3, obstacles=20, K=1024, N=50),
        # A new map for the EST model: smoothed at 1.5 m, ragged sides.
        _map("map-est", model="est", W=1537, H=1025, res=0.05, sigma=1.5, obstacles=9,
             K=1000, N=40),
        # The serving trace's 64 requests (c3) arriving at once.
        {"name": "serve-burst", "kind": "serve", "requests": 64, "min_n": 40, "max_n": 160,
         "chunk": 16, "slots": 64},
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["plan", "plan", "sampled", "sampled", "est", "rk4", "grad", "map",
                       "map", "serve"])
    terrain = rng.choice(["fbm", "bumps", "slopes"])
    ground = {"terrain": terrain, "W": log_int(200, 1600), "H": log_int(200, 1600),
              "res": {"fbm": 0.1, "bumps": 0.2, "slopes": 0.05}[terrain],
              "v0": round(rng.uniform(5.0, 20.0), 2)}
    if kind == "plan":
        K = log_int(50, 65536)
        N = rng.randint(20, min(200, max(30, 200 * 65536 // K)))
        return _plan(None, K=K, N=N, dt=rng.choice([0.01, 0.02]),
                     select=rng.choice(["argmin", "argmin", "softmin"]),
                     costmap=rng.random() < 0.4, final=rng.random() < 0.4, **ground)
    if kind == "sampled":
        draws = rng.choice(["uniform", "gauss"])
        if draws == "uniform" and rng.random() < 0.6:
            return _plan(None, K=log_int(4000, 200000), N=rng.randint(8, 16),
                         S=rng.randint(10, 50), dt=0.25, draws=draws, vehicle="paper",
                         **{**ground, "v0": round(rng.uniform(4.0, 9.0), 2)})
        return _plan(None, K=log_int(500, 200000), N=rng.randint(20, 100), draws=draws,
                     costmap=rng.random() < 0.3, final=rng.random() < 0.4, **ground)
    if kind == "est":
        return _plan(None, model="est", K=log_int(1000, 204000), N=rng.randint(8, 16),
                     S=rng.randint(8, 50), dt=0.25, draws="held", select="none",
                     costmap=rng.random() < 0.3, final=rng.random() < 0.5, vehicle="paper",
                     **{**ground, "v0": round(rng.uniform(4.0, 9.0), 2)})
    if kind == "rk4":
        return _plan(None, model="rk4", K=log_int(200, 20000), N=rng.randint(20, 120),
                     select="none", costmap=rng.random() < 0.3, final=True, **ground)
    if kind == "grad":
        S = rng.choice([1, 1, 2, 5])
        return _grad(None, K=log_int(16, 6000), N=rng.randint(20, 120) // S + 1, S=S,
                     dt=0.02 * S, every=rng.choice([1, 5, 10, 16, 33]),
                     costmap=rng.random() < 0.3, **ground)
    if kind == "map":
        return _map(None, model=rng.choice(["srb", "est"]), W=log_int(200, 2000),
                    H=log_int(200, 2000), res=rng.choice([0.05, 0.1]),
                    sigma=rng.choice([0.1, 0.3, 0.3, 0.6, 1.5]), obstacles=rng.randint(0, 40),
                    K=log_int(64, 4000), N=rng.randint(20, 60))
    return {"kind": "serve", "requests": rng.randint(1, 64), "min_n": 40,
            "max_n": rng.randint(60, 160), "chunk": rng.choice([8, 16, 32]),
            "slots": rng.choice([4, 16, 64])}


def _plan(name, model="srb", K=64, N=50, S=1, dt=0.02, draws="given", std0=0.1, std1=0.2,
          terrain="fbm", W=512, H=512, res=0.1, v0=10.0, vehicle="workload", select="argmin",
          costmap=False, final=False):
    """draws: given (Gaussian candidates in memory), held (uniform steering
    rates in memory), uniform / gauss (drawn inside the rollout kernel)."""
    c = dict(kind="plan", model=model, K=K, N=N, S=S, dt=dt, draws=draws, std0=std0, std1=std1,
             terrain=terrain, W=W, H=H, res=res, v0=v0, vehicle=vehicle, select=select,
             costmap=costmap, final=final)
    return dict(c, name=name) if name else c


def _grad(name, K=1024, N=100, S=1, dt=0.02, every=10, terrain="fbm", W=512, H=512, res=0.1,
          v0=15.0, costmap=False):
    c = _plan(name, K=K, N=N, S=S, dt=dt, terrain=terrain, W=W, H=H, res=res, v0=v0,
              select="none", costmap=costmap)
    return dict(c, kind="grad", every=every)


def _map(name, model="srb", W=512, H=512, res=0.05, sigma=0.3, obstacles=8, K=1024, N=50):
    c = _plan(name, model=model, K=K, N=N, terrain="slopes", W=W, H=H, res=res, v0=8.0,
              select="argmin" if model == "srb" else "none", costmap=True)
    return dict(c, kind="map", sigma=sigma, obstacles=obstacles)


# ----------------------------------------------------------------- the inputs

def _gen(seed, salt):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + salt) & 0x7FFFFFFFFFFF)
    return g


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device="cuda", dtype=torch.float64)


def _heights(case, seed):
    """A [H][W] float32 heightmap of the case's kind: a sum of Gaussian bumps,
    five octaves of lattice noise with two berms, or alternating side slopes
    with berms and ruts (the terrains of inputs.py, made on the GPU)."""
    W, H, res, g = case["W"], case["H"], case["res"], _gen(seed, 1)
    x = res * torch.arange(W, device="cuda", dtype=torch.float64)
    y = res * torch.arange(H, device="cuda", dtype=torch.float64)
    X, Y = x[None, :], y[:, None]
    ex, ey = W * res, H * res
    if case["terrain"] == "bumps":
        r = _rand(g, 4, 40)
        amp, wid = 0.4 * r[0], 0.5 + 2.5 * r[1]
        gx = torch.exp(-(x[None, :] - ex * r[2][:, None]) ** 2 / (2 * wid[:, None] ** 2))
        gy = torch.exp(-(y[None, :] - ey * r[3][:, None]) ** 2 / (2 * wid[:, None] ** 2))
        h = (gy * amp[:, None]).T @ gx
    elif case["terrain"] == "fbm":
        h = torch.zeros(H, W, device="cuda", dtype=torch.float64)
        for o in range(5):
            h += 0.5 ** o * _lattice_noise(g, x, y, 12.8 * 0.5 ** o)
        h = 0.6 * (h - h.min()) / (h.max() - h.min())
        off = (2.0 * _rand(g, 2) - 1.0).tolist()
        for part, ang, o in ((0.4, 30.0, off[0]), (0.63, -30.0, off[1])):
            h += _ridge(X, Y, part * ex + o, ey / 2, ang, 0.3, 0.4)
    else:
        h = math.tan(math.radians(15.0)) * (Y - ey / 2) * torch.tanh(4 * torch.sin(X * math.pi / 10))
        h = 3.0 * torch.tanh(h / 3.0)
        r = _rand(g, 2, 64).tolist()
        at, i = 5.0, 0
        while at < ex - 5.0 and i < 64:
            at += 12.0 + 6.0 * r[0][i]
            h += _ridge(X, Y, at, ey / 2, 60.0 * r[1][i] - 30.0, 0.5, 1.0)
            i += 1
        for yr in (ey / 2 - 0.75, ey / 2 + 0.75):
            h -= 0.3 * torch.exp(-((Y - yr) ** 2) / (2 * 0.3 ** 2))
    return h.float().contiguous()


def _ridge(X, Y, xc, yc, angle, height, sigma):
    a = math.radians(angle)
    d = (X - xc) * math.cos(a) - (Y - yc) * math.sin(a)
    return height * torch.exp(-d * d / (2 * sigma * sigma))


def _lattice_noise(g, x, y, spacing):
    gx, gy = x / spacing, y / spacing
    ix, iy = gx.floor().long(), gy.floor().long()
    lat = 2.0 * _rand(g, int(iy.max()) + 2, int(ix.max()) + 2) - 1.0
    tx, ty = gx - ix, gy - iy
    fx = (tx ** 3 * (tx * (tx * 6 - 15) + 10))[None, :]
    fy = (ty ** 3 * (ty * (ty * 6 - 15) + 10))[:, None]
    lo, hi = lat[iy], lat[iy + 1]
    a = lo[:, ix] * (1 - fx) + lo[:, ix + 1] * fx
    b = hi[:, ix] * (1 - fx) + hi[:, ix + 1] * fx
    return a * (1 - fy) + b * fy


def _settled(h, res, x, y, psi, v0, hR):
    """Initial state at rest on the plane through the ground around (x, y),
    body speed v0, as 13 floats."""
    H, W = h.shape
    i = min(max(int(round(x / res)), 0), W - 1)
    j = min(max(int(round(y / res)), 0), H - 1)
    n = max(1, int(round(2.0 / res)))
    i0, i1, j0, j1 = max(i - n, 0), min(i + n, W - 1), max(j - n, 0), min(j + n, H - 1)
    patch = h[j0:j1 + 1, i0:i1 + 1].double().cpu().numpy()
    px, py = np.meshgrid(res * np.arange(i0, i1 + 1) - x, res * np.arange(j0, j1 + 1) - y)
    A = np.stack([np.ones(px.size), px.ravel(), py.ravel()], 1)
    f0, a, b = np.linalg.lstsq(A, patch.ravel(), rcond=None)[0]
    nrm = np.array([-a, -b, 1.0]) / math.sqrt(1 + a * a + b * b)
    c, s = math.cos(psi), math.sin(psi)
    n1 = (c * nrm[0] + s * nrm[1], -s * nrm[0] + c * nrm[1])
    phi = -math.asin(max(-1.0, min(1.0, n1[1])))
    theta = math.atan2(n1[0], nrm[2])
    st = [x, y, f0 + hR / nrm[2], psi, theta, phi, v0] + [0.0] * 6
    return [float(np.float32(v)) for v in st]


def _candidates(case, seed, K, N):
    """Controls [N][2][K]: Gaussian around a sinusoidal steering-rate nominal
    (candidate 0 is the nominal), or uniform steering rates."""
    g = _gen(seed, 2)
    if case["draws"] == "held":
        u = torch.zeros(N, 2, K, device="cuda")
        u[:, 0] = (2.0 * torch.rand(N, K, generator=g, device="cuda") - 1.0)
        return u
    u = torch.randn(N, 2, K, generator=g, device="cuda")
    u[:, 0] *= case["std0"]
    u[:, 1] *= case["std1"]
    u[:, :, 0] = 0.0
    u[:, 0] += _nominal(g, N, case["dt"])[:, :1]
    return u.contiguous()


def _nominal(g, N, dt):
    r = _rand(g, 3).tolist()
    t = dt * torch.arange(N, device="cuda", dtype=torch.float64)
    nom = torch.zeros(N, 2, device="cuda")
    nom[:, 0] = (0.5 * r[0] * torch.sin(2 * math.pi * ((0.2 + 0.8 * r[1]) * t + r[2]))).float()
    return nom


def _polygons(case, seed):
    """Obstacle dodecagons off the start, and the path boundary 1 m inside the map."""
    g = _gen(seed, 3)
    ex, ey = case["W"] * case["res"], case["H"] * case["res"]
    n = case.get("obstacles", 6)
    r = _rand(g, 4, max(n, 1)).tolist()
    polys = []
    for i in range(n):
        cx, cy = ex * (0.3 + 0.65 * r[0][i]), ey * (0.1 + 0.8 * r[1][i])
        rad, ph = 0.8 + 1.2 * r[2][i], 2 * math.pi * r[3][i]
        polys.append((0, [(cx + rad * math.cos(ph + math.pi * q / 6),
                           cy + rad * math.sin(ph + math.pi * q / 6)) for q in range(12)]))
    x1, y1 = (case["W"] - 1) * case["res"] - 1.0, (case["H"] - 1) * case["res"] - 1.0
    polys.append((1, [(1.0, 1.0), (x1, 1.0), (x1, y1), (1.0, y1)]))
    verts = np.concatenate([np.asarray(v, np.float32) for _, v in polys])
    offsets = np.concatenate([[0], np.cumsum([len(v) for _, v in polys])]).astype(int)
    return torch.from_numpy(verts).cuda(), [int(o) for o in offsets], [k for k, _ in polys]


def _problem(case, seed):
    """Vehicle, cost, integration, heights and initial state of a case."""
    veh = dict(inputs.PAPER_VEHICLE if case["vehicle"] == "paper" else inputs.WORKLOAD_VEHICLE)
    h = _heights(case, seed)
    ex, ey = case["W"] * case["res"], case["H"] * case["res"]
    r = _rand(_gen(seed, 4), 3).tolist()
    x, y = ex * (0.12 + 0.1 * r[0]), ey * (0.45 + 0.1 * r[1])
    psi = 0.4 * (r[2] - 0.5)
    cost = dict(inputs.BASE_COST, goal_x=float(np.float32(0.9 * ex)), goal_y=float(np.float32(ey / 2)))
    integ = dict(inputs.BASE_INTEG, dt=case["dt"], substeps=case["S"],
                 method=P.PLAN_RK4 if case["model"] == "rk4" else P.PLAN_EULER)
    s0 = _settled(h, case["res"], x, y, psi, case["v0"], veh["hR"])
    if case["model"] == "est":
        s0 = [s0[0], s0[1], s0[3], 0.0, 0.0, 0.0, s0[6]]
    return veh, cost, integ, h, s0


def _spec(case, seed):
    nom = _nominal(_gen(seed, 5), case["N"], case["dt"]) if case["draws"] == "gauss" else None
    if nom is None:
        return dict(kind=P.PLAN_SAMPLE_UNIFORM, seed=int(seed) + 11, stream=3, scale=(1.0, 0.0),
                    nominal=None, keep=False)
    return dict(kind=P.PLAN_SAMPLE_GAUSSIAN, seed=int(seed) + 11, stream=3,
                scale=(case["std0"], case["std1"]), nominal=nom, keep=True)


def _serve_sizes(case):
    """(K, N) of each request of a burst: the case's own, whatever the seed."""
    r = np.random.default_rng([case["requests"], case["min_n"], case["max_n"], 3000])
    return [(int(r.choice([512, 1024, 2048, 4096, 8192])),
             int(r.integers(case["min_n"], case["max_n"] + 1))) for _ in range(case["requests"])]


def _serve_requests(case, seed):
    r = np.random.default_rng(int(seed))
    out = []
    for i, (K, N) in enumerate(_serve_sizes(case)):
        v0, psi = float(r.uniform(5.0, 20.0)), float(r.uniform(0.0, 2 * math.pi))
        one = _plan(None, K=K, N=N, terrain="fbm", W=256, H=256, res=0.1, v0=v0)
        h = _heights(one, int(seed) * 131 + i)
        s0 = _settled(h, 0.1, 12.8, 12.8, psi, v0, inputs.WORKLOAD_VEHICLE["hR"])
        d = 1.5 * v0 * N * 0.02
        gx = min(max(12.8 + d * math.cos(psi), 2.0), 23.5)
        gy = min(max(12.8 + d * math.sin(psi), 2.0), 23.5)
        cost = dict(inputs.BASE_COST, goal_x=float(np.float32(gx)), goal_y=float(np.float32(gy)))
        out.append((h, s0, cost, _candidates(one, int(seed) * 131 + i, K, N)))
    return out


def prepare(case, seed):
    if case["kind"] == "serve":
        reqs = _serve_requests(case, seed)
        maxN = max(u.shape[0] for *_, u in reqs)
        srv = P.Server(inputs.WORKLOAD_VEHICLE, case["slots"], 8192, maxN, 256, 256, 4 << 30,
                       case["chunk"])
        total = sum(u.shape[0] for *_, u in reqs)
        flat = torch.zeros(2 * total, device="cuda")
        plans, at = [], 0
        for *_, u in reqs:
            plans.append(flat[2 * at:2 * (at + u.shape[0])].view(-1, 2))
            at += u.shape[0]
        integ = dict(inputs.BASE_INTEG)
        return {"case": case, "srv": srv, "reqs": reqs, "plans": plans, "flat": flat, "integ": integ}
    K, N = case["K"], case["N"]
    veh, cost, integ, h, s0 = _problem(case, seed)
    pl = P.Planner(veh, cost, integ, K, N, case["W"], case["H"])
    st = {"case": case, "pl": pl, "s0": s0, "J": torch.empty(K, device="cuda"),
          "plan": torch.empty(N, 2, device="cuda"), "h": h, "final": None}
    if case["final"]:
        st["final"] = torch.empty(7 if case["model"] == "est" else 13, K, device="cuda")
    if case["draws"] in ("uniform", "gauss"):
        s = _spec(case, seed)
        st["nominal"] = s["nominal"]  # kept alive for the calls that use the spec
        st["spec"] = P.sample_spec(s["kind"], s["seed"], s["stream"], s["scale"], s["nominal"],
                                   s["keep"], N)
    else:
        st["u"] = _candidates(case, seed, K, N)
    if case["kind"] == "map":
        st["verts"], st["offsets"], st["kinds"] = _polygons(case, seed)
        st["smooth"], st["costmap"] = torch.empty_like(h), torch.empty_like(h)
        return st
    cm = None
    if case["costmap"]:
        verts, offsets, kinds = _polygons(case, seed)
        cm = torch.empty_like(h)
        pl.costmap_polygons(verts, offsets, kinds, cm, 0.0, 0.0, case["res"], SIGMA_OBSTACLE,
                            EPS_OBSTACLE)
    pl.set_terrain(h, 0.0, 0.0, case["res"], cm)
    if case["kind"] == "grad":
        st["grad"] = torch.empty(N, 2, K, device="cuda")
    return st


# ------------------------------------------------------------------- one pass

def run(st):
    case = st["case"]
    if case["kind"] == "serve":
        srv, ids = st["srv"], []
        for (h, s0, cost, u), plan in zip(st["reqs"], st["plans"]):
            ids.append(srv.submit(h, 0.0, 0.0, 0.1, s0, u, cost, st["integ"], plan))
        srv.drain()
        srv.completions(len(ids))
        res = [srv.result(i) for i in ids]
        return {"plans": st["flat"], "k": np.array([r["best_k"] for r in res]),
                "J": np.array([r["best_cost"] for r in res], np.float32)}
    pl, s0, J, plan, final = st["pl"], st["s0"], st["J"], st["plan"], st["final"]
    if case["kind"] == "grad":
        pl.rollout_grad(s0, st["u"], J, st["grad"], checkpoint_every=case["every"])
        return {"J": J, "grad": st["grad"]}
    out = {"J": J}
    if case["kind"] == "map":
        pl.smooth_terrain(st["h"], case["res"], case["sigma"], st["smooth"])
        pl.costmap_polygons(st["verts"], st["offsets"], st["kinds"], st["costmap"], 0.0, 0.0,
                            case["res"], SIGMA_OBSTACLE, EPS_OBSTACLE)
        pl.set_terrain(st["smooth"], 0.0, 0.0, case["res"], st["costmap"])
        out.update(smooth=st["smooth"], costmap=st["costmap"])
    if final is not None:
        out["final"] = final
    best = None
    if case["model"] == "est":
        pl.rollout_est(s0, st["u"], J, final)
    elif "spec" in st:
        if case["select"] == "argmin":
            best = pl.rollout_sampled_argmin(s0, st["spec"], case["N"], J, plan, final)
        else:
            pl.rollout_sampled(s0, st["spec"], case["N"], J, final)
    elif case["select"] == "argmin":
        best = pl.rollout_argmin(s0, st["u"], J, plan, final)
    else:
        pl.rollout(s0, st["u"], J, final)
        if case["select"] == "softmin":
            best = pl.select(st["u"], J, plan, P.PLAN_SOFTMIN, LAMBDA)
    if best is not None:
        out.update(plan=plan, k=best[0], best=best[1])
    return out


# ------------------------------------------------------------------- its work

def work(case):
    """Inputs read once, outputs written once, and the models' operations."""
    if case["kind"] == "serve":
        sizes = _serve_sizes(case)
        return {"bytes": sum(4 * 256 * 256 + 8 * K * N + 8 * N for K, N in sizes),
                "flops": sum(SRB_STEP * K * N for K, N in sizes)}
    K, N, S, nodes = case["K"], case["N"], case["S"], case["W"] * case["H"]
    step = {"srb": SRB_STEP + (SRB_COSTMAP if case["costmap"] else 0), "est": EST_STEP,
            "rk4": RK4_STEP}[case["model"]]
    flops = float(step) * K * N * S
    nbytes = 4.0 * K + 8 * N
    if case["draws"] in ("given", "held"):
        nbytes += 8.0 * K * N
    if case["final"]:
        nbytes += 4.0 * K * (7 if case["model"] == "est" else 13)
    if case["kind"] == "grad":
        flops += float(ADJOINT_STEP) * K * N * S
        nbytes += 8.0 * K * N
    if case["kind"] == "map":
        # heights read, smoothed heights, costmap and packed cells written;
        # two passes of taps, the boundary and the nodes near an obstacle
        taps = 2 * math.ceil(3 * case["sigma"] / case["res"] - 1e-6) + 1
        nbytes += 4.0 * nodes * 3 + 64.0 * nodes
        flops += 2.0 * taps * nodes + 4.0 * nodes
    return {"bytes": nbytes, "flops": flops}


# ---------------------------------------------------- the same, in 64 bits

class _Ground:
    """Height, slopes (central differences, one-sided on the border) and cost
    rate at nodes of R grids [R][H][W], bilinear between them, clamped to the edge."""

    def __init__(self, h, res, cm=None):
        h = h.double()
        self.res, (self.R, self.H, self.W) = res, h.shape
        fx, fy = torch.empty_like(h), torch.empty_like(h)
        fx[:, :, 1:-1] = (h[:, :, 2:] - h[:, :, :-2]) / (2 * res)
        fx[:, :, 0], fx[:, :, -1] = (h[:, :, 1] - h[:, :, 0]) / res, (h[:, :, -1] - h[:, :, -2]) / res
        fy[:, 1:-1] = (h[:, 2:] - h[:, :-2]) / (2 * res)
        fy[:, 0], fy[:, -1] = (h[:, 1] - h[:, 0]) / res, (h[:, -1] - h[:, -2]) / res
        chans = [h, fx, fy] + ([cm.double()] if cm is not None else [])
        self.t = torch.stack(chans, -1).view(-1, len(chans))

    def at(self, g, x, y):
        u = (x / self.res).clamp(0, self.W - 1)
        v = (y / self.res).clamp(0, self.H - 1)
        i, j = u.detach().floor().clamp(max=self.W - 2).long(), v.detach().floor().clamp(max=self.H - 2).long()
        tx, ty = (u - i)[..., None], (v - j)[..., None]
        q = (g * self.H + j) * self.W + i
        return ((1 - ty) * ((1 - tx) * self.t[q] + tx * self.t[q + 1]) +
                ty * ((1 - tx) * self.t[q + self.W] + tx * self.t[q + self.W + 1]))


def _srb(veh, cost, ground, g, st, dd, ax):
    """State derivative [13][K] and running cost rate [K] of the SRB model."""
    V = veh
    x, y, z, psi, th, ph, vx, vy, vz, wx, wy, wz, delta = st
    sps, cps, sth, cth, sph, cph = psi.sin(), psi.cos(), th.sin(), th.cos(), ph.sin(), ph.cos()
    R = ((cps * cth, cps * sph * sth - cph * sps, sph * sps + cph * cps * sth),
         (cth * sps, cph * cps + sph * sps * sth, cph * sps * sth - cps * sph),
         (-sth, cth * sph, cph * cth))
    gB = [-V["g"] * R[2][c] for c in range(3)]
    L = V["Lf"] + V["Lr"]
    FxR = 0.5 * V["M"] * (ax + wy * vz - wz * vy - gB[0])
    Fy = Fz = Mx = My = Mz = 0.0
    csum = 0.0
    for i in range(4):
        front = i < 2
        r = (V["Lf"] if front else -V["Lr"], (-0.5 if i & 1 else 0.5) * V["e"], -V["hR"])
        Pw = [p + R[q][0] * r[0] + R[q][1] * r[1] + R[q][2] * r[2] for q, p in enumerate((x, y, z))]
        vi = (vx + wy * r[2] - wz * r[1], vy + wz * r[0] - wx * r[2], vz + wx * r[1] - wy * r[0])
        T = ground.at(g, Pw[0], Pw[1])
        n = [-R[0][c] * T[..., 1] - R[1][c] * T[..., 2] + R[2][c] for c in range(3)]
        chi = (Pw[2] - T[..., 0]) / n[2]
        chid = (n[0] * (vi[0] - chi * wy) + n[1] * (vi[1] + chi * wx) + n[2] * vi[2]) / n[2]
        k, b = (V["kf"], V["bf"]) if front else (V["kr"], V["br"])
        Fk = (0.5 * V["g"] * V["M"] * (V["Lr"] if front else V["Lf"]) / L - k * chi).clamp(min=0.0)
        Fb = torch.where(Fk > 0, torch.maximum(-b * chid, -Fk), torch.zeros_like(Fk))
        fz = Fk + Fb
        alpha = torch.atan(vi[1] / vi[0]) - (delta if front else 0.0)
        Ca = V["C"] * alpha
        fy = -fz * V["mu"] * Ca / torch.sqrt(V["mu"] ** 2 + Ca ** 2)
        fy = fy * delta.cos() if front else fy
        fx = 0.0 if front else FxR
        Fy, Fz = Fy + fy, Fz + fz
        Mx = Mx + r[1] * fz - r[2] * fy
        My = My + r[2] * fx - r[0] * fz
        Mz = Mz + r[0] * fy - r[1] * fx
        if T.shape[-1] > 3:
            csum = csum + T[..., 3]
    psid = (sph * wy + cph * wz) / cth
    d = (R[0][0] * vx + R[0][1] * vy + R[0][2] * vz, R[1][0] * vx + R[1][1] * vy + R[1][2] * vz,
         R[2][0] * vx + R[2][1] * vy + R[2][2] * vz,
         psid, cph * wy - sph * wz, wx + sth * psid, ax,
         Fy / V["M"] + gB[1] + wx * vz - wz * vx, Fz / V["M"] + gB[2] + wy * vx - wx * vy,
         (Mx + (V["Jyy"] - V["Jzz"]) * wy * wz) / V["Jxx"],
         (My - (V["Jxx"] - V["Jzz"]) * wx * wz) / V["Jyy"],
         (Mz + (V["Jxx"] - V["Jyy"]) * wx * wy) / V["Jzz"], dd)
    rbar, bar = math.hypot(V["hR"], 0.5 * V["e"]), math.atan(2 * V["hR"] / V["e"])
    ang = ph.abs() + bar
    U = V["M"] * V["g"] * rbar * (1 - ang.sin()) * cth
    U = torch.where(ang > 0.5 * math.pi, -U, U)
    eps = 0.1 * V["M"] * V["g"] * (rbar - V["hR"])
    rate = cost["w_t"] + cost["w_c"] * dd ** 2 + cost["sigma"] * (1 - U / eps).clamp(min=0.0) ** 2
    return torch.stack(d), rate + csum


def _est(veh, cost, ground, g, st, dd, ax):
    """State derivative [7][K] and running cost rate [K] of the EST model."""
    V = veh
    x, y, psi, vy, wz, delta, vx = st
    T = ground.at(g, x, y)
    fx, fy = T[..., 1], T[..., 2]
    s = torch.sqrt(1 + fx ** 2 + fy ** 2)
    th, ph = torch.asin(-fx / s), torch.atan(fy)
    sth, cth, sph, cph, sps, cps = th.sin(), th.cos(), ph.sin(), ph.cos(), psi.sin(), psi.cos()
    R11, R12 = cth * cps, -cth * sps
    R21, R22 = cps * sph * sth + cph * sps, -sph * sth * sps + cph * cps
    gBy, gBz = -V["g"] * (cph * sth * sps + cps * sph), -V["g"] * cph * cth
    L = V["Lf"] + V["Lr"]
    axb = ax - wz * vy
    Fzf = -V["M"] * V["Lr"] / L * gBz - V["M"] * V["hR"] / L * axb
    Fzr = -V["M"] * V["Lf"] / L * gBz + V["M"] * V["hR"] / L * axb

    def tire(Fz, alpha):
        Ca = V["C"] * alpha
        return -Fz * V["mu"] * Ca / torch.sqrt(V["mu"] ** 2 + Ca ** 2)

    Fyf = tire(Fzf, torch.atan((vy + wz * V["Lf"]) / vx) - delta)
    Fyr = tire(Fzr, torch.atan((vy - wz * V["Lr"]) / vx))
    ay = (Fyf + Fyr) / V["M"]
    bar = V["g"] * V["e"] / (2 * V["hR"])
    rate = cost["w_t"] + cost["w_c"] * dd ** 2 + cost["sigma"] * (1 + (ay.abs() - bar) / (0.1 * bar)).clamp(min=0.0) ** 2
    if T.shape[-1] > 3:
        R13, R23 = sth, -cth * sph
        for i in range(4):
            rx, ry = V["Lf"] if i < 2 else -V["Lr"], (-0.5 if i & 1 else 0.5) * V["e"]
            rate = rate + ground.at(g, x + R11 * rx + R12 * ry - R13 * V["hR"],
                                    y + R21 * rx + R22 * ry - R23 * V["hR"])[..., 3]
    return torch.stack((R11 * vx + R12 * vy, R21 * vx + R22 * vy, wz, ay + gBy - wz * vx,
                        (Fyf * V["Lf"] * delta.cos() - Fyr * V["Lr"]) / V["Jzz"], dd, ax)), rate


def _rollout(model, veh, cost, integ, ground, g, s0, u, goal, n_steps=None):
    """Costs [K] and final states of controls u [N][2][K]; g, goal ([2][K]) and
    n_steps say each candidate's grid, goal and horizon."""
    K = u.shape[2]
    rhs, D, V = (_est, 5, 6) if model == "est" else (_srb, 12, 6)
    st = s0.clone() if s0.dim() == 2 else s0[:, None].expand(-1, K).clone()
    J = torch.zeros(K, device=u.device, dtype=torch.float64)
    S, h = integ["substeps"], integ["dt"] / integ["substeps"]
    lim, rate = veh["delta_max"], veh["delta_rate_max"]
    for n in range(u.shape[0]):
        dd, ax = u[n, 0].clamp(-rate, rate), integ["accel_max"] * u[n, 1].clamp(-1, 1)
        for _ in range(S):
            at_goal = (st[0] - goal[0]) ** 2 + (st[1] - goal[1]) ** 2 <= cost["goal_r"] ** 2
            live = ~at_goal if n_steps is None else ~at_goal & (n < n_steps)
            d, L = rhs(veh, cost, ground, g, st, dd, ax)
            if model == "rk4":
                d2, L2 = rhs(veh, cost, ground, g, st + 0.5 * h * d, dd, ax)
                d3, L3 = rhs(veh, cost, ground, g, st + 0.5 * h * d2, dd, ax)
                d4, L4 = rhs(veh, cost, ground, g, st + h * d3, dd, ax)
                d, L = (d + 2 * d2 + 2 * d3 + d4) / 6, (L + 2 * L2 + 2 * L3 + L4) / 6
            new = list(st + h * d)
            new[D] = new[D].clamp(-lim, lim)
            new[V] = new[V].clamp(min=integ["vx_min"])
            st = torch.where(live, torch.stack(new), st)
            J = torch.where(live, J + h * L, J)
    J = J + cost["w_g"] * torch.sqrt((st[0] - goal[0]) ** 2 + (st[1] - goal[1]) ** 2)
    ok = torch.isfinite(J) & torch.isfinite(st).all(0)
    return torch.where(ok, J, torch.full_like(J, math.inf)), st


def _smoothed(h, res, sigma):
    r = math.ceil(3 * sigma / res - 1e-6)
    d = torch.arange(-r, r + 1, device=h.device, dtype=torch.float64) * res
    w = torch.exp(-d * d / (2 * sigma * sigma))
    w = w / w.sum()
    out = h.double()
    for dim in (1, 0):
        n = out.shape[dim]
        acc = torch.zeros_like(out)
        for q in range(2 * r + 1):
            i = (torch.arange(n, device=h.device) + q - r).clamp(0, n - 1)
            acc += w[q] * out.index_select(dim, i)
        out = acc
    return out


def _distance_cost(case, verts, offsets, kinds):
    px = case["res"] * torch.arange(case["W"], device="cuda", dtype=torch.float64)[None, :]
    py = case["res"] * torch.arange(case["H"], device="cuda", dtype=torch.float64)[:, None]
    v = verts.double().tolist()
    c = torch.zeros(case["H"], case["W"], device="cuda", dtype=torch.float64)
    for p, kind in enumerate(kinds):
        poly = v[offsets[p]:offsets[p + 1]]
        d2 = torch.full_like(c, math.inf)
        inside = torch.zeros_like(c, dtype=torch.bool)
        for (ax, ay), (bx, by) in zip(poly[-1:] + poly[:-1], poly):
            ex, ey = bx - ax, by - ay
            t = (((px - ax) * ex + (py - ay) * ey) / max(ex * ex + ey * ey, 1e-300)).clamp(0, 1)
            d2 = torch.minimum(d2, (ax + t * ex - px) ** 2 + (ay + t * ey - py) ** 2)
            if ay != by:
                inside ^= ((ay > py) != (by > py)) & (px < ax + (py - ay) * ex / ey)
        sd = torch.where(inside == (kind == 0), -d2.sqrt(), d2.sqrt())
        c += SIGMA_OBSTACLE * (1 - sd / EPS_OBSTACLE).clamp(min=0.0) ** 2
    return c


def _philox(case, seed, K):
    """Controls [N][2][K] of the generator that the library documents."""
    s, N = _spec(case, seed), case["N"]
    u = torch.zeros(N, 2, K, device="cuda", dtype=torch.float64)
    M0, M1 = 0xD2E7470EE14C6C93, 0xCA5A826395121157
    low = np.uint64(0xFFFFFFFF)

    def mul(m, c):  # high and low 64 bits of m * c
        mh, ml, s32 = np.uint64(m >> 32), np.uint64(m & 0xFFFFFFFF), np.uint64(32)
        ch, cl = c >> s32, c & low
        t = ml * cl
        mid = mh * cl + (t >> s32)
        mid2 = ml * ch + (mid & low)
        return mh * ch + (mid >> s32) + (mid2 >> s32), np.uint64(m) * c

    for blk in range((N + 3) // 4):
        c = [np.arange(K, dtype=np.uint64), np.full(K, blk, np.uint64), np.zeros(K, np.uint64), np.zeros(K, np.uint64)]
        k0, k1 = s["seed"], s["stream"]
        for _ in range(10):
            (h0, l0), (h1, l1) = mul(M0, c[0]), mul(M1, c[2])
            c = [h1 ^ c[1] ^ np.uint64(k0), l1, h0 ^ c[3] ^ np.uint64(k1), l0]
            k0, k1 = (k0 + 0x9E3779B97F4A7C15) % 2 ** 64, (k1 + 0xBB67AE8584CAA73B) % 2 ** 64
        for j in range(min(4, N - 4 * blk)):
            a = torch.from_numpy((c[j] >> np.uint64(40)).astype(np.float64)).cuda()
            b = torch.from_numpy(((c[j] >> np.uint64(16)) & np.uint64(0xFFFFFF)).astype(np.float64)).cuda()
            if s["kind"] == P.PLAN_SAMPLE_UNIFORM:
                za, zb = 2 * a / 2 ** 24 - 1, 2 * b / 2 ** 24 - 1
            else:
                r = torch.sqrt(-2 * torch.log((a + 1) / 2 ** 24))
                za, zb = r * torch.cos(2 * math.pi * b / 2 ** 24), r * torch.sin(2 * math.pi * b / 2 ** 24)
            u[4 * blk + j, 0], u[4 * blk + j, 1] = s["scale"][0] * za, s["scale"][1] * zb
    if s["keep"]:
        u[:, :, 0] = 0.0
    if s["nominal"] is not None:
        u += s["nominal"].double()[:, :, None]
    return u


def exact(case, seed):
    f64 = dict(device="cuda", dtype=torch.float64)
    if case["kind"] == "serve":
        reqs = _serve_requests(case, seed)
        maxN, best = max(u.shape[0] for *_, u in reqs), []
        ground = _Ground(torch.stack([h for h, *_ in reqs]), 0.1)
        cat = {q: [] for q in ("g", "s0", "u", "goal", "n")}
        for i, (_, s0, cost, u) in enumerate(reqs):
            N, _, K = u.shape
            cat["g"].append(torch.full((K,), i, device="cuda"))
            cat["n"].append(torch.full((K,), N, device="cuda"))
            cat["s0"].append(torch.tensor(s0, **f64)[:, None].expand(-1, K))
            cat["goal"].append(torch.tensor([cost["goal_x"], cost["goal_y"]], **f64)[:, None].expand(-1, K))
            cat["u"].append(torch.cat([u.double(), torch.zeros(maxN - N, 2, K, **f64)]))
        a = {q: torch.cat(v, -1) for q, v in cat.items()}
        J, _ = _rollout("srb", inputs.WORKLOAD_VEHICLE, inputs.BASE_COST, inputs.BASE_INTEG, ground,
                        a["g"], a["s0"], a["u"], a["goal"], a["n"])
        for i in range(len(reqs)):
            best.append(float(J[a["g"] == i].min()))
        return {"plans": None, "k": None, "J": np.array(best)}
    veh, cost, integ, h, s0 = _problem(case, seed)
    cm, out = None, {}
    if case["costmap"]:
        cm = _distance_cost(case, *_polygons(case, seed))
    if case["kind"] == "map":
        h = _smoothed(h, case["res"], case["sigma"])
        out = {"smooth": h, "costmap": cm}
    ground = _Ground(h[None], case["res"], None if cm is None else cm[None])
    s0 = torch.tensor(s0, **f64)
    goal = torch.tensor([cost["goal_x"], cost["goal_y"]], **f64)
    drawn = case["draws"] in ("uniform", "gauss")
    u = _philox(case, seed, case["K"]) if drawn else _candidates(case, seed, case["K"], case["N"]).double()
    if case["kind"] == "grad":
        u.requires_grad_(True)
        J, _ = _rollout("srb", veh, cost, integ, ground, 0, s0, u, goal)
        grad, = torch.autograd.grad(J[torch.isfinite(J)].sum(), u)
        return {"J": J.detach(), "grad": torch.where(torch.isfinite(J), grad, torch.zeros_like(grad))}
    J, st = _rollout(case["model"], veh, cost, integ, ground, 0, s0, u, goal)
    out["J"] = J
    if case["final"]:
        out["final"] = st
    if case["select"] == "argmin" and case["model"] != "est":
        out.update(plan=None, k=None, best=None)
    elif case["select"] == "softmin":
        w = torch.exp(-(J - J.min()) / LAMBDA)
        lim = torch.tensor([veh["delta_rate_max"], 1.0], **f64)[None, :, None]
        mean = (torch.maximum(torch.minimum(u, lim), -lim) * w).sum(-1) / w.sum()
        out.update(plan=mean, k=None, best=None)
    return out
