"""The workloads that the performance of this framework is measured on.

A case is one call, or one short sequence of calls, that a program makes through the public
entry points (Plan, rollout_loss, Lattice). The kinds:

  run      a simulation: initial state, a number of steps, the moments (Plan.init/step/moments)
  annulus  the annular channel, walls and body force; equilibrium walls run a fixed number of
           steps, bounce-back walls run to the steady state with residual checks
  batch    many uneven clouds of one plan stepped together
  graph    build, initial state and steps of several clouds replayed as one HIP graph
  build    a plan from point coordinates and its first use: the interpolation operator (FP64),
           the first step (FP32) or a gradient through two steps (plans with the adjoint)
  grad     loss and gradient of a rollout on a plan in hand (checkpointed, or every state kept)
  lattice  the standard lattice Boltzmann method on a regular lattice

Clouds are lattices jittered by 0.3 spacings, and rings of jittered nodes for the annulus. What an
FP32 plan gives is kept in FP32, as its state is; what an FP64 plan gives stays FP64.
"""
import math
import random

import torch

from paper_2306_01525_amd import Params, Plan
from paper_2306_01525_amd.autograd import rollout_loss
from paper_2306_01525_amd.lbm import Lattice

DEVICE = "cuda"
EX = (0, 1, 0, -1, 0, 1, -1, -1, 1)
EY = (0, 0, 1, 0, -1, 1, 1, -1, -1)
WK = (4 / 9,) + (1 / 9,) * 4 + (1 / 36,) * 4
OPP = (0, 3, 4, 1, 2, 7, 8, 5, 6)
TWO_PI = 2.0 * math.pi


# ------------------------------------------------------------------------------- the cases
def listed():
    return [
        # the smallest workload: 1,600 nodes, own-node stencils, 200 steps. What a launch costs.
        dict(name="run_1600_f32", kind="run", nx=40, ny=40, K=12, degree=2, own=1, f64=0, tau=0.8, steps=200),
        # one point of a convergence study: FP64, 25 nodes with quadratic polynomials, h = 1/80
        dict(name="run_6400_f64", kind="run", nx=80, ny=80, K=25, degree=2, own=0, f64=1, tau=0.8, steps=100),
        # the Taylor-Green vortex at full size, FP32 and FP64
        dict(name="run_262144_f32", kind="run", nx=512, ny=512, K=30, degree=4, own=0, f64=0, tau=0.6, steps=20),
        dict(name="run_262144_f64", kind="run", nx=512, ny=512, K=30, degree=4, own=0, f64=1, tau=0.6, steps=10),
        # the annular channel: h = 1/40 with bounce-back walls, checked every 100 steps, and the
        # large FP32 channel with equilibrium walls
        dict(name="annulus_15k_bounce_f64", kind="annulus", rings=40, K=15, degree=2, f64=1, wall=2, tau=1.0, steps=200),
        dict(name="annulus_490k_f32", kind="annulus", rings=228, K=20, degree=3, f64=0, wall=1, tau=0.7, steps=20),
        # 64 clouds of 10,000 to 200,000 nodes stepped together
        dict(name="batch_64_f32", kind="batch", clouds=64, n_min=10000, n_max=200000, mix=4, steps=10),
        # serving: a handful of new clouds built, initialised and stepped in one graph launch
        dict(name="graph_8_f32", kind="graph", clouds=8, n_min=5000, n_max=60000, mix=9, steps=50),
        # a new cloud: its plan and first step, and a study's plan and interpolation
        dict(name="build_262144_f32", kind="build", nx=512, ny=512, K=30, degree=4, own=0, f64=0, adjoint=0, tau=0.6),
        dict(name="build_10201_f64", kind="build", nx=101, ny=101, K=25, degree=2, own=0, f64=1, adjoint=0, tau=0.8),
        # the gradient of a rollout with respect to the initial velocity and tau
        dict(name="grad_262144_f32", kind="grad", nx=512, ny=512, K=30, degree=4, own=0, f64=0, tau=0.6, steps=50,
             segment=25, keep=0),
        # the standard method on a large lattice
        dict(name="lattice_2048_f32", kind="lattice", nx=2048, ny=2048, f64=0, tau=0.6, steps=20),
    ]


# stencil size and polynomial degree as this repository's workloads, studies and tests use them
STENCILS = ((15, 2), (20, 2), (20, 3), (25, 2), (25, 3), (25, 4), (30, 4))


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _cloud(rng, n_max):
    n = _log(rng, 900, n_max)
    nx = max(24, int(math.sqrt(n * _log(rng, 0.7, 1.4))))
    ny = max(24, int(n / nx))
    own = int(rng.random() < 0.25)
    K, degree = rng.choice(((12, 2),) + STENCILS) if own else rng.choice(STENCILS[1:])
    return dict(nx=nx, ny=ny, K=K, degree=degree, own=own, f64=int(rng.random() < 0.5), tau=round(rng.uniform(0.6, 1.0), 3))


def draw(rng):
    kind = rng.choice(("run", "run", "run", "annulus", "annulus", "batch", "graph", "build", "build", "build", "grad", "lattice"))
    if kind == "run":
        c = dict(kind=kind, **_cloud(rng, 400000))
        c["steps"] = rng.randint(10, 60) if c["nx"] * c["ny"] < 50000 else rng.randint(5, 20)
        return c
    if kind == "annulus":
        rings, wall = int(_log(rng, 12, 220)), rng.choice((1, 2))
        K, degree = rng.choice(STENCILS[:4]) if wall == 2 else rng.choice(STENCILS[2:4])
        return dict(kind=kind, rings=rings, K=K, degree=degree, f64=int(rng.random() < 0.5), wall=wall,
                    tau=1.0 if wall == 2 else round(rng.uniform(0.7, 1.0), 3), steps=200 if rings < 60 and wall == 2 else rng.randint(10, 20))
    if kind in ("batch", "graph"):
        n_min = int(_log(rng, 1000, 20000))
        return dict(kind=kind, clouds=rng.randint(2, 24) if kind == "batch" else rng.randint(2, 10), n_min=n_min,
                    n_max=int(n_min * rng.uniform(2, 8)), mix=rng.randrange(1 << 20), steps=rng.randint(3, 20))
    if kind == "build":
        return dict(kind=kind, **_cloud(rng, 300000), adjoint=int(rng.random() < 0.4))
    if kind == "grad":
        return dict(kind=kind, **_cloud(rng, 200000), steps=rng.randint(6, 30), segment=rng.randint(3, 12), keep=int(rng.random() < 0.4))
    n = _log(rng, 400, 4000000)
    nx = max(17, int(math.sqrt(n * _log(rng, 0.4, 2.5))))
    return dict(kind=kind, nx=nx, ny=max(17, int(n / nx)), f64=int(rng.random() < 0.5), tau=round(rng.uniform(0.55, 1.0), 3),
                steps=rng.randint(10, 20) if n > 50000 else rng.randint(40, 120))


# ------------------------------------------------------------------------------ the inputs
def _gen(seed):
    return torch.Generator(device=DEVICE).manual_seed(int(seed))


def _uniform(g, n, lo, hi):
    return torch.rand(n, generator=g, device=DEVICE, dtype=torch.float64) * (hi - lo) + lo


def _lattice_cloud(nx, ny, g):
    """nx x ny nodes on [0, 2 pi) x [0, 2 pi ny / nx), jittered: x, y, period, spacing."""
    h = TWO_PI / nx
    lx, ly = TWO_PI, h * ny
    k = torch.arange(nx * ny, device=DEVICE)
    out = []
    for c, length in ((k % nx, lx), (k // nx, ly)):
        v = torch.remainder(c.double() * h + _uniform(g, nx * ny, -0.3 * h, 0.3 * h), length)
        out.append(torch.where(v >= length, v - length, v).contiguous())
    return out[0], out[1], (lx, ly), h


def _vortex(x, y, period, g):
    """A Taylor-Green vortex of speed 0.01 with a random phase, with another mode at a tenth of it."""
    p = _uniform(g, 4, 0.0, TWO_PI).tolist()
    kx, ky = TWO_PI / period[0], TWO_PI / period[1]
    u = 0.01 * torch.sin(kx * x + p[0]) * torch.cos(ky * y + p[1]) + 0.001 * torch.sin(2 * ky * y + p[2])
    v = -0.01 * torch.cos(kx * x + p[0]) * torch.sin(ky * y + p[1]) + 0.001 * torch.cos(3 * kx * x + p[3])
    return u, v


def _rings(rings, g):
    """Nodes between r = 1 and r = 2: `rings` + 1 circles, the first and the last of them the walls, with
    evenly spaced nodes at a random phase, those between the walls jittered by 0.2 spacings."""
    h = 1.0 / rings
    xs, ys = [], []
    phase = _uniform(g, rings + 1, 0.0, TWO_PI).tolist()
    count = [round(TWO_PI * (1.0 + j * h) / h) for j in range(rings + 1)]
    for j in [0, rings] + list(range(1, rings)):
        a = torch.arange(count[j], device=DEVICE, dtype=torch.float64) * (TWO_PI / count[j]) + phase[j]
        xs.append((1.0 + j * h) * torch.cos(a))
        ys.append((1.0 + j * h) * torch.sin(a))
    x, y = torch.cat(xs), torch.cat(ys)
    walls = count[0] + count[rings]
    for v in (x, y):
        v[walls:] += _uniform(g, v.numel() - walls, -0.2 * h, 0.2 * h)
    r = torch.hypot(x, y)
    kind = torch.zeros(x.numel(), dtype=torch.uint8, device=DEVICE)
    kind[:walls] = 1
    out = torch.where(r < 1.5, -1.0, 1.0).double() / r   # outward normal of the fluid domain
    return x, y, kind, (out * x).contiguous(), (out * y).contiguous(), h


def _mix(case):
    """Sizes and parameters of a batch's clouds: 20, 25 or 30 stencil nodes for degree 2, 3 or 4."""
    r = random.Random(case["mix"])
    out = []
    for _ in range(case["clouds"]):
        side = int(round(math.sqrt(_log(r, case["n_min"], case["n_max"]))))
        degree = r.randint(2, 4)
        out.append(dict(nx=side, ny=side, K={2: 20, 3: 25, 4: 30}[degree], degree=degree, tau=r.uniform(0.6, 1.0)))
    return out


def _batch_inputs(case, seed):
    g = _gen(seed)
    clouds, us, vs = [], [], []
    for c in _mix(case):
        x, y, period, h = _lattice_cloud(c["nx"], c["ny"], g)
        u, v = _vortex(x, y, period, g)
        clouds.append((x, y, period, h, c))
        us.append(u)
        vs.append(v)
    return clouds, us, vs


def _channel(case, h):
    """Streaming distance and force of the annulus: 1/160 and 1e-6 for bounce-back walls; the node spacing,
    and the force carried over to it, for equilibrium walls."""
    return (1.0 / 160.0, 1e-6) if case["wall"] == 2 else (h, 1e-6 * (160.0 * h) ** 3)


def _target(u, v, g):
    n = u.numel()
    noise = torch.randn(2, n, generator=g, device=DEVICE, dtype=torch.float64)
    return 0.9 * u + 1e-4 * noise[0], 0.9 * v + 1e-4 * noise[1]


def _params(case, h, **more):
    return Params(dx=h, K=case["K"], degree=case["degree"], tau=case["tau"], stencil_mode=case.get("own", 0),
                  precision=case["f64"], **more)


def _lattice_fields(case, g):
    k = torch.arange(case["nx"] * case["ny"], device=DEVICE)
    return _vortex((k % case["nx"]).double(), (k // case["nx"]).double(), (case["nx"], case["ny"]), g)


# ------------------------------------------------------------------------- preparing and running
def _tuned(plan, u, v):
    if plan.params.precision == 0:
        plan.autotune(plan.init(u, v), plan.new_state())
    return plan


def prepare(case, seed):
    kind, g = case["kind"], _gen(seed)
    if kind in ("run", "build", "grad"):
        x, y, period, h = _lattice_cloud(case["nx"], case["ny"], g)
        u, v = _vortex(x, y, period, g)
        adjoint = int(kind == "grad" or case.get("adjoint", 0))
        s = dict(case=case, x=x, y=y, period=period, u=u, v=v, params=_params(case, h, with_adjoint=adjoint))
        if adjoint:
            s["target"] = _target(u, v, g)
            kept = torch.float64 if case["f64"] else torch.float32   # what the program optimises
            s["u"], s["v"] = (t.to(kept).requires_grad_() for t in (u, v))
            s["tau"] = torch.tensor(case["tau"], dtype=torch.float64, device=DEVICE, requires_grad=True)
        if kind != "build":
            s["plan"] = Plan.build(x, y, period, s["params"])
            if kind == "run":
                _tuned(s["plan"], u, v)
                s["a"], s["b"] = s["plan"].new_state(), s["plan"].new_state()
        return s
    if kind == "annulus":
        x, y, walls, nx, ny, h = _rings(case["rings"], g)
        dx, force = _channel(case, h)
        plan = Plan.build(x, y, (0.0, 0.0), _params(case, dx, force_kind=1, force_mag=force, wall_kind=case["wall"]),
                          node_type=walls, normals=(nx, ny))
        u, v = _swirl(x, y, g)
        _tuned(plan, u, v)
        return dict(case=case, plan=plan, u=u, v=v, a=plan.new_state(), b=plan.new_state())
    if kind in ("batch", "graph"):
        clouds, us, vs = _batch_inputs(case, seed)
        args = [(x, y, period, None) for x, y, period, _, _ in clouds]
        params = [Params(dx=h, K=c["K"], degree=c["degree"], tau=c["tau"]) for _, _, _, h, c in clouds]
        u, v = torch.cat(us), torch.cat(vs)
        if kind == "batch":
            plan = _tuned(Plan.build_batch(args, params), u, v)
            return dict(case=case, plan=plan, u=u, v=v, a=plan.new_state(), b=plan.new_state())
        stream = torch.cuda.Stream()
        plan, a, b, result = Plan.build_graph(args, params, u, v, case["steps"], stream, variant=7)
        return dict(case=case, plan=plan, a=a, b=b, result=result, stream=stream)
    lat = Lattice(case["nx"], case["ny"], case["tau"], case["f64"])
    u, v = _lattice_fields(case, g)
    return dict(case=case, lat=lat, u=u, v=v, a=lat.new_state(), b=lat.new_state())


def _swirl(x, y, g):
    """A weak flow along the channel, at rest at the walls."""
    r = torch.hypot(x, y)
    a = _uniform(g, 2, 1e-3, 3e-3).tolist()
    s = (r - 1.0) * (2.0 - r) * (a[0] + a[1] * torch.cos(3.0 * torch.atan2(y, x)))
    return -s * y / r, s * x / r


def _fields(case, *t):
    """Fields as the program keeps them: an FP32 plan's in FP32, as its state."""
    return [v if case["f64"] else v.float() for v in t]


def _gradient(s, plan, steps, segment, keep):
    for t in (s["u"], s["v"], s["tau"]):
        t.grad = None
    J = rollout_loss(plan, s["u"].double(), s["v"].double(), s["tau"], steps, *s["target"], segment=segment, store_all=bool(keep))
    J.backward()
    return dict(loss=_fields(s["case"], J.detach())[0], du=s["u"].grad, dv=s["v"].grad,
                dtau=_fields(s["case"], s["tau"].grad)[0])


def run(state):
    s, case = state, state["case"]
    kind = case["kind"]
    if kind == "build":
        plan = Plan.build(s["x"], s["y"], s["period"], s["params"])
        if case["adjoint"]:
            return _gradient(s, plan, 2, 1, 0)
        if case["f64"]:
            return dict(values=plan.interpolate(s["u"]))
        out = plan.step(plan.init(s["u"], s["v"]), plan.new_state(), 1)
        return dict(fields=_fields(case, *plan.moments(out)), state=out)
    if kind == "grad":
        return _gradient(s, s["plan"], case["steps"], case["segment"], case["keep"])
    if kind == "graph":
        now = torch.cuda.current_stream()
        s["stream"].wait_stream(now)
        s["plan"].graph_launch(s["stream"])
        now.wait_stream(s["stream"])
        return dict(fields=[v.float() for v in s["plan"].moments(s["result"])], state=s["result"])
    if kind == "annulus" and case["wall"] == 2:
        out, _, residual, _ = s["plan"].run_to_steady(s["plan"].init(s["u"], s["v"], g=s["a"]), tol=1e-12,
                                                      check_every=case["steps"] // 2, max_steps=case["steps"] // 2 * 2)
        return dict(fields=_fields(case, *s["plan"].moments(out)), state=out, residual=residual)
    sim = s["lat"] if kind == "lattice" else s["plan"]
    out = sim.step(sim.init(s["u"], s["v"], g=s["a"]), s["b"], case["steps"])
    fields = sim.moments(out)
    return dict(fields=[v.float() for v in fields] if kind == "batch" else _fields(case, *fields), state=out)


# ------------------------------------------------------------------------------------ work
def _sizes(case):
    """(nodes, K, degree) of the case's clouds."""
    if case["kind"] in ("batch", "graph"):
        return [(c["nx"] * c["ny"], c["K"], c["degree"]) for c in _mix(case)]
    if case["kind"] == "annulus":
        h = 1.0 / case["rings"]
        return [(sum(round(TWO_PI * (1.0 + j * h) / h) for j in range(case["rings"] + 1)), case["K"], case["degree"])]
    return [(case["nx"] * case["ny"], case.get("K", 0), case.get("degree", 0))]


def _build_work(n, K, degree, elem):
    """Coordinates in; stencils, owners and weights out; a factorisation per node and eight solves."""
    N = K + (degree + 1) * (degree + 2) // 2
    return n * (16 + 4 * K + 32 + 8 * K * elem), n * (2.0 / 3.0 * N ** 3 + 8 * 2 * N * N)


def work(case):
    """Each step reads the weights, the stencil and owner indices and the state once and writes the state
    once (the weights of all but the smallest clouds do not stay on the chip from step to step)."""
    kind, elem = case["kind"], 8 if case.get("f64") else 4
    total, flops = 0.0, 0.0
    for n, K, degree in _sizes(case):
        if kind == "lattice":
            total += case["steps"] * n * 18 * elem + n * (16 + 24)
            flops += case["steps"] * n * 130
            continue
        step = n * (8 * K * elem + 4 * K + 18 * elem + (0 if case.get("own") else 32))
        step_flops = n * (16 * K + 130)
        back = n * (8 * K * (elem + 2) + 32 + 27 * elem)   # transposed weights, f, both adjoint states
        if kind in ("build", "graph"):
            b, f = _build_work(n, K, degree, elem)
            total, flops = total + b, flops + f
        if kind == "build":
            steps, reversed_steps = (2, 2) if case["adjoint"] else (1, 0)
        elif kind == "grad":
            # every state is needed again by the reversed steps: the checkpointed forms step twice
            steps, reversed_steps = case["steps"] * (1 if case["keep"] else 2), case["steps"]
        else:
            steps, reversed_steps = case["steps"], 0
        total += steps * step + reversed_steps * back + n * (16 + 24)
        flops += steps * step_flops + reversed_steps * n * (16 * K + 300)
    return {"bytes": total, "flops": flops}


# ------------------------------------------------------------- the same in 64 bits, plain torch
def _wrap(d, length):
    return d - length * torch.round(d / length) if length > 0 else d


def _nearest(px, py, x, y, period, K):
    """The K nodes closest to every point (px, py), nearest first: [points, K]. Candidates come from a grid
    of cells about two spacings wide, from the block of cells that holds every node within the K-th."""
    n = x.numel()
    lo = [0.0, 0.0] if period[0] > 0 else [float(x.min()), float(y.min())]
    ext = list(period) if period[0] > 0 else [float(x.max()) - lo[0] + 1e-9, float(y.max()) - lo[1] + 1e-9]
    area = ext[0] * ext[1] if period[0] > 0 else 3.0 * math.pi
    size = 2.0 * math.sqrt(area / n)
    nc = [max(1, int(e / size)) for e in ext]
    w = [e / c for e, c in zip(ext, nc)]
    reach = 3 if K > 1 else 2
    if period[0] > 0 and min(nc) < 2 * reach + 1:
        cand = None
    else:
        cell = lambda a, b: (((a - lo[0]) / w[0]).floor().long(), ((b - lo[1]) / w[1]).floor().long())  # noqa: E731
        cx, cy = cell(x, y)
        cid = cy.clamp(0, nc[1] - 1) * nc[0] + cx.clamp(0, nc[0] - 1)
        order = torch.argsort(cid, stable=True)
        count = torch.bincount(cid, minlength=nc[0] * nc[1])
        first = torch.cumsum(count, 0) - count
        cap = int(count.max())
        table = torch.full((nc[0] * nc[1] + 1, cap), n, device=DEVICE)
        table[cid[order], torch.arange(n, device=DEVICE) - first[cid[order]]] = order
        cand = True
    out = torch.empty(px.numel(), K, dtype=torch.long, device=DEVICE)
    for a in range(0, px.numel(), 16384):
        qx, qy = px[a:a + 16384], py[a:a + 16384]
        if cand is None:
            idx = torch.arange(n, device=DEVICE).expand(qx.numel(), n)
        else:
            qcx, qcy = cell(torch.remainder(qx, period[0]), torch.remainder(qy, period[1])) if period[0] > 0 else cell(qx, qy)
            o = torch.arange(-reach, reach + 1, device=DEVICE)
            ox, oy = (t.reshape(-1) for t in torch.meshgrid(o, o, indexing="ij"))
            bx, by = qcx[:, None] + ox, qcy[:, None] + oy
            if period[0] > 0:
                c = torch.remainder(by, nc[1]) * nc[0] + torch.remainder(bx, nc[0])
            else:
                c = torch.where((bx >= 0) & (bx < nc[0]) & (by >= 0) & (by < nc[1]), by * nc[0] + bx, nc[0] * nc[1])
            idx = table[c].reshape(qx.numel(), -1)
        near = idx.clamp(max=n - 1)
        d2 = _wrap(x[near] - qx[:, None], period[0]) ** 2 + _wrap(y[near] - qy[:, None], period[1]) ** 2
        d2 = torch.where(idx < n, d2, torch.inf)
        best = torch.topk(d2, K, dim=1, largest=False, sorted=True)
        if cand and float(best.values.max()) > (reach * min(w)) ** 2:
            raise ValueError("the search block is too small")
        out[a:a + 16384] = torch.gather(near, 1, best.indices)
    return out


def _monomials(x, y, degree):
    return torch.stack([x ** (d - j) * y ** j for d in range(degree + 1) for j in range(d + 1)], -1)


def _inverse(A):
    """Inverses of a batch of matrices by Gauss-Jordan elimination with partial pivoting."""
    B, N, _ = A.shape
    M = torch.cat([A, torch.eye(N, dtype=A.dtype, device=A.device).expand(B, N, N)], 2)
    at = torch.arange(B, device=A.device)
    for k in range(N):
        p = k + M[:, k:, k].abs().argmax(1)
        top = M[at, p]
        M[at, p] = M[:, k]
        top = top / top[:, k:k + 1]
        M -= M[:, :, k:k + 1] * top[:, None, :]
        M[:, k] = top
    return M[:, :, N:].contiguous()


def _operator(x, y, period, dx, K, degree, own):
    """Gather indices and weights of the streaming operator, [n, 8, K] each: the r^3 interpolant with
    polynomials on the stencil of the departure point's closest node (or of the node itself)."""
    n = x.numel()
    nbr = _nearest(x, y, x, y, period, K)
    if own:
        owner = torch.arange(n, device=DEVICE)[:, None].expand(n, 8)
    else:
        owner = torch.stack([_nearest(x - EX[k] * dx, y - EY[k] * dx, x, y, period, 1)[:, 0] for k in range(1, 9)], 1)
    sx = _wrap(x[nbr] - x[:, None], period[0])
    sy = _wrap(y[nbr] - y[:, None], period[1])
    rad = torch.hypot(sx, sy).amax(1)
    sx, sy = sx / rad[:, None], sy / rad[:, None]
    M = (degree + 1) * (degree + 2) // 2
    W = torch.empty(n, 8, K, dtype=torch.float64, device=DEVICE)
    phi = torch.zeros(n, K + M, K + M, dtype=torch.float64, device=DEVICE)
    inv = torch.empty_like(phi)
    for a in range(0, n, 32768):
        s = slice(a, a + 32768)
        phi[s, :K, :K] = torch.hypot(sx[s, :, None] - sx[s, None, :], sy[s, :, None] - sy[s, None, :]) ** 3
        phi[s, :K, K:] = _monomials(sx[s], sy[s], degree)
        phi[s, K:, :K] = phi[s, :K, K:].transpose(1, 2)
        inv[s] = _inverse(phi[s])
    for k in range(8):
        for a in range(0, n, 32768):
            s = slice(a, a + 32768)
            o = owner[s, k]
            qx = _wrap(x[s] - EX[k + 1] * dx - x[o], period[0]) / rad[o]
            qy = _wrap(y[s] - EY[k + 1] * dx - y[o], period[1]) / rad[o]
            b = torch.cat([torch.hypot(sx[o] - qx[:, None], sy[o] - qy[:, None]) ** 3, _monomials(qx, qy, degree)], 1)
            w = (inv[o] * b[:, None, :]).sum(2)
            w = w + (inv[o] * (b - (phi[o] * w[:, None, :]).sum(2))[:, None, :]).sum(2)
            W[s, k] = w[:, :K]
    return nbr[owner], W


def _feq(rho, u, v):
    uu = u * u + v * v
    e = [EX[k] * u + EY[k] * v for k in range(9)]
    return torch.stack([WK[k] * rho * (1 + 3 * e[k] + 4.5 * e[k] * e[k] - 1.5 * uu) for k in range(9)])


def _moments(f):
    rho = f.sum(0)
    return rho, sum(EX[k] * f[k] for k in range(9)) / rho, sum(EY[k] * f[k] for k in range(9)) / rho


def _collided(f, tau, force=None):
    out = f - (f - _feq(*_moments(f))) / tau
    if force is not None:
        out = out + torch.stack([3.0 * WK[k] * (EX[k] * force[0] + EY[k] * force[1]) for k in range(9)])
    return out


def _streamed(g, op):
    idx, W = op
    return torch.stack([g[0]] + [(W[:, k - 1] * g[k][idx[:, k - 1]]).sum(1) for k in range(1, 9)])


def _simulated(u, v, op, tau, steps):
    f = _feq(torch.ones_like(u), u, v)
    for _ in range(steps):
        f = _streamed(_collided(f, tau), op)
    return f


def _exact_gradient(case, seed, steps):
    g = _gen(seed)
    x, y, period, h = _lattice_cloud(case["nx"], case["ny"], g)
    u, v = _vortex(x, y, period, g)
    tx, ty = _target(u, v, g)
    op = _operator(x, y, period, h, case["K"], case["degree"], case["own"])
    if not case["f64"]:
        u, v = u.float().double(), v.float().double()
    u, v = u.requires_grad_(), v.requires_grad_()
    tau = torch.tensor(case["tau"], dtype=torch.float64, device=DEVICE, requires_grad=True)
    _, a, b = _moments(_simulated(u, v, op, tau, steps))
    J = 0.5 * ((a - tx) ** 2 + (b - ty) ** 2).sum()
    J.backward()
    return dict(loss=J.detach(), du=u.grad, dv=v.grad, dtau=tau.grad)


def _exact_annulus(case, seed):
    g = _gen(seed)
    x, y, walls, nx, ny, h = _rings(case["rings"], g)
    u, v = _swirl(x, y, g)
    dx, force = _channel(case, h)
    op = _operator(x, y, (0.0, 0.0), dx, case["K"], case["degree"], 0)
    r = torch.hypot(x, y)
    a = torch.stack([-force * y / r, force * x / r])
    wall = walls.bool()
    held = wall if case["wall"] == 1 else torch.zeros_like(wall)
    a[:, held] = 0.0
    enters = [wall & (EX[k] * nx + EY[k] * ny < 0.0) for k in range(9)]
    rest = _feq(torch.ones_like(x), 0.0 * x, 0.0 * x)
    f = torch.where(held, rest, _feq(torch.ones_like(x), u, v))
    steps = case["steps"] // 2 * 2 if case["wall"] == 2 else case["steps"]
    old = None
    for t in range(steps):
        f = _streamed(torch.where(held, rest, _collided(f, case["tau"], a)), op)
        if case["wall"] == 2:
            f = torch.stack([torch.where(enters[k], f[OPP[k]], f[k]) for k in range(9)])
        f = torch.where(held, rest, f)
        if t + 1 == steps // 2:
            old = torch.hypot(*_moments(f)[1:])
    m = _moments(f)
    out = dict(fields=list(m), state=None)
    if case["wall"] == 2:
        new = torch.hypot(*m[1:])
        out["residual"] = float((((new - old) ** 2).sum() / (new * new).sum()).sqrt())
    return out


def exact(case, seed):
    """What run() gives, in 64 bits. The states are in the plan's own node order and have no value here, but
    for the regular lattice's (an FP32 one holds the difference from rest)."""
    kind = case["kind"]
    if kind == "annulus":
        return _exact_annulus(case, seed)
    if kind == "grad" or (kind == "build" and case["adjoint"]):
        return _exact_gradient(case, seed, case["steps"] if kind == "grad" else 2)
    if kind in ("run", "build"):
        g = _gen(seed)
        x, y, period, h = _lattice_cloud(case["nx"], case["ny"], g)
        u, v = _vortex(x, y, period, g)
        op = _operator(x, y, period, h, case["K"], case["degree"], case["own"])
        if kind == "build" and case["f64"]:
            return dict(values=torch.stack([(op[1][:, k] * u[op[0][:, k]]).sum(1) for k in range(8)]))
        f = _simulated(u, v, op, case["tau"], case["steps"] if kind == "run" else 1)
        return dict(fields=list(_moments(f)), state=None)
    if kind in ("batch", "graph"):
        clouds, us, vs = _batch_inputs(case, seed)
        parts = []
        for (x, y, period, h, c), u, v in zip(clouds, us, vs):
            op = _operator(x, y, period, h, c["K"], c["degree"], 0)
            parts.append(_moments(_simulated(u, v, op, c["tau"], case["steps"])))
            del op
        return dict(fields=[torch.cat([p[i] for p in parts]) for i in range(3)], state=None)
    u, v = _lattice_fields(case, _gen(seed))
    nx, ny = case["nx"], case["ny"]
    f = _feq(torch.ones_like(u), u, v)
    for t in range(case["steps"]):
        g = f if t == 0 else _collided(f, case["tau"])   # the first collision leaves an equilibrium as it is
        f = torch.stack([torch.roll(g[k].view(ny, nx), (EY[k], EX[k]), (0, 1)).reshape(-1) for k in range(9)])
    state = _collided(f, case["tau"])
    if not case["f64"]:
        state = state - torch.tensor(WK, dtype=torch.float64, device=DEVICE)[:, None]
    return dict(fields=list(_moments(f)), state=state.reshape(-1))
