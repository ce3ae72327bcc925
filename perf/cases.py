"""The work that users of this library have it do, as cases that can be timed and checked.

A case is a dict of plain values.  `prepare` makes what a program holds before
the call (grids on the GPU, a plan, a batch, a server), `run` is one pass
through the public entry points, `work` its unavoidable traffic and arithmetic,
and `exact` the same result from plain torch operations in float64.

A sweep is run the way a time-stepping program runs it: the plan and the two
buffers are kept, and every pass continues from the state that the last one
left.
"""
import math
import random

import numpy as np
import torch

import paper_2001_01473_amd as s5d

DEVICE = "cuda:0"
TORCH = {"f32": torch.float32, "f64": torch.float64}

# Most cell updates times stencil points of a drawn case: far below the
# largest listed sweep's 1.3e12.
DRAW_TERMS = 1.0e11


def listed():
    return [
        # The smallest sweep in earnest: a 512^2 float64 Jacobi solve whose grid
        # stays in the caches, so launches and latency count.
        dict(name="star2d1r f64 512^2", kind="sweep", ndim=2, radius=1, box=False, dtype="f64",
             accum="plain", expr="linear", i0=512, i1=512, i2=0, steps=100),
        # The headline: the 5-point star at 16384^2 over 1000 steps.
        dict(name="star2d1r f32 16384^2", kind="sweep", ndim=2, radius=1, box=False, dtype="f32",
             accum="plain", expr="linear", i0=16384, i1=16384, i2=0, steps=1000),
        # A 25-point box in double precision on a ragged grid.
        dict(name="box2d2r f64 3001x5003", kind="sweep", ndim=2, radius=2, box=True, dtype="f64",
             accum="plain", expr="linear", i0=3001, i1=5003, i2=0, steps=100),
        # The 7-point star of heat and diffusion solvers at 512^3.
        dict(name="star3d1r f32 512^3", kind="sweep", ndim=3, radius=1, box=False, dtype="f32",
             accum="plain", expr="linear", i0=512, i1=512, i2=512, steps=100),
        # A 27-point box in double precision, ragged and mid-sized.
        dict(name="box3d1r f64 250x301x190", kind="sweep", ndim=3, radius=1, box=True, dtype="f64",
             accum="plain", expr="linear", i0=250, i1=301, i2=190, steps=60),
        # A high-order star one step per call: a wave solver that injects
        # sources or records receivers between the steps.
        dict(name="star3d4r f32 one step", kind="sweep", ndim=3, radius=4, box=False, dtype="f32",
             accum="plain", expr="linear", i0=420, i1=512, i2=483, steps=1),
        # Compensated float32 accumulation on a 13-point star.
        dict(name="star3d2r f32c 256^3", kind="sweep", ndim=3, radius=2, box=False, dtype="f32",
             accum="compensated", expr="linear", i0=256, i1=256, i2=256, steps=50),
        # The Jacobi program with a divisor (j2d5pt of the paper's Fig. 4).
        dict(name="j2d5pt f32 8000^2", kind="sweep", ndim=2, radius=1, box=False, dtype="f32",
             accum="plain", expr="div", i0=8000, i1=8000, i2=0, steps=100),
        # Heterogeneous media: per-cell weights of a 5-point star.
        dict(name="varcoef2d1r f32 4096x4000", kind="sweep", ndim=2, radius=1, box=False, dtype="f32",
             accum="plain", expr="varcoef", i0=4096, i1=4000, i2=0, steps=50),
        # An ensemble of uneven grids advanced together, replayed as a graph.
        dict(name="batch of 24 stars", kind="batch", n=24, lo=256, hi=2048, mix=1476, dtype="f32",
             steps=200, graph=True),
        # Mixed requests through the serving loop, from submission to results.
        dict(name="server, 12 requests", kind="server", n=12, lo2=512, hi2=2048, lo3=64, hi3=160,
             tlo=10, thi=200, mix=1477),
        # The accuracy check after a run: float32 result, float64 reference.
        dict(name="error norms f32/f64", kind="norms", n=512 * 512 * 257 + 3, got="f32", ref="f64"),
    ]


def draw(rng):
    kind = rng.choice(["sweep2", "sweep2", "sweep2", "sweep3", "sweep3", "sweep3", "expr", "expr",
                       "batch", "server", "norms"])

    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    if kind == "batch":
        lo = logint(64, 512)
        return dict(kind="batch", n=rng.randint(3, 32), lo=lo, hi=lo * rng.randint(2, 5), mix=rng.randrange(1 << 20),
                    dtype=rng.choice(["f32", "f32", "f64"]), steps=rng.randint(20, 200), graph=rng.random() < 0.5)
    if kind == "server":
        return dict(kind="server", n=rng.randint(3, 16), lo2=logint(200, 600), hi2=logint(700, 2500),
                    lo3=logint(32, 72), hi3=logint(90, 180), tlo=10, thi=logint(40, 200), mix=rng.randrange(1 << 20))
    if kind == "norms":
        return dict(kind="norms", n=logint(1000, 1.3e8), got=rng.choice(["f32", "f64"]), ref=rng.choice(["f32", "f64"]))
    case = dict(kind="sweep", ndim=2, radius=1, box=False, dtype=rng.choice(["f32", "f64"]), accum="plain",
                expr="linear")
    if kind == "expr":
        case["ndim"], case["radius"], case["box"], case["expr"] = rng.choice([
            (2, 1, False, "div"), (2, 2, False, "div"), (2, 1, True, "div"), (3, 1, True, "div"),
            (2, 1, False, "gradient"), (2, 1, False, "varcoef"), (2, 2, False, "varcoef"), (2, 1, True, "varcoef")])
    else:
        case["ndim"] = 2 if kind == "sweep2" else 3
        case["radius"] = rng.choice([1, 1, 2, 2, 3, 4])
        case["box"] = rng.random() < 0.5
        if case["dtype"] == "f32" and rng.random() < 0.25:
            case["accum"] = "compensated"
    lo, hi = (100, 9000) if case["ndim"] == 2 else (40, 512)
    i = [logint(lo, hi) for _ in range(case["ndim"])] + [0]
    case["i0"], case["i1"], case["i2"] = i[:3]
    points = _points(case)
    heavy = 8 if case["expr"] != "linear" or case["accum"] == "compensated" else 1
    most = DRAW_TERMS / (math.prod(v for v in i if v) * points * heavy)
    case["steps"] = max(1, min(int(most), rng.choice([1, logint(2, 30), logint(20, 300), logint(20, 300)])))
    return case


def _points(case):
    e = 2 * case["radius"] + 1
    return e ** case["ndim"] if case["box"] else 2 * case["radius"] * case["ndim"] + 1


def _interior(case):
    return tuple(case[k] for k in ("i0", "i1", "i2")[:case["ndim"]])


def _weights(case, seed):
    """The coefficients as the grid's type holds them: positive, the plain
    stencils' summing to about one."""
    u = np.random.default_rng(seed).random(_points(case))
    if case["expr"] == "div":
        c = np.append(u, u.sum())
    elif case["expr"] == "gradient":
        c = np.array([0.3, 1.5])
    elif case["expr"] == "varcoef":
        return None
    else:
        c = u / u.sum()
    return c.astype(np.float32).astype(np.float64) if case["dtype"] == "f32" else c


def _rand(shape, dtype, seed, k=0):
    gen = torch.Generator(device=DEVICE).manual_seed((seed * 1000003 + k) % (1 << 62))
    return torch.rand(shape, dtype=TORCH[dtype], device=DEVICE, generator=gen)


def _grid(case, seed, k=0):
    return _rand(tuple(i + 2 * case["radius"] for i in _interior(case)), case["dtype"], seed, k)


def _fields(case, seed):
    if case["expr"] != "varcoef":
        return None
    f = _rand((_points(case),) + _interior(case), case["dtype"], seed, 7)
    f /= f.sum(dim=0, keepdim=True)
    return f


def _plan(case, seed):
    return s5d.Plan(ndim=case["ndim"], radius=case["radius"], box=case["box"], dtype=case["dtype"],
                    interior=_interior(case), steps=case["steps"], coeffs=_weights(case, seed),
                    accum=case["accum"], expr=case["expr"])


def _members(case):
    """The sweeps of a batch or of a server's request stream, as cases."""
    r = random.Random(case["mix"])
    out = []
    for _ in range(case["n"]):
        m = dict(kind="sweep", accum="plain", expr="linear", box=False, i2=0)
        if case["kind"] == "batch":
            m.update(ndim=2, radius=r.randint(1, 2), dtype=case["dtype"], i0=r.randint(case["lo"], case["hi"]),
                     i1=r.randint(case["lo"], case["hi"]), steps=case["steps"])
        else:
            m.update(ndim=r.choice([2, 3]), radius=r.randint(1, 2), box=r.random() < 0.5,
                     dtype=r.choice(["f32", "f64"]), steps=r.randint(case["tlo"], case["thi"]))
            lo, hi = (case["lo2"], case["hi2"]) if m["ndim"] == 2 else (case["lo3"], case["hi3"])
            m["i0"], m["i1"] = r.randint(lo, hi), r.randint(lo, hi)
            if m["ndim"] == 3:
                m["i2"] = r.randint(lo, hi)
        out.append(m)
    return out


def prepare(case, seed):
    if case["kind"] == "norms":
        ref = _rand((case["n"],), "f64", seed)
        noise = _rand((case["n"],), "f64", seed, 1)
        got = ref * (1.0 + 1e-6 * (noise - 0.5))
        return dict(kind="norms", got=got.to(TORCH[case["got"]]), ref=ref.to(TORCH[case["ref"]]))
    if case["kind"] == "sweep":
        x = _grid(case, seed)
        return dict(kind="sweep", plan=_plan(case, seed), x=x, y=torch.empty_like(x), fields=_fields(case, seed))
    members = _members(case)
    grids = [_grid(m, seed, k) for k, m in enumerate(members)]
    plans = [_plan(m, seed + k) for k, m in enumerate(members)]
    other = [torch.empty_like(g) for g in grids]
    if case["kind"] == "batch":
        return dict(kind="batch", x=grids, y=other, init=[g.clone() for g in grids],
                    batch=s5d.Batch(plans, grids, other, graph=case["graph"]))
    return dict(kind="server", plans=plans, init=grids, out=other, server=s5d.Server(hbm_budget_bytes=16 << 30))


def run(state):
    if state["kind"] == "norms":
        return s5d.error_norms(state["got"], state["ref"])
    if state["kind"] == "sweep":
        idx = state["plan"].run(state["x"], state["y"], fields=state["fields"])
        if idx == 1:
            state["x"], state["y"] = state["y"], state["x"]
        return state["x"]
    if state["kind"] == "batch":
        # a batch is bound to its buffers: each pass starts from the members' initial states
        torch._foreach_copy_(state["x"], state["init"])
        return [(x, y)[i] for i, x, y in zip(state["batch"].run(), state["x"], state["y"])]
    server = state["server"]
    ids = [server.submit(p, g, keep_result=True) for p, g in zip(state["plans"], state["init"])]
    running, queued = server.tick()
    while running or queued:
        running, queued = server.tick()
    server.sync()
    for i, out in zip(ids, state["out"]):
        server.fetch(i, out)
    return state["out"]


def work(case):
    if case["kind"] == "norms":
        size = {"f32": 4, "f64": 8}
        return {"bytes": case["n"] * (size[case["got"]] + size[case["ref"]]), "flops": 5 * case["n"]}
    if case["kind"] != "sweep":
        parts = [work(m) for m in _members(case)]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    cells, points = math.prod(_interior(case)), _points(case)
    size = 4 if case["dtype"] == "f32" else 8
    words = 2 + (points if case["expr"] == "varcoef" else 0)
    per_cell = 19 if case["expr"] == "gradient" else 2 * points - 1 + (1 if case["expr"] == "div" else 0)
    if case["accum"] == "compensated":
        per_cell = 11 * points  # product, its error, the two-sum and the error sum of every term
    return {"bytes": cells * size * words, "flops": cells * per_cell * case["steps"]}


def _offsets(case):
    r, nd = case["radius"], case["ndim"]
    rng = range(-r, r + 1)
    every = [(a, b) for a in rng for b in rng] if nd == 2 else [(a, b, c) for a in rng for b in rng for c in rng]
    return every if case["box"] else [o for o in every if sum(1 for v in o if v) <= 1]


def _exact_sweep(case, seed, k=0, weights_seed=None):
    r, steps = case["radius"], case["steps"]
    interior = _interior(case)
    a = _grid(case, seed, k).double()
    b = a.clone()
    fields = _fields(case, seed)
    weights = _weights(case, seed if weights_seed is None else weights_seed)
    offsets = _offsets(case)

    def view(t, off):
        return t[tuple(slice(r + o, r + o + n) for o, n in zip(off, interior))]

    centre = (0,) * case["ndim"]
    for _ in range(steps):
        out = view(b, centre)
        if case["expr"] == "gradient":
            f = view(a, centre)
            s = torch.full_like(f, weights[1])
            for off in offsets:
                if off != centre:
                    s.add_((f - view(a, off)).square_())
            torch.add(s.sqrt_().reciprocal_(), f, alpha=weights[0], out=out)
        elif case["expr"] == "varcoef":
            torch.mul(view(a, offsets[0]), fields[0], out=out)
            for c, off in zip(fields[1:], offsets[1:]):
                out.addcmul_(view(a, off), c.double())
        else:
            torch.mul(view(a, offsets[0]), weights[0], out=out)
            for c, off in zip(weights[1:], offsets[1:]):
                out.add_(view(a, off), alpha=float(c))
            if case["expr"] == "div":
                out.div_(weights[-1])
        a, b = b, a
    return a


def exact(case, seed):
    if case["kind"] == "norms":
        s = prepare(case, seed)
        g, o = s["got"].double(), s["ref"].double()
        d = (g - o).abs()
        rel = torch.where(o != 0, d / o.abs(), d)
        return torch.stack([d.max(), o.abs().max(), rel.max(), d.square().mean().sqrt(), o.square().mean().sqrt()])
    if case["kind"] == "sweep":
        if math.prod(_interior(case)) * case["steps"] * _points(case) > 1e12:
            return None  # over 20 seconds of passes over memory
        return _exact_sweep(case, seed)
    return [_exact_sweep(m, seed, k, seed + k) for k, m in enumerate(_members(case))]
