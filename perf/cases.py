"""Timed calls of the FMM library: what programs that use it have it do.

A case is a dict of plain values.  ``prepare`` makes what the program holds
before the call (points, charges, the plan of a fixed point set), ``run`` is
one call through the package's public entry points, ``work`` counts the bytes
and operations the method cannot do without, ``exact`` is the direct sum in
64 bits.  Kinds of call:

* ``forward``   -- potentials (and fields) of one charge vector, cached plan
* ``graph``     -- the same, replayed from a captured HIP graph
* ``rebuild``   -- points that moved: new tree and lists, then one evaluation
* ``gradient``  -- the energy and its gradient in charges and positions
* ``vectors``   -- several charge vectors on one plan
* ``problems``  -- several independent problems in one plan
* ``probes``    -- charges and separate probe points: two charge vectors
  forward and their adjoint (one step of an inverse design)
* ``direct``    -- the direct sum at some of the points
"""
from __future__ import annotations

import math

import torch

import paper_2511_15269_amd as fmm

MAX_EXACT_PAIRS = 3.2e11  # direct-sum pairs that stay within a few seconds


def listed():
    return [
        # One gradient step of the active-shielding inverse design: 384
        # charges, 2048 probes.  The smallest calls; launches and latency.
        dict(name="shield_step", kind="probes", n=384, m=2048, p=8, leaf=16, splits=2,
             theta=0.6, precision="fp64"),
        # A small system inside a solver's loop, captured once and replayed.
        dict(name="cube4k_graph", kind="graph", dist="cube", n=4096, p=6, leaf=64, splits=2,
             theta=0.6, precision="fp64", field=True),
        # The paper's three-digit setting (potential only) on a surface of
        # ordinary size, the point count no power of two.
        dict(name="sphere30k_set1", kind="forward", dist="sphere", n=30011, p=5, leaf=128,
             splits=2, theta=0.7, precision="fp32", field=False),
        # Moving points: tree, lists and one pass for every step.
        dict(name="cube100k_rebuild", kind="rebuild", dist="cube", n=100003, p=8, leaf=128,
             splits=3, theta=0.8, precision="fp64", field=True),
        # The reference count of a sampled accuracy check: 8192 targets
        # against a million charges.
        dict(name="direct8k_of_1m", kind="direct", dist="cube", n=1 << 20, m=8192,
             precision="fp64", field=True),
        # The benchmark's pass: a million points, potential and field, FP64.
        dict(name="cube1m_fp64", kind="forward", dist="cube", n=1 << 20, p=8, leaf=128, splits=3,
             theta=0.8, precision="fp64", field=True),
        # Energy gradients of a gravity-like, strongly non-uniform set in FP32.
        dict(name="plummer200k_grad", kind="gradient", dist="plummer", n=200003, p=8, leaf=128,
             splits=3, theta=0.5, precision="fp32"),
        # One geometry, 32 charge vectors per pass.
        dict(name="cube256k_32vec", kind="vectors", dist="cube", n=1 << 18, vectors=32, p=8,
             leaf=128, splits=3, theta=0.8, precision="fp32", field=True),
        # Sixteen independent problems of uneven sizes in one plan.
        dict(name="uneven16", kind="problems", problems=16, lo=10000, hi=250000, sizes_seed=100,
             p=8, leaf=128, splits=3, theta=0.6, precision="fp32", field=True),
        # Clustered points at the highest order in FP32.
        dict(name="cluster500k_p10", kind="forward", dist="cluster", n=500009, p=10, leaf=128,
             splits=3, theta=0.7, precision="fp32", field=True),
        # The paper's six-digit setting (potential only).
        dict(name="cube524k_set2", kind="forward", dist="cube", n=524289, p=9, leaf=256, splits=2,
             theta=0.5, precision="fp32", field=False),
        # The paper's nine-digit setting (potential only, FP64).
        dict(name="cube262k_set3", kind="forward", dist="cube", n=1 << 18, p=10, leaf=256,
             splits=2, theta=0.27, precision="fp64", field=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges.  Separation parameters go with the
    order (looser ones at low order), as a user picks them for an accuracy."""
    kind = rng.choice(["forward", "forward", "forward", "graph", "rebuild", "gradient",
                       "vectors", "problems", "probes", "direct"])
    prec = rng.choice(["fp64", "fp32"])
    splits = rng.choice([1, 2, 3])
    leaf = rng.choice([32, 64, 100, 128, 256])
    p = rng.randint(4, 10)
    theta = round(rng.uniform(0.5, 0.8), 2)
    if kind == "direct":
        return dict(kind=kind, dist=rng.choice(["cube", "sphere"]), n=_log_int(rng, 4000, 1 << 20),
                    m=_log_int(rng, 100, 8000), precision=prec, field=rng.random() < 0.5)
    base = dict(kind=kind, p=p, splits=splits, leaf=leaf, theta=theta, precision=prec)
    if kind == "probes":
        return dict(base, n=_log_int(rng, 300, 20000), m=_log_int(rng, 1000, 60000),
                    leaf=rng.choice([16, 32, 64]))
    if kind == "problems":
        return dict(base, problems=rng.randint(2, 12), lo=3000, hi=100000,
                    sizes_seed=rng.randrange(1000), field=rng.random() < 0.7)
    if kind == "vectors":
        return dict(base, dist=rng.choice(["cube", "sphere"]), n=_log_int(rng, 4000, 130000),
                    vectors=rng.choice([2, 5, 16, 32]), precision="fp32", field=True)
    dist = rng.choice(["cube", "cube", "sphere", "cluster", "plummer"])
    base.update(dist=dist)
    if kind == "gradient":
        return dict(base, n=_log_int(rng, 4000, 100000))
    base.update(field=rng.random() < 0.6)
    if kind == "graph":
        return dict(base, n=_log_int(rng, 2000, 60000))
    if kind == "rebuild":
        return dict(base, n=_log_int(rng, 4000, 100000))
    top = 200000 if dist in ("plummer", "cluster") else 600000
    return dict(base, n=_log_int(rng, 2000, top))


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, dtype=torch.float64, device="cuda")


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, dtype=torch.float64, device="cuda")


def _directions(g, n):
    d = _randn(g, n, 3)
    return d / d.norm(dim=1, keepdim=True)


def _points(g, dist, n):
    """Points of a distribution and one vector of its charges."""
    if dist == "cube":
        return _rand(g, n, 3), 2.0 * _rand(g, n) - 1.0
    if dist == "sphere":
        return _directions(g, n), 2.0 * _rand(g, n) - 1.0
    if dist == "cluster":  # eight Gaussians and 5% of the points on a unit sphere
        centres = _rand(g, 8, 3)
        ns = n // 20
        shell = 0.5 + _directions(g, ns)
        lab = torch.randint(0, 8, (n - ns,), generator=g, device="cuda")
        pos = torch.cat([shell, centres[lab] + 0.01 * _randn(g, n - ns, 3)])
        return pos, torch.where(_rand(g, n) < 0.5, -1.0, 1.0).to(torch.float64)
    if dist == "plummer":  # scale 0.1, charges in (0, 1]
        u = _rand(g, n).clamp_min(1e-300)
        r = 0.1 / torch.sqrt(u ** (-2.0 / 3.0) - 1.0)
        return r[:, None] * _directions(g, n), 1.0 - _rand(g, n)
    raise KeyError(dist)


def _sizes(case):
    import random
    r = random.Random(case["sizes_seed"])
    return [_log_int(r, case["lo"], case["hi"]) for _ in range(case["problems"])]


def _spiral(n, radius):
    """n points spread evenly over a sphere (golden-angle spiral)."""
    k = torch.arange(n, dtype=torch.float64, device="cuda")
    z = 1.0 - (2.0 * k + 1.0) / n
    rho = torch.sqrt((1.0 - z * z).clamp_min(0.0))
    phi = k * (math.pi * (3.0 - math.sqrt(5.0)))
    return radius * torch.stack([rho * torch.cos(phi), rho * torch.sin(phi), z], dim=1)


def _inputs(case, seed):
    """Positions and charges in 64 bits (charges already rounded to the
    plan's precision), and the extra inputs of the kind."""
    g = _gen(seed)
    dt = _dtype(case)
    kind, extra = case["kind"], {}
    if kind == "probes":
        # a third of the charges regular on radius 2, the others random on
        # radius 5; probes even on radii 1.5 and 2.5
        ns = case["n"] // 3
        pos = torch.cat([_spiral(ns, 2.0), 5.0 * _directions(g, case["n"] - ns)])
        mi = case["m"] // 2
        extra["targets"] = torch.cat([_spiral(mi, 1.5), _spiral(case["m"] - mi, 2.5)])
        qa = 2.0 * _rand(g, case["n"]) - 1.0
        qb = qa.clone()
        qb[ns:] = 0.0
        q = torch.stack([qa, qb])
        extra["up"] = (2.0 * _rand(g, 2, case["m"]) - 1.0).to(dt)
    elif kind == "problems":
        sizes = _sizes(case)
        pos, q = _rand(g, sum(sizes), 3), 2.0 * _rand(g, sum(sizes)) - 1.0
        extra["sizes"] = sizes
    else:
        pos, q = _points(g, case["dist"], case["n"])
        if kind == "vectors":
            q = 2.0 * _rand(g, case["vectors"], case["n"]) - 1.0
        if kind == "direct":
            extra["at"] = torch.randperm(case["n"], generator=g, device="cuda")[: case["m"]]
    return pos, q.to(dt), extra


def _dtype(case):
    return torch.float64 if case["precision"] == "fp64" else torch.float32


def _plan(case, pos, extra):
    rhs = {"vectors": case.get("vectors", 1), "probes": 2}.get(case["kind"], 1)
    return fmm.Plan(pos, p=case["p"], leaf_max=case["leaf"], splits=case["splits"],
                    theta=case["theta"], precision=case["precision"], max_rhs=rhs,
                    sizes=extra.get("sizes"), targets=extra.get("targets"))


def prepare(case, seed):
    pos, q, extra = _inputs(case, seed)
    st = dict(case=case, pos=pos, q=q, **extra)
    if case["kind"] not in ("direct", "rebuild"):
        st["plan"] = _plan(case, pos, extra)
    if case["kind"] == "graph":
        st["graph"] = fmm.Graph(st["plan"], q, field=case["field"])
    return st


def run(st):
    case, q = st["case"], st["q"]
    kind = case["kind"]
    if kind == "direct":
        return fmm.direct(st["pos"], q, st["at"], field=case["field"])
    if kind == "rebuild":
        return _plan(case, st["pos"], {}).evaluate(q, field=case["field"])
    if kind == "graph":
        st["graph"].launch()
        return st["graph"].pot, st["graph"].field
    if kind == "probes":
        u, _ = st["plan"].evaluate(q, field=False)
        g, _ = st["plan"].adjoint(q, st["up"], None)
        return u, g
    if kind == "gradient":
        qq = q.detach().requires_grad_(True)
        xx = st["pos"].detach().requires_grad_(True)
        e = fmm.fmm_energy(st["plan"], qq, xx)
        gq, gx = torch.autograd.grad(e, (qq, xx))
        return e.detach(), gq, gx
    return st["plan"].evaluate(q, field=case["field"])


# ------------------------------------------------------------------ counts

def _m2l_flops(p):
    """One rotation-based multipole-to-local translation: two polar
    rotations and a shift along z, azimuthal rotations, rotation matrices."""
    rot = sum(2 * n * n + 2 * n + 1 for n in range(p + 1))
    return 6.0 * rot + 4 * p * (p + 1) + 4 * (p + 1) * (p + 2) * (2 * p + 3) // 6


def work(case):
    es = 8 if case["precision"] == "fp64" else 4
    kind = case["kind"]
    if kind == "direct":
        out = 4 if case["field"] else 1
        return {"bytes": float(case["n"] * (24 + es) + case["m"] * (8 + out * es)),
                "flops": (20.0 if case["field"] else 10.0) * case["n"] * case["m"]}
    pos, q, extra = _inputs(case, 0)
    info = _plan(case, pos, extra).info()
    n = pos.shape[0]
    m = case["m"] if kind == "probes" else n
    vec = q.shape[0] if q.dim() == 2 else 1
    with_field = kind == "gradient" or case.get("field", False)
    passes = 2 if kind in ("gradient", "probes") else 1
    K = (case["p"] + 1) ** 2
    flops = ((20.0 if with_field else 10.0) * info["p2p_interactions"]
             + _m2l_flops(case["p"]) * info["n_m2l"]
             + (6.0 * n + (8.0 if with_field else 2.0) * m) * K)
    out = 4 if with_field else 1
    moved = 24.0 * (n + (m if kind == "probes" else 0)) + vec * es * (n + out * m)
    return {"bytes": passes * moved, "flops": passes * vec * flops}


# ------------------------------------------------------------------- exact

def _direct(src, q, tgt, same, field):
    """-1/(4 pi) sum q/r at tgt for every row of q, and minus its gradient,
    in 64 bits; same[i] is the source that target i coincides with (or None).
    Few pairs are taken as differences, many through a matrix product."""
    n, m, R = src.shape[0], tgt.shape[0], q.shape[0]
    centre = src.mean(dim=0)
    src, tgt = src - centre, tgt - centre
    q = q.double()
    if field:  # q, q x, q y, q z side by side
        w = torch.cat([q[:, :, None], q[:, :, None] * src[None]], dim=2)
        w = w.permute(1, 0, 2).reshape(n, 4 * R)
    s2, t2 = (src * src).sum(1), (tgt * tgt).sum(1)
    qt, st = q.t().contiguous(), src.t().contiguous()
    u = torch.empty(m, R, dtype=torch.float64, device=src.device)
    f = torch.empty(m, R, 3, dtype=torch.float64, device=src.device) if field else None
    step = max(1, (1 << 28) // n)
    for a in range(0, m, step):
        b = min(m, a + step)
        if n * m <= 1.0e10:
            d = [tgt[a:b, c, None] - src[None, :, c] for c in range(3)]
            r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2]
        else:
            d = None
            r2 = torch.addmm(s2[None, :], tgt[a:b], st, alpha=-2.0).add_(t2[a:b, None])
        if same is not None:
            r2[torch.arange(b - a, device=src.device), same[a:b]] = math.inf
        inv = r2.rsqrt_()
        u[a:b] = inv @ qt
        if field and d is not None:
            inv.pow_(3)
            for c in range(3):
                f[a:b, :, c] = d[c].mul_(inv) @ qt
        elif field:
            s = (inv.pow_(3) @ w).reshape(b - a, R, 4)
            f[a:b] = s[:, :, :1] * tgt[a:b, None, :] - s[:, :, 1:]
    c = 1.0 / (4.0 * math.pi)
    # u = -c sum q/r, grad u = c sum q (x - x_j)/r^3, field = -grad u
    return -c * u.t(), (-c * f.permute(1, 0, 2) if field else None)


def exact(case, seed):
    kind = case["kind"]
    if kind == "problems":
        pairs = float(sum(s * s for s in _sizes(case)))
    elif kind in ("direct", "probes"):
        pairs = float(case["n"] * case["m"])
    else:
        pairs = float(case["n"] ** 2)
    if pairs > MAX_EXACT_PAIRS:
        return None
    pos, q, extra = _inputs(case, seed)
    field = kind == "gradient" or case.get("field", False)
    qq = q.double().reshape(-1, pos.shape[0])
    if kind == "probes":
        u, _ = _direct(pos, qq, extra["targets"], None, False)
        g, _ = _direct(extra["targets"], extra["up"].double(), pos, None, False)
        return u, g
    if kind == "problems":
        us, fs, o = [], [], 0
        for s in extra["sizes"]:
            x = pos[o:o + s]
            u, f = _direct(x, qq[:, o:o + s], x, torch.arange(s, device=x.device), field)
            us.append(u)
            fs.append(f)
            o += s
        return torch.cat(us, 1)[0], (torch.cat(fs, 1)[0] if field else None)
    at = extra["at"] if kind == "direct" else torch.arange(pos.shape[0], device=pos.device)
    u, f = _direct(pos, qq, pos[at], at, field)
    if kind == "gradient":  # E = 1/2 sum q u: dE/dq = u, dE/dx = q grad u
        return 0.5 * (qq[0] * u[0]).sum(), u[0], -qq[0][:, None] * f[0]
    if kind in ("vectors", "graph"):
        return u, f
    return u[0], (f[0] if field else None)
