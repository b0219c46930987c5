"""The work this library is timed on: one case per form of use, from the
smallest call to the largest.

``listed()`` names the cases, ``draw(rng)`` gives further ones of the same
ranges, ``prepare``/``run`` make a program's state and one pass through the
public entry points, ``work`` counts what a pass cannot do without, ``exact``
gives the same results in plain 64-bit torch where that is affordable.

Inputs are drawn on the GPU from the seed alone, with the distributions of
``workloads.py`` (uniform square and cube, jittered Lamb-Oseen lattice,
Gaussian mixture).  Plans keep their default launch shapes.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_0905_2637_amd as fm

DEVICE = "cuda"
# direct sums up to this many pairs are affordable in plain torch
MOST_PAIRS = 6.0e10


def listed():
    return [
        # One small evaluation (a few thousand vortex particles, the size of a
        # quick study or of one member of an ensemble): launch latency.
        dict(name="small_4k", form="particles", dist="uniform", n=4096, depth=4, p=12, sigma=0.005,
             precision="fp64", kernel="gaussian"),
        # Point vortices (singular kernel), an odd count that fills no tile.
        dict(name="point_vortices_100k", form="particles", dist="uniform", n=100_003, depth=5, p=12, sigma=0.0,
             precision="fp64", kernel="singular"),
        # The allocation-free call of a serving loop, an odd count.
        dict(name="static_200k", form="static", dist="uniform", n=200_003, depth=6, p=17, sigma=0.004,
             precision="fp64", kernel="gaussian"),
        # The usual vortex-method evaluation: a million particles of a vortex
        # on a jittered lattice, FP64.
        dict(name="vortex_1m", form="particles", dist="lattice", n=1 << 20, depth=8, p=17, sigma=0.002,
             precision="fp64", kernel="gaussian"),
        # Clustered particles (very uneven leaves) in mixed precision.
        dict(name="clusters_4m_mixed", form="particles", dist="mixture", n=1 << 22, depth=9, p=17, sigma=0.001,
             precision="mixed", kernel="gaussian"),
        # The largest run: 2^26 particles, FP64.
        dict(name="uniform_64m", form="particles", dist="uniform", n=1 << 26, depth=11, p=20, sigma=2e-4,
             precision="fp64", kernel="gaussian"),
        # The velocity field of a vortex probed on a lattice of points.
        dict(name="probe_1m", form="points", dist="lattice", n=1 << 20, m=1 << 20, depth=8, p=17, sigma=0.002,
             precision="fp64", kernel="gaussian"),
        # Many independent problems of uneven size in one call, mixed.
        dict(name="batch_512_mixed", form="batch", instances=512, low=2048, high=65536, sizes=4, p=12, sigma=0.005,
             precision="mixed", kernel="gaussian"),
        # Vortex-method time stepping on the particles' bounding square.
        dict(name="steps_1m", form="steps", dist="lattice", n=1 << 20, depth=8, p=17, sigma=0.002,
             precision="fp64", kernel="gaussian", steps=2),
        # Lennard-Jones forces of a dense two-dimensional fluid.
        dict(name="lennard_jones_1m", form="lj", n=1 << 20, depth=8),
        # The fast Gauss transform of a million sources.
        dict(name="gauss_1m", form="gauss", dist="lattice", n=1 << 20, depth=6, p=12, sigma=0.02),
        # The three-dimensional Laplace form, a million charges.
        dict(name="octree_1m", form="octree", n=1 << 20, depth=5, p=6),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    form = rng.choice(["particles", "particles", "mixed", "singular", "static", "points", "batch", "steps", "lj",
                       "gauss", "octree", "octree"])
    per_leaf = _log(rng, 8, 48)
    depth_of = lambda n: max(2, min(11, int(round(math.log(max(1.0, n / per_leaf), 4)))))  # noqa: E731
    sigma_of = lambda d: round(2.0 ** -d * rng.uniform(0.08, 0.5), 6)  # noqa: E731  core against leaf width
    if form in ("particles", "mixed", "singular"):
        n = _log(rng, 2000, 1 << 24)
        d = depth_of(n)
        mixed = form == "mixed"
        return dict(form="particles", dist=rng.choice(["uniform", "uniform", "mixture"]) if n < (1 << 22) else "uniform",
                    n=n, depth=d, p=rng.randint(8, 20 if mixed else 24), sigma=sigma_of(d),
                    precision="mixed" if mixed else "fp64", kernel="singular" if form == "singular" else "gaussian")
    if form == "static":
        n = _log(rng, 2000, 200_000)
        d = min(6, depth_of(n))
        return dict(form="static", dist="uniform", n=n, depth=d, p=rng.randint(8, 17), sigma=sigma_of(d),
                    precision=rng.choice(["fp64", "mixed"]), kernel="gaussian")
    if form == "points":
        n = _log(rng, 2000, 1 << 21)
        d = depth_of(n)
        return dict(form="points", dist=rng.choice(["uniform", "mixture"]), n=n, m=_log(rng, 1000, 1 << 21), depth=d,
                    p=rng.randint(8, 20), sigma=sigma_of(d), precision="fp64", kernel="gaussian")
    if form == "batch":
        low = _log(rng, 256, 8192)
        return dict(form="batch", instances=_log(rng, 8, 256), low=low, high=low * rng.randint(2, 16),
                    sizes=rng.randrange(1 << 20), p=rng.randint(8, 17), sigma=0.005,
                    precision=rng.choice(["fp64", "mixed"]), kernel="gaussian")
    if form == "steps":
        side = _log(rng, 64, 1200)
        d = max(2, int(round(math.log(side * side / 16.0, 4))))
        return dict(form="steps", dist="lattice", n=side * side, depth=d, p=rng.randint(8, 20),
                    sigma=round(2.0 / side, 6), precision="fp64", kernel="gaussian", steps=rng.randint(1, 3))
    if form == "lj":
        side = _log(rng, 64, 1500)
        return dict(form="lj", n=side * side, depth=max(1, int(math.floor(math.log2(side / 2.6)))))
    if form == "gauss":
        n = _log(rng, 2000, 1 << 21)
        d = rng.randint(3, 6)
        return dict(form="gauss", dist="uniform", n=n, depth=d, p=rng.randint(8, 16),
                    sigma=round(2.0 ** -d * rng.uniform(0.8, 1.6), 6))
    depth = rng.randint(2, 5)
    n = min(1 << 20, int(8 ** depth * _log(rng, 8, 48)))
    return dict(form="octree", n=max(2000, n - rng.randrange(1, 500)), depth=depth, p=rng.randint(3, 7 if depth == 5 else 9))


# ---- inputs ------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device=DEVICE).manual_seed(int(seed))


def _rand(gen, n, lo=0.0, hi=1.0):
    return torch.rand(n, dtype=torch.float64, device=DEVICE, generator=gen) * (hi - lo) + lo


def _uniform(gen, n):
    """Positions uniform in the unit square, circulations U(-1, 1)."""
    x = _rand(gen, n)
    y = _rand(gen, n)
    return x, y, _rand(gen, n, -1.0, 1.0)


def _lattice(gen, n, core=0.1):
    """A Lamb-Oseen vortex on a jittered cell-centred lattice (n a square)."""
    side = math.isqrt(n)
    h = 1.0 / side
    c = (torch.arange(side, dtype=torch.float64, device=DEVICE) + 0.5) * h
    y, x = torch.meshgrid(c, c, indexing="ij")
    x = x.reshape(-1) + _rand(gen, n, -0.25 * h, 0.25 * h)
    y = y.reshape(-1) + _rand(gen, n, -0.25 * h, 0.25 * h)
    r2 = (x - 0.5) ** 2 + (y - 0.5) ** 2
    return x, y, h * h / (math.pi * core * core) * torch.exp(-r2 / (core * core))


def _mixture(gen, n, components=16):
    """An equal-weight Gaussian mixture in the unit square (means and widths
    the same for every seed), circulations N(0, 1), in random order."""
    fixed = np.random.default_rng(3)
    means = torch.as_tensor(fixed.random((components, 2)), device=DEVICE)
    stds = torch.as_tensor(fixed.uniform(0.01, 0.1, components), device=DEVICE)
    comp = torch.randint(components, (n,), device=DEVICE, generator=gen)
    xy = torch.full((n, 2), -1.0, dtype=torch.float64, device=DEVICE)
    while True:
        out = ((xy < 0.0) | (xy >= 1.0)).any(dim=1).nonzero().reshape(-1)
        if out.numel() == 0:
            break
        c = comp[out]
        z = torch.randn((out.numel(), 2), dtype=torch.float64, device=DEVICE, generator=gen)
        xy[out] = z * stds[c].unsqueeze(1) + means[c]
    g = torch.randn(n, dtype=torch.float64, device=DEVICE, generator=gen)
    return xy[:, 0].contiguous(), xy[:, 1].contiguous(), g


def _batch_sizes(case):
    r = np.random.default_rng(case["sizes"])
    counts = np.rint(np.exp(r.uniform(math.log(case["low"]), math.log(case["high"]), case["instances"]))).astype(int)
    depths = [max(2, int(math.floor(math.log(c / 64.0, 4.0) + 0.5))) for c in counts]
    return [int(c) for c in counts], depths


def _lj_length(case):
    return 1.0 / math.isqrt(case["n"]) / 1.12


def _inputs(case, seed):
    """The arrays a program holds before the call (x, y, gamma, then what the form adds)."""
    gen = _gen(seed)
    form = case["form"]
    if form == "octree":
        n = case["n"]
        return tuple(_rand(gen, n) for _ in range(3)) + (_rand(gen, n, -1.0, 1.0),)
    if form == "batch":
        return _uniform(gen, sum(_batch_sizes(case)[0]))
    if form == "lj":
        n = case["n"]
        side = math.isqrt(n)
        a = 1.0 / side
        c = (torch.arange(side, dtype=torch.float64, device=DEVICE) + 0.5) * a
        y, x = torch.meshgrid(c, c, indexing="ij")
        return (x.reshape(-1) + _rand(gen, n, -0.2 * a, 0.2 * a), y.reshape(-1) + _rand(gen, n, -0.2 * a, 0.2 * a),
                torch.zeros(n, dtype=torch.float64, device=DEVICE))
    arrays = {"uniform": _uniform, "lattice": _lattice, "mixture": _mixture}[case["dist"]](gen, case["n"])
    if form == "points":
        if case["dist"] == "lattice":     # a vertex lattice: every leaf edge carries points
            side = math.isqrt(case["m"])
            c = torch.arange(side, dtype=torch.float64, device=DEVICE) / side
            ty, tx = torch.meshgrid(c, c, indexing="ij")
            return arrays + (tx.reshape(-1).contiguous(), ty.reshape(-1).contiguous())
        return arrays + (_rand(gen, case["m"]), _rand(gen, case["m"]))
    return arrays


# ---- one pass ----------------------------------------------------------------

def prepare(case, seed):
    arrays = _inputs(case, seed)
    form, n = case["form"], int(arrays[0].shape[0])
    st = {"case": case, "in": arrays}
    if form == "octree":
        st["plan"] = fm.Plan3D(n, case["p"], case["depth"])
        st["out"] = tuple(torch.empty(n, dtype=torch.float64, device=DEVICE) for _ in range(4))
        return st
    m = case.get("m", n)
    st["out"] = tuple(torch.empty(m, dtype=torch.float64, device=DEVICE) for _ in range(2))
    if form in ("particles", "points"):
        st["plan"] = fm.Plan(n, case["sigma"], case["p"], case["depth"], precision=case["precision"],
                             kernel=case["kernel"], fp32_fine_levels=min(2, case["depth"] - 1),
                             m_max=m if form == "points" else 0)
    elif form == "batch":
        counts, depths = _batch_sizes(case)
        st["plan"] = fm.BatchPlan(counts, depths, case["sigma"], case["p"], precision=case["precision"],
                                  fp32_fine_levels=min(2, max(depths) - 1), kernel=case["kernel"])
    elif form == "steps":
        st["plan"] = fm.Plan(n, case["sigma"], case["p"], case["depth"], domain=None)
        st["scratch"] = torch.empty(4 * n, dtype=torch.float64, device=DEVICE)
    elif form == "lj":
        s = _lj_length(case)
        st["plan"] = fm.Plan(n, s, 8, case["depth"], kernel="lennard-jones", lj_epsilon=1.0, cutoff=2.5 * s)
    elif form == "gauss":
        st["plan"] = fm.Plan(n, case["sigma"], case["p"], case["depth"], kernel="gauss-transform")
    return st


def run(state):
    case, a, out = state["case"], state["in"], state["out"]
    form = case["form"]
    if form == "static":
        return fm.evaluate_static(*a, case["sigma"], case["p"], case["depth"], precision=case["precision"],
                                  fp32_fine_levels=min(2, case["depth"] - 1), kernel=case["kernel"], u=out[0],
                                  v=out[1])
    plan = state["plan"]
    if form == "octree":
        return plan.evaluate(*a, out=out, check=False)
    if form == "points":
        return plan.evaluate_at(*a, u=out[0], v=out[1], check=False)
    if form == "steps":
        return plan.advance_rk2(*a, 1e-4, case["steps"], scratch=state["scratch"])
    return plan.evaluate(*a, u=out[0], v=out[1], check=False)


# ---- what a pass cannot do without ---------------------------------------------

def _far_flops(n, m, depth, p):
    """P2M, M2M, M2L (8 p^2 per list pair), L2L, L2P of one quadtree."""
    boxes = sum(4 ** l for l in range(2, depth + 1))
    pairs = sum(3 * (2 ** l - 2) * (9 * 2 ** l - 10) for l in range(2, depth + 1))
    return 8.0 * p * (n + m) + 4.0 * p * p * boxes + 8.0 * p * p * pairs


def work(case):
    form = case["form"]
    n = case.get("n", 0)
    if form == "octree":
        T = (case["p"] + 1) * (case["p"] + 2) * (case["p"] + 3) // 6
        # harmonic expansions of degree p carry (p + 1)^2 independent terms
        side = 2 ** case["depth"]
        near = n * (n / side ** 3) * ((3 * side - 2) / side) ** 3
        H = (case["p"] + 1) ** 2
        pairs = 0.0
        for l in range(2, case["depth"] + 1):
            s = 2 ** l
            pairs += (6.0 * s / 2 * 2 - 8) ** 3 - (3.0 * s - 2) ** 3
        return {"bytes": 64.0 * n, "flops": 16.0 * near + 2.0 * H * H * pairs + 10.0 * T * n}
    if form == "gauss":
        # two separable passes over the box range, p^2 terms per particle
        w = 2.0 ** -case["depth"]
        nc = min(2 ** case["depth"] - 1, math.ceil(math.sqrt(math.log(1e16)) * math.sqrt(2.0) * case["sigma"] / w))
        boxes = 4 ** case["depth"]
        return {"bytes": 40.0 * n, "flops": 4.0 * n * case["p"] ** 2 + 4.0 * (2 * nc + 1) * boxes * case["p"] ** 3}
    if form == "lj":
        return {"bytes": 32.0 * n, "flops": 14.0 * n * math.pi * 2.5 ** 2 / 1.12 ** 2}
    if form == "batch":
        counts, depths = _batch_sizes(case)
        return {"bytes": 40.0 * sum(counts),
                "flops": sum(14.0 * c * c * ((3 * 2 ** d - 2) / 4 ** d) ** 2 + _far_flops(c, c, d, case["p"])
                             for c, d in zip(counts, depths))}
    m = case.get("m", n)
    d = case["depth"]
    evals = 2 * case["steps"] if form == "steps" else 1
    near = 14.0 * n * m * ((3 * 2 ** d - 2) / 4 ** d) ** 2
    return {"bytes": evals * (24.0 * n + 16.0 * m + (16.0 * m if form == "points" else 0.0)),
            "flops": evals * (near + _far_flops(n, m, d, case["p"]))}


# ---- the same in plain 64-bit torch ----------------------------------------------

def _leaf(x, y, x0, y0, width, depth):
    side = 2 ** depth
    s = side / width
    return (((x - x0) * s).floor().clamp(0, side - 1), ((y - y0) * s).floor().clamp(0, side - 1))


def _split_sum(x, y, g, tx, ty, sigma, depth, x0=0.0, y0=0.0, width=1.0):
    """sum_j gamma_j K(t - x_j): the Gaussian kernel where the leaves touch, the
    singular one elsewhere (sigma = 0: the singular kernel everywhere)."""
    n, m = x.shape[0], tx.shape[0]
    u = torch.empty(m, dtype=torch.float64, device=x.device)
    v = torch.empty_like(u)
    lx, ly = _leaf(x, y, x0, y0, width, depth)
    rows = max(1, int(1.5e8 // max(1, n)))
    for a in range(0, m, rows):
        b = min(m, a + rows)
        dx = tx[a:b, None] - x[None]
        dy = ty[a:b, None] - y[None]
        r2 = dx * dx + dy * dy
        f = torch.where(r2 > 0.0, 1.0 / r2, 0.0)
        if sigma > 0.0:
            kx, ky = _leaf(tx[a:b], ty[a:b], x0, y0, width, depth)
            touch = ((kx[:, None] - lx[None]).abs() <= 1) & ((ky[:, None] - ly[None]).abs() <= 1)
            f = torch.where(touch, f * -torch.expm1(r2 * (-0.5 / (sigma * sigma))), f)
        f *= g[None]
        u[a:b] = -(f * dy).sum(1) / (2.0 * math.pi)
        v[a:b] = (f * dx).sum(1) / (2.0 * math.pi)
    return u, v


def _exact_lj(case, x, y):
    """Forces by a cell list of the cutoff's width, padded to the fullest cell."""
    s = _lj_length(case)
    rc = 2.5 * s
    n, side = x.shape[0], max(1, int(math.floor(1.0 / rc)))
    cx, cy = ((c * side).floor().clamp(0, side - 1).long() for c in (x, y))
    order = torch.argsort(cy * side + cx, stable=True)
    count = torch.bincount(cy * side + cx, minlength=side * side)
    start = count.cumsum(0) - count
    fx, fy = torch.zeros_like(x), torch.zeros_like(x)
    for ay in (-1, 0, 1):
        for ax in (-1, 0, 1):
            ok = (cx + ax >= 0) & (cx + ax < side) & (cy + ay >= 0) & (cy + ay < side)
            cell = ((cy + ay) * side + cx + ax).clamp(0, side * side - 1)
            for k in range(int(count.max())):
                have = ok & (k < count[cell])
                j = order[(start[cell] + k).clamp(max=n - 1)]
                dx, dy = x - x[j], y - y[j]
                r2 = dx * dx + dy * dy
                use = have & (r2 > 0.0) & (r2 < rc * rc)
                q = (s * s / torch.where(use, r2, 1.0)) ** 3
                f = torch.where(use, 24.0 * q * (2.0 * q - 1.0) / torch.where(use, r2, 1.0), 0.0)
                fx += f * dx
                fy += f * dy
    return fx, fy


def _exact_gauss(case, x, y, g):
    """The plain sum over the sources within the range at which a term falls
    below 1e-17 of its strength, by strips of target rows and columns."""
    sigma = case["sigma"]
    reach = math.sqrt(2.0 * math.log(1e17)) * sigma
    strips = max(1, min(48, int(1.0 / (0.5 * reach))))
    row = (y * strips).floor().clamp(0, strips - 1).long()
    out = torch.zeros_like(x)
    for r in range(strips):
        near = ((y >= r / strips - reach) & (y < (r + 1) / strips + reach)).nonzero().reshape(-1)
        mine = (row == r).nonzero().reshape(-1)
        col = (x[mine] * strips).floor().clamp(0, strips - 1).long()
        for c in range(strips):
            t = mine[col == c]
            if t.numel() == 0:
                continue
            s = near[(x[near] >= c / strips - reach) & (x[near] < (c + 1) / strips + reach)]
            sx, sy, sg = x[s], y[s], g[s]
            rows = max(1, int(1e8 // max(1, s.numel())))
            for a in range(0, t.numel(), rows):
                k = t[a:a + rows]
                dx = x[k][:, None] - sx[None]
                dy = y[k][:, None] - sy[None]
                out[k] = (torch.exp((dx * dx + dy * dy) * (-0.5 / (sigma * sigma))) * sg[None]).sum(1)
    return out, torch.zeros_like(out)


def _exact_octree(x, y, z, q):
    n = x.shape[0]
    out = tuple(torch.empty_like(x) for _ in range(4))
    rows = max(1, int(1.5e8 // n))
    for a in range(0, n, rows):
        b = min(n, a + rows)
        d = [c[a:b, None] - c[None] for c in (x, y, z)]
        r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2]
        ir = torch.where(r2 > 0.0, 1.0 / torch.sqrt(r2), 0.0)
        qr = q[None] * ir
        out[0][a:b] = qr.sum(1)
        qr *= ir * ir
        for k in range(3):
            out[1 + k][a:b] = -(qr * d[k]).sum(1)
    return out


def exact(case, seed):
    a = _inputs(case, seed)
    form, n = case["form"], int(a[0].shape[0])
    if form == "lj":
        return _exact_lj(case, a[0], a[1])
    if form == "gauss":
        reach = 8.85 * case["sigma"]
        share = min(1.0, 2.5 * reach) ** 2
        return _exact_gauss(case, *a) if n * n * share <= 2.5e11 else None
    if form == "octree":
        return _exact_octree(*a) if float(n) * n <= MOST_PAIRS else None
    if form == "batch":
        counts, depths = _batch_sizes(case)
        if sum(float(c) * c for c in counts) > MOST_PAIRS:
            return None
        parts, at = [], 0
        for c, d in zip(counts, depths):
            x, y, g = (t[at:at + c] for t in a)
            parts.append(_split_sum(x, y, g, x, y, case["sigma"], d))
            at += c
        return tuple(torch.cat([q[k] for q in parts]) for k in range(2))
    if form == "steps":
        if float(n) * n * 2 * case["steps"] > MOST_PAIRS:
            return None
        x, y, g = a

        def velocity(px, py):
            x0, y0 = float(px.min()), float(py.min())
            w = max(float(px.max()) - x0, float(py.max()) - y0)
            return _split_sum(px, py, g, px, py, case["sigma"], case["depth"], x0, y0, w)

        for _ in range(case["steps"]):
            u, v = velocity(x, y)
            u, v = velocity(x + 0.5e-4 * u, y + 0.5e-4 * v)
            x, y = x + 1e-4 * u, y + 1e-4 * v
        return x, y
    tx, ty = (a[3], a[4]) if form == "points" else (a[0], a[1])
    if float(n) * tx.shape[0] > MOST_PAIRS:
        return None
    return _split_sum(a[0], a[1], a[2], tx, ty, 0.0 if case["kernel"] == "singular" else case["sigma"], case["depth"])
