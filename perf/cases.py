"""The work that a program has this library do, as timed cases.

Every case goes through the public binding (paper_1409_8112_amd.rtg): whole
all-pairs queries, batches, fixed-shape plans, the request loop and the query
index.  Sizes, radii and parameters are those of the benchmark's workloads,
of the paper's parameter table (its m and c~ are k and alpha here) or generic.

A case is a dict of plain values:
  op      all_pairs, noalloc, batched, plan, serve, index_query, index_fresh
  n, d    points and dimension (batched, plan, serve: n is the upper end of
          the instances' sizes, n_lo the lower, dims the dimensions they draw
          from, count how many, mix the seed of their sizes and dimensions)
  kind    uniform in the unit cube, or clustered (80% in 64 Gaussian clusters)
  r       radius; k, alpha grids and cell-size factor
  rotate, upper, robots   random orientations, one-sided lists, MR-metric
  m       query points (index_query, index_fresh)

The outputs are neighbour lists: whole numbers, the same for the same inputs
whatever computes them, so exact() has no 64-bit value to give for them.  The
library's lists are valid until they are released, so a pass copies the
columns into the program's own storage (room for more than are expected,
zeros past the last), one copy for a batch.
"""
from __future__ import annotations

import functools
import math
import random

import numpy as np
import torch

from paper_1409_8112_amd import rtg, workloads

GIB = 1 << 30


# --- radii -------------------------------------------------------------------

@functools.lru_cache(maxsize=None)
def _ball_sample(d: int) -> np.ndarray:
    rng = np.random.default_rng(12345)
    g = rng.standard_normal((8192, d))
    g /= np.linalg.norm(g, axis=1, keepdims=True)
    return np.abs(g * rng.random(len(g))[:, None] ** (1.0 / d))


def _neighbours(n: int, d: int, r: float) -> float:
    """Mean neighbours within r of one of n uniform points in the unit cube."""
    inside = np.prod(np.clip(1.0 - r * _ball_sample(d), 0.0, None), axis=1).mean()
    return (n - 1) * workloads.unit_ball_volume(d) * r ** d * float(inside)


@functools.lru_cache(maxsize=None)
def _radius_for(n: int, d: int, neighbours: float) -> float:
    """The radius at which _neighbours(n, d, r) is the given mean."""
    lo, hi = 0.0, math.sqrt(d)
    for _ in range(50):
        mid = 0.5 * (lo + hi)
        lo, hi = (mid, hi) if _neighbours(n, d, mid) < neighbours else (lo, mid)
    return 0.5 * (lo + hi)


def _cluster_radius(n: int, d: int) -> float:
    """A radius for about 30 neighbours in clustered points (sigma 0.02)."""
    density = 0.8 * n / 64 / ((4.0 * math.pi) ** (d / 2.0) * 0.02 ** d)
    return (30.0 / (workloads.unit_ball_volume(d) * density)) ** (1.0 / d)


# --- cases -------------------------------------------------------------------

def _case(name=None, **kw) -> dict:
    c = {"op": "all_pairs", "kind": "uniform", "rotate": True, "upper": False, "robots": 0}
    if name:
        c["name"] = name
    c.update(kw)
    return c


def listed() -> list[dict]:
    return [
        # The smallest roadmap of the paper's table: a planner that grows its
        # sample set calls this again and again (shift-only, as the paper ran).
        _case("table_n200_d3", n=200, d=3, r=workloads.fmt_radius(200, 3), k=20, alpha=1.275,
              rotate=False),
        # The benchmark's small workload: one latency-bound query.
        _case("small_d3", n=2000, d=3, r=0.1, k=4, alpha=2.0),
        # A mid-size roadmap with the table's many narrow grids.
        _case("table_n6400_d6", n=6400, d=6, r=workloads.fmt_radius(6400, 6), k=25, alpha=1.225,
              rotate=False),
        # The parameter study's setting (high dimension, hundreds of
        # neighbours within the FMT* radius) at its chosen parameters.
        _case("study_d9", n=102400, d=9, r=workloads.fmt_radius(102400, 9), k=25, alpha=1.4),
        # Planar points, an odd count, each pair stored once.
        _case("upper_d2", n=300007, d=2, r=_radius_for(300007, 2, 15.0), k=6, alpha=2.0,
              upper=True),
        # Two robots in 3-D under the sum-of-distances metric.
        _case("robots_d6", n=200003, d=6, r=_radius_for(200003, 6, 60.0), k=8, alpha=2.0,
              robots=2),
        # The benchmark's default workload.
        _case("uniform_d6", n=1_000_000, d=6, r=workloads.R_UNIFORM_1E6_D6, k=8, alpha=2.0),
        # The benchmark's largest: uneven occupancy in 12 dimensions.
        _case("clustered_d12", n=4_000_000, d=12, r=workloads.R_CLUSTERED_4E6_D12, k=8, alpha=2.0,
              kind="clustered"),
        # A batch of independent instances of mixed sizes and dimensions.
        _case("batch_32", op="batched", count=32, n_lo=1000, n=64000, dims="2,3,6,9", mix=1,
              k=6, alpha=2.0),
        # A burst of requests to the serving loop, all awaited.
        _case("serve_16", op="serve", count=16, n_lo=500, n=200000, dims="3,6,12", mix=2,
              k=8, alpha=2.0),
        # New points looked up in the index of a large set.
        _case("query_1e6_d3", op="index_query", n=1_000_000, d=3, m=1_000_000,
              r=_radius_for(1_000_000, 3, 15.0), k=8, alpha=2.0),
        # A fresh index and a first set of lookups, as when the points change
        # each time: latency counts.
        _case("index_fresh_d6", op="index_fresh", n=50021, d=6, m=5003,
              r=_radius_for(50021, 6, 15.0), k=8, alpha=2.0),
    ]


def _log_int(rng: random.Random, lo: float, hi: float) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random) -> dict:
    what = rng.choice(["plain", "plain", "table", "table", "upper", "robots", "clustered", "noalloc",
                       "batched", "plan", "serve", "index_query", "index_fresh"])
    d = rng.randint(2, 12)
    if what in ("plain", "upper", "noalloc"):
        top = {"plain": 1e6, "upper": 1e6, "noalloc": 5e4}[what]
        n = _log_int(rng, 100, top if d <= 6 else min(top, 1.5e5))
        c = _case(n=n, d=d, r=_radius_for(n, d, float(rng.choice([8, 15, 20, 30]))),
                  k=rng.randint(4, 10), alpha=2.0, rotate=rng.random() < 0.8,
                  upper=what == "upper")
        if what == "noalloc":
            c["op"] = "noalloc"
        return c
    if what == "table":
        n = _log_int(rng, 100, 1e5)
        k = rng.choice([20, 25, 30] if d >= 6 else [20])
        alpha = round(rng.uniform(1.15, 1.3) if d < 6 else rng.uniform(1.225, 1.4), 3)
        return _case(n=n, d=d, r=workloads.fmt_radius(n, d), k=k, alpha=alpha,
                     rotate=rng.random() < 0.5)
    if what == "robots":
        b = rng.choice([2, 3])
        d = b * rng.randint(2, 3)
        n = _log_int(rng, 2000, 3e5)
        return _case(n=n, d=d, r=_radius_for(n, d, 40.0), k=8, alpha=2.0, robots=b)
    if what == "clustered":
        d = rng.randint(6, 12)
        n = _log_int(rng, 2e4, 2e6)
        return _case(n=n, d=d, r=_cluster_radius(n, d), k=rng.randint(6, 8), alpha=2.0,
                     kind="clustered")
    if what in ("batched", "plan", "serve"):
        return _case(op=what, count=rng.randint(4, 32 if what != "serve" else 16),
                     n_lo=rng.choice([500, 1000]), n=_log_int(rng, 1e4, 1e5),
                     dims=rng.choice(["2,3,6,9", "3,6,12", "3", "6"]), mix=rng.randrange(1 << 20),
                     k=rng.choice([6, 8]), alpha=2.0)
    n = _log_int(rng, 1000, 1e6 if what == "index_query" and d <= 6 else 1e5)
    m = _log_int(rng, 100, n if d != 6 else min(n, 6e4))
    return _case(op=what, n=n, d=d, m=m, r=_radius_for(n, d, 15.0), k=rng.randint(4, 10), alpha=2.0)


# --- inputs --------------------------------------------------------------------

def _points(n: int, d: int, kind: str, gen: torch.Generator) -> torch.Tensor:
    dev = gen.device
    if kind == "uniform":
        return torch.rand((n, d), generator=gen, device=dev)
    n_cl = int(round(0.8 * n))
    centres = torch.rand((64, d), generator=gen, device=dev)
    which = torch.randint(0, 64, (n_cl,), generator=gen, device=dev)
    cl = centres[which] + 0.02 * torch.randn((n_cl, d), generator=gen, device=dev)
    pts = torch.cat([cl.clamp_(0.0, 1.0), torch.rand((n - n_cl, d), generator=gen, device=dev)])
    return pts[torch.randperm(n, generator=gen, device=dev)].contiguous()


def _instances(case: dict) -> list[tuple[int, int, float]]:
    """(n, d, r) of a batch's or burst's instances: ~15 neighbours at the
    geometric-mean size, the radius scaled as (ln n / n)^(1/d)."""
    rng = random.Random(case["mix"])
    dims = [int(x) for x in case["dims"].split(",")]
    n_mid = int(round(math.sqrt(case["n_lo"] * case["n"])))
    out = []
    for _ in range(case["count"]):
        n, d = _log_int(rng, case["n_lo"], case["n"]), rng.choice(dims)
        gamma = _radius_for(n_mid, d, 15.0) / (math.log(n_mid) / n_mid) ** (1.0 / d)
        out.append((n, d, workloads.prm_radius(n, d, gamma)))
    return out


def _parts(case: dict) -> list[tuple[int, int, int, float]]:
    """(n, d, rows, mean neighbours) of each list a pass makes."""
    if case["op"] in ("batched", "plan", "serve"):
        return [(n, d, n, _neighbours(n, d, r)) for n, d, r in _instances(case)]
    n, d = case["n"], case["d"]
    nb = 30.0 if case["kind"] == "clustered" else _neighbours(n, d, case["r"])
    if case["robots"]:
        # the sum of the robots' distances is at most r in a smaller ball
        b, e = case["robots"], d // case["robots"]
        nb *= (math.gamma(e + 1.0) ** b / math.gamma(d + 1.0)
               * workloads.unit_ball_volume(e) ** b / workloads.unit_ball_volume(d))
    return [(n, d, case.get("m", n), nb)]


def _room(case: dict) -> int:
    """Column entries the program keeps room for."""
    spare = 2.5 if case["kind"] == "clustered" else 1.3
    return 4096 + int(sum(spare * rows * nb for _, _, rows, nb in _parts(case)))


def _flags(case: dict) -> int:
    return ((0 if case["rotate"] else rtg.NO_ROTATE) | (rtg.UPPER_ONLY if case["upper"] else 0)
            | (rtg.robots(case["robots"]) if case["robots"] else 0))


def prepare(case: dict, seed: int) -> dict:
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(seed)
    rtg_seed = seed % 1000
    op = case["op"]
    s = {"case": case, "seed": rtg_seed, "flags": _flags(case), "held": [],
         "col": torch.zeros(_room(case), dtype=torch.int32, device="cuda:0")}
    if op in ("batched", "plan", "serve"):
        s["ctx"] = rtg.Context(0, arena_bytes=6 * GIB)
        s["queries"] = [dict(points=_points(n, d, case["kind"], gen), r=r, k=case["k"],
                             alpha=case["alpha"], seed=rtg_seed + q, flags=s["flags"])
                        for q, (n, d, r) in enumerate(_instances(case))]
        if op == "plan":
            s["plan"] = s["ctx"].plan_create(s["queries"])
        return s
    n, d = case["n"], case["d"]
    s["ctx"] = rtg.Context(0, arena_bytes=(16 if n > 500_000 else 6) * GIB)
    s["points"] = _points(n, d, case["kind"], gen)
    if op == "noalloc":
        s["row_ptr"] = torch.zeros(n + 1, dtype=torch.int64, device="cuda:0")
    if op in ("index_query", "index_fresh"):
        s["queries"] = _points(case["m"], d, case["kind"], gen)
    if op == "index_query":
        s["index"] = s["ctx"].index_build(s["points"], case["r"], case["k"], case["alpha"],
                                          rtg_seed, s["flags"])
    return s


def run(s: dict):
    c, ctx = s["case"], s["ctx"]
    op = c["op"]
    if s["held"]:  # the previous pass's lists have been used
        ctx.release_many(s["held"])
        s["held"] = []
    if op == "noalloc":
        ctx.all_pairs_noalloc(s["points"], c["r"], c["k"], c["alpha"], s["seed"], s["row_ptr"],
                              s["col"], s["flags"])
        return s["row_ptr"], s["col"]
    if op == "batched":
        res = ctx.all_pairs_batched(s["queries"])
    elif op == "plan":
        res = s["plan"].run(s["queries"])
    elif op == "serve":
        tickets = []
        for q in s["queries"]:
            t = ctx.submit(q["points"], q["r"], q["k"], q["alpha"], q["seed"], q["flags"])
            while t is None:
                t = ctx.submit(q["points"], q["r"], q["k"], q["alpha"], q["seed"], q["flags"])
            tickets.append(t)
        res = [ctx.wait(t) for t in tickets]
    elif op == "index_query":
        res = [ctx.index_query(s["index"], s["queries"])]
    elif op == "index_fresh":
        index = ctx.index_build(s["points"], c["r"], c["k"], c["alpha"], s["seed"], s["flags"])
        res = [ctx.index_query(index, s["queries"])]
        ctx.release(index)
    else:
        res = [ctx.all_pairs(s["points"], c["r"], c["k"], c["alpha"], s["seed"], s["flags"])]
    s["held"] = res
    if len(res) == 1:
        s["col"][:res[0].nnz].copy_(res[0].col)
    else:
        torch.cat([r.col for r in res], out=s["col"][:sum(r.nnz for r in res)])
    return [r.row_ptr for r in res] + [s["col"]]


def exact(case: dict, seed: int):
    return None  # whole numbers: equal, or wrong


# --- work ----------------------------------------------------------------------

def work(case: dict) -> dict:
    """Points (and queries) read once and lists written once; the cells of
    every point under every grid (2 d^2 + 2 d operations) and one distance
    (3 d) per listed neighbour."""
    nbytes = flops = 0.0
    for n, d, rows, nb in _parts(case):
        lists = rows * nb * (0.5 if case["upper"] else 1.0)
        built = rows if case["op"] == "index_query" else n
        nbytes += 4.0 * n * d + (4.0 * rows * d if "m" in case else 0.0) + 8.0 * (rows + 1) + 4.0 * lists
        flops += built * case["k"] * (2.0 * d * d + 2.0 * d) + 3.0 * d * lists
    return {"bytes": nbytes, "flops": flops}
