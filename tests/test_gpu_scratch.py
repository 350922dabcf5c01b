"""Device-memory budgets in which calls have to run."""
import numpy as np
import pytest

import oracle
from paper_1409_8112_amd import workloads

pytestmark = pytest.mark.gpu


def _radius(n, d, neighbours):
    return (neighbours / (n * workloads.unit_ball_volume(d))) ** (1.0 / d)


def _lists(res):
    out = [r.to_numpy() for r in res]
    for r in res:
        r.release()
    return out


def all_pairs(n, d, k, neighbours, flags=0):
    pts, r = workloads.uniform_points(n, d, seed=1), _radius(n, d, neighbours)

    def run(ctx):
        import torch
        return _lists([ctx.all_pairs(torch.from_numpy(pts).cuda(), r, k, 2.0, 3, flags)])

    return run, lambda: [oracle.rtg(pts, r, k, 2.0, 3, flags)]


def batch(count, n, d, k, neighbours):
    pts = [workloads.uniform_points(n, d, seed=q) for q in range(count)]
    r = _radius(n, d, neighbours)

    def run(ctx):
        import torch
        return _lists(ctx.all_pairs_batched(
            [dict(points=torch.from_numpy(p).cuda(), r=r, k=k, alpha=2.0, seed=q)
             for q, p in enumerate(pts)]))

    return run, lambda: [oracle.rtg(p, r, k, 2.0, q) for q, p in enumerate(pts)]


# Budgets in KiB, to the next 64: the least that the pass of the call takes
# with lists built from large buckets only.
PASSES = {
    "rows of 120 in one grid": (all_pairs(20000, 2, 1, 120.0), 21568),
    "nine instances": (batch(9, 3000, 3, 4, 15.0), 8320),
}


@pytest.mark.parametrize("name", PASSES)
def test_small_buckets_give_way(name):
    """Lists of few entries are built from many small buckets where memory
    allows: no call needs more memory for that."""
    from paper_1409_8112_amd import rtg
    (run, want), kib = PASSES[name]
    with rtg.Context(0, arena_bytes=kib << 10) as ctx:
        got = run(ctx)
    for (rp, col), ref in zip(got, want()):
        assert np.array_equal(rp, ref.row_ptr) and np.array_equal(col, ref.col)


def index_query(n, d, m, k, neighbours, robots=0, calls=2):
    pts, qs = workloads.uniform_points(n, d, seed=1), workloads.uniform_points(m, d, seed=2)
    r = _radius(n, d, neighbours)

    def run(ctx):
        import torch
        from paper_1409_8112_amd import rtg
        flags = rtg.robots(robots) if robots else 0
        index = ctx.index_build(torch.from_numpy(pts).cuda(), r, k, 2.0, 3, flags)
        q = torch.from_numpy(qs).cuda()
        return [x for _ in range(calls) for x in _lists([ctx.index_query(index, q)])]

    rows = np.arange(0, m, max(1, m // 400))  # rows do not depend on one another

    def want():
        from paper_1409_8112_amd import rtg
        flags = oracle.robots(robots) if robots else 0
        return rows, oracle.rtg_query(pts, qs[rows], r, 2.0, *rtg.make_transforms(3, k, d), flags)

    return run, want


# Budgets in KiB, to the next 64, of the index and the call: the least that a
# call takes whose queries run as given, read the points by index and put
# their pairs into one segment.
QUERIES = {
    "few queries": (index_query(2000, 2, 100, 8, 15.0), 8384),
    "n / 8 queries": (index_query(50000, 3, 6250, 8, 15.0), 13696),
    "unordered": (index_query(50000, 3, 60000, 8, 15.0), 30656),
    "ordered": (index_query(50000, 3, 70000, 8, 15.0), 35072),
    "ordered, many grids": (index_query(2000, 3, 70000, 20, 15.0), 37120),
    "ordered, few pairs": (index_query(2000, 3, 400000, 4, 3.0), 127360),
    "more pairs than guessed": (index_query(50000, 3, 70000, 8, 80.0), 107840),
    "two robots": (index_query(2000, 4, 2000, 8, 30.0, robots=2), 8896),
    "two robots, ordered": (index_query(50000, 4, 70000, 8, 30.0, robots=2), 41024),
}


@pytest.mark.parametrize("name", QUERIES)
def test_queries_in_the_least_memory(name):
    """What a query call has for speed only (the order of the queries, the
    index's tables, output segments) is given up where memory is short."""
    from paper_1409_8112_amd import rtg
    (run, want), kib = QUERIES[name]
    with rtg.Context(0, arena_bytes=kib << 10) as ctx:
        got = run(ctx)
    rows, ref = want()
    for rp, col in got:
        assert np.array_equal(np.diff(rp)[rows], np.diff(ref.row_ptr))
        assert np.array_equal(np.concatenate([col[rp[i]:rp[i + 1]] for i in rows]), ref.col)
