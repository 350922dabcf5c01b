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
