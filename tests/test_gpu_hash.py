"""Cells sorted by a hash: its width, instances of one pass with different
cell factors, and a plan whose runs change between hashed and exact keys."""
import numpy as np
import pytest

import oracle
from paper_1409_8112_amd import workloads

pytestmark = pytest.mark.gpu


def _dev(p):
    import torch
    return torch.from_numpy(p).cuda()


@pytest.mark.parametrize("n,passes", [(1 << 21, 3), ((1 << 21) + 1, 4)])
def test_hash_is_wider_for_more_points(n, passes):
    """More points than 2^21 take more than 24 bits (which would put unrelated
    points of sparse sets into one run); the lists are those of the exact keys, which
    the sort-unique rule keeps."""
    from paper_1409_8112_amd import rtg
    pts = _dev(workloads.clustered_points(n, 12, seed=2, n_clusters=16000, sigma=0.01))
    with rtg.Context(0, arena_bytes=4 << 30) as ctx:
        got = ctx.all_pairs(pts, 0.028, 2, 2.0, 3)
        assert ctx.stats()["key_passes"] == passes
        ref = ctx.all_pairs(pts, 0.028, 2, 2.0, 3, rtg.DEDUP_SORT)
        assert ctx.stats()["key_passes"] > 4
        (rp, col), (rp2, col2) = got.to_numpy(), ref.to_numpy()
    assert len(col) > 10_000
    assert np.array_equal(rp, rp2) and np.array_equal(col, col2)


def test_hashed_instances_of_different_cell_factors():
    """One pass of instances whose cells differ in size: the signature fields
    are as wide as the least factor needs."""
    from paper_1409_8112_amd import rtg
    qs = []
    for q, alpha in enumerate((0.9, 2.0, 3.0)):
        pts = workloads.clustered_points(45_000 + q, 12, seed=q, n_clusters=150, sigma=0.01)
        qs.append((pts, 0.028, 8, alpha, 5 + q))
    with rtg.Context(0, arena_bytes=4 << 30) as ctx:
        res = ctx.all_pairs_batched([dict(points=_dev(p), r=r, k=k, alpha=a, seed=s)
                                     for p, r, k, a, s in qs])
        assert ctx.stats()["key_passes"] == 3
        for x, (p, r, k, a, s) in zip(res, qs):
            rp, col = x.to_numpy()
            ref = oracle.rtg(p, r, k, a, s)
            assert len(ref.col) > 1000
            assert np.array_equal(rp, ref.row_ptr) and np.array_equal(col, ref.col)


def test_plan_between_hashed_and_exact_keys():
    """The radius of a plan's run decides the width of its cells."""
    from paper_1409_8112_amd import rtg
    n, d, k = 66_000, 12, 8
    pts = [workloads.clustered_points(n, d, seed=q, n_clusters=3000, sigma=0.01) for q in (1, 2)]
    dev = [_dev(p) for p in pts]
    run = {}
    for name, r, passes in (("hashed", 0.028, 3), ("exact", 0.1, 5)):
        run[name] = (r, passes, [oracle.rtg(p, r, k, 2.0, q, rtg.NO_ROTATE)
                                 for q, p in enumerate(pts)])

    def queries(r):
        return [dict(points=p, r=r, k=k, alpha=2.0, seed=q, flags=rtg.NO_ROTATE)
                for q, p in enumerate(dev)]

    with rtg.Context(0, arena_bytes=4 << 30) as ctx, ctx.plan_create(queries(0.028)) as plan:
        for name in ("hashed", "hashed", "hashed", "exact", "exact", "hashed", "exact", "hashed"):
            r, passes, refs = run[name]
            res = plan.run(queries(r))
            assert ctx.stats()["key_passes"] == passes
            for x, ref in zip(res, refs):
                rp, col = x.to_numpy()
                assert len(ref.col) > 1000
                assert np.array_equal(rp, ref.row_ptr) and np.array_equal(col, ref.col)
            ctx.release_many(res)
        assert plan.info()["replays"] >= 2
