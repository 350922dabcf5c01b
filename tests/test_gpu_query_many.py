"""Query mode with many queries: every row bit-exact with the oracle."""
import numpy as np
import pytest

import oracle
from paper_1409_8112_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,r", [(6, 0.25), (3, 0.05)])
def test_many_queries_every_row(d, r):
    """More queries than one wave per SIMD of the key kernel (65536)."""
    import torch
    from paper_1409_8112_amd import rtg
    k, alpha, seed = 5, 2.0, 9
    pts = workloads.uniform_points(20011, d, seed=5)
    qs = workloads.uniform_points(150001, d, seed=6)
    with rtg.Context(0, arena_bytes=4 << 30) as ctx:
        index = ctx.index_build(torch.from_numpy(pts).cuda(), r, k, alpha, seed)
        res = ctx.index_query(index, torch.from_numpy(qs).cuda())
        rp, col = res.to_numpy()
    R, u = rtg.make_transforms(seed, k, d)
    ref = oracle.rtg_query(pts, qs, r, alpha, R, u)
    assert np.array_equal(rp, ref.row_ptr) and np.array_equal(col, ref.col)


def _query(ctx, index, qs):
    import torch
    res = ctx.index_query(index, torch.from_numpy(qs).cuda())
    got = res.to_numpy()
    res.release()
    return got


@pytest.mark.parametrize("d", [2, 6, 13])
@pytest.mark.parametrize("m", [1, 4095, 4096, 65535, 65536, 65537])
def test_lanes_and_order_thresholds(d, m):
    """Either side of the sizes where queries take fewer lanes each and where
    they are ordered by place; a dimension without kernels of its own."""
    import torch
    from paper_1409_8112_amd import rtg
    k, alpha, seed = 3, 2.0, 4
    r = {2: 0.03, 6: 0.35, 13: 0.8}[d]
    pts = workloads.uniform_points(1501, d, seed=7)
    qs = workloads.uniform_points(m, d, seed=8)
    qs[:min(m, 100)] = pts[:min(m, 100)]
    with rtg.Context(0, arena_bytes=2 << 30) as ctx:
        index = ctx.index_build(torch.from_numpy(pts).cuda(), r, k, alpha, seed)
        rp, col = _query(ctx, index, qs)
    ref = oracle.rtg_query(pts, qs, r, alpha, *rtg.make_transforms(seed, k, d))
    assert np.array_equal(rp, ref.row_ptr) and np.array_equal(col, ref.col)


def test_index_extras_give_way():
    """The index's tables go back when other calls need the memory; its
    queries and theirs then run as without them."""
    import torch
    from paper_1409_8112_amd import rtg
    k, alpha, seed, r = 8, 2.0, 4, 0.02
    pts = workloads.uniform_points(30000, 3, seed=7)
    qs = workloads.uniform_points(70000, 3, seed=8)
    ref = oracle.rtg_query(pts, qs, r, alpha, *rtg.make_transforms(seed, k, 3))
    dev = torch.from_numpy(pts).cuda()
    with rtg.Context(0, arena_bytes=160 << 20) as ctx:
        index = ctx.index_build(dev, r, k, alpha, seed)
        rp, col = _query(ctx, index, qs)
        assert np.array_equal(rp, ref.row_ptr) and np.array_equal(col, ref.col)
        held = []
        with pytest.raises(rtg.RTGError) as e:
            for _ in range(2000):
                held.append(ctx.all_pairs(dev, 0.03, k, alpha, seed))
        assert e.value.code == rtg.ENOMEM
        ctx.release_many(held)
        rp, col = _query(ctx, index, qs)
        assert np.array_equal(rp, ref.row_ptr) and np.array_equal(col, ref.col)


@pytest.mark.parametrize("m,runs", [(1, 1), (5, 1), (20, 2)])
def test_many_pairs_of_few_queries_run_once(m, runs):
    """Some hundred thousand pairs that one block finds: they fit the first
    guess of their number, so one launch does, and one more for the cells
    of so many points that a query's own lanes do not finish.  More pairs than
    the guess run both again."""
    import torch
    from paper_1409_8112_amd import rtg
    pts = workloads.uniform_points(200_000, 3, seed=7)
    qs = (0.5 + 0.02 * workloads.uniform_points(m, 3, seed=8)).astype(np.float32)
    with rtg.Context(0, arena_bytes=1 << 30) as ctx:
        index = ctx.index_build(torch.from_numpy(pts).cuda(), 0.45, 4, 2.0, 3)
        rp, col = _query(ctx, index, qs)
        launches = ctx.stats()["kernel_launches"][rtg.KERNELS.index("pairs")]
    ref = oracle.rtg_query(pts, qs, 0.45, 2.0, *rtg.make_transforms(3, 4, 3))
    assert np.array_equal(rp, ref.row_ptr) and np.array_equal(col, ref.col)
    assert len(col) > 50_000 * m and (len(col) < 1 << 20) == (runs == 1)
    assert launches == 2 * runs


@pytest.mark.parametrize("d", [1, 3, 6, 13])
@pytest.mark.parametrize("m", [1, 70, 5000, 70000])
@pytest.mark.parametrize("crowd", [128, 256, 257, 1025, 3000, 9000])
def test_crowded_cells(d, m, crowd):
    """Cells of as many points as a query's own lanes test, and of more, which
    a wave finishes: with and without tables, in order and as given."""
    import torch
    from paper_1409_8112_amd import rtg
    rng = np.random.default_rng(crowd + d)
    r, k, alpha, seed = 0.03, 3, 2.0, 5
    pts = rng.random((4000 + crowd, d)).astype(np.float32)
    pts[::2][:crowd // 2] = (0.4 + 0.001 * rng.random((crowd // 2, d)))
    pts[1::2][:crowd - crowd // 2] = (0.7 + 0.02 * rng.random((crowd - crowd // 2, d)))
    qs = rng.random((m, d)).astype(np.float32)
    near = rng.permutation(m)[:min(m, 60)]
    qs[near] = pts[rng.integers(0, crowd, len(near))] + 0.001
    with rtg.Context(0, arena_bytes=4 << 30) as ctx:
        index = ctx.index_build(torch.from_numpy(pts).cuda(), r, k, alpha, seed)
        rp, col = _query(ctx, index, qs)
    rows = np.union1d(near, rng.permutation(m)[:100])
    ref = oracle.rtg_query(pts, qs[rows], r, alpha, *rtg.make_transforms(seed, k, d))
    assert np.array_equal(np.diff(rp)[rows], np.diff(ref.row_ptr))
    assert np.array_equal(np.concatenate([col[rp[i]:rp[i + 1]] for i in rows]), ref.col)
