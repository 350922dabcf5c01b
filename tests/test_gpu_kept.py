"""What a context keeps between calls for speed only is given back."""
import threading
import time

import numpy as np
import pytest

import oracle
from paper_1409_8112_amd import workloads

pytestmark = pytest.mark.gpu


def _dev(p):
    import torch
    return torch.from_numpy(p).cuda()


def _equal(res, ref):
    rp, col = res.to_numpy()
    assert np.array_equal(rp, ref.row_ptr) and np.array_equal(col, ref.col)
    res.release()


def test_batch_lanes_yield_to_the_request_loop():
    """The request loop starts while another thread's blocking call holds the
    context: the batched call's extra lanes go all the same, and later batches
    keep none."""
    from paper_1409_8112_amd import rtg
    pts = [workloads.uniform_points(700 + 301 * q, (2, 3, 6)[q % 3], seed=q) for q in range(9)]
    r = {2: 0.05, 3: 0.1, 6: 0.4}
    queries = [dict(points=_dev(p), r=r[p.shape[1]], k=3, alpha=2.0, seed=q)
               for q, p in enumerate(pts)]
    refs = [oracle.rtg(p, r[p.shape[1]], 3, 2.0, q) for q, p in enumerate(pts)]
    long_pts = _dev(workloads.uniform_points(300_000, 6, seed=1))
    with rtg.Context(0, arena_bytes=4 << 30) as ctx:
        def batch():
            for x, ref in zip(ctx.all_pairs_batched(queries), refs):
                _equal(x, ref)

        batch()
        assert ctx.debug_kept()["lanes"] == 2
        running = []
        blocking = threading.Thread(target=lambda: running.append(
            ctx.tune_params(long_pts, 0.12, 0.9, reps=3)))
        blocking.start()
        time.sleep(0.05)
        q = queries[0]
        ticket = ctx.submit(q["points"], q["r"], q["k"], q["alpha"], q["seed"])
        assert not running  # (the call was still running)
        assert ctx.debug_kept()["lanes"] == 0
        _equal(ctx.wait(ticket), refs[0])
        blocking.join()
        batch()
        assert ctx.debug_kept()["lanes"] == 0


def test_index_tables_yield_to_requests():
    """The tables of an index go back when the request loop needs the memory."""
    from paper_1409_8112_amd import rtg
    k, alpha, seed, r = 8, 2.0, 4, 0.02
    pts = workloads.uniform_points(30000, 3, seed=7)
    qs = workloads.uniform_points(5000, 3, seed=8)
    ref = oracle.rtg_query(pts, qs, r, alpha, *rtg.make_transforms(seed, k, 3))
    want = oracle.rtg(pts, r, k, alpha, seed)
    dev, dq = _dev(pts), _dev(qs)
    with rtg.Context(0, arena_bytes=80 << 20) as ctx:
        index = ctx.index_build(dev, r, k, alpha, seed)
        _equal(ctx.index_query(index, dq), ref)
        assert ctx.debug_kept()["index_table_bytes"] > 0
        held = []
        while ctx.debug_kept()["index_table_bytes"]:
            ticket = ctx.submit(dev, r, k, alpha, seed)
            assert ticket is not None and len(held) < 1000
            held.append(ctx.wait(ticket))
        for x in held:
            _equal(x, want)
        _equal(ctx.index_query(index, dq), ref)
        assert ctx.debug_kept()["index_table_bytes"] > 0


def test_index_tables_count_as_free():
    """The tables of several indexes do not split a call into more passes."""
    from paper_1409_8112_amd import rtg
    pts, qs = _dev(workloads.uniform_points(20000, 3, seed=7)), _dev(workloads.uniform_points(2500, 3, seed=8))
    other = workloads.uniform_points(100_000, 3, seed=9)
    dev = _dev(other)

    def passes(mib, tables):
        with rtg.Context(0, arena_bytes=mib << 20) as ctx:
            kept = [ctx.index_build(pts, 0.03, 8, 2.0, q) for q in range(8)]
            if tables:
                for ix in kept:
                    ctx.index_query(ix, qs).release()
                assert ctx.debug_kept()["index_table_bytes"] > 8 << 20
            res = ctx.all_pairs(dev, 0.02, 8, 2.0, 1)
            grids = ctx.stats()["transforms_per_sort"]
            rp, col = res.to_numpy()
            assert not tables or ctx.debug_kept()["index_table_bytes"] == 0
            return grids, rp, col

    ref = oracle.rtg(other, 0.02, 8, 2.0, 1)
    for mib in range(60, 120, 2):  # the least budget of one pass, without tables
        try:
            if passes(mib, False)[0] == 8:
                break
        except rtg.RTGError as e:
            assert e.code == rtg.ENOMEM
    grids, rp, col = passes(mib, True)
    assert grids == 8
    assert np.array_equal(rp, ref.row_ptr) and np.array_equal(col, ref.col)
