"""General pipeline at the edges of its tiles and groups: lists bit-exact with
the oracle."""
import numpy as np
import pytest

import oracle
from paper_1409_8112_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import os
    from paper_1409_8112_amd import rtg
    old = os.environ.get("RTG_SMALL")
    os.environ["RTG_SMALL"] = "0"  # the general pipeline at every size
    try:
        c = rtg.Context(0, arena_bytes=4 << 30)
    finally:
        if old is None:
            del os.environ["RTG_SMALL"]
        else:
            os.environ["RTG_SMALL"] = old
    yield c
    c.close()


def _check(ctx, pts, r, k, alpha, seed, flags=0):
    import torch
    res = ctx.all_pairs(torch.from_numpy(pts).cuda(), r, k, alpha, seed, flags)
    rp, col = res.to_numpy()
    res.release()
    ref = oracle.rtg(pts, r, k, alpha, seed, flags)
    assert np.array_equal(rp, ref.row_ptr) and np.array_equal(col, ref.col)


@pytest.mark.parametrize("n", [2, 63, 64, 65, 1023, 1024, 1025, 4095, 4096, 4097, 8193])
@pytest.mark.parametrize("k", [1, 3])
def test_runs_over_group_and_tile_ends(ctx, n, k):
    """Cells of about 40 points: runs of equal keys that start, end and
    cross at every place of the 64-key groups, the waves and the tiles."""
    pts = workloads.uniform_points(n, 2, seed=n)
    _check(ctx, pts, float(np.sqrt(10.0 / n)), k, 2.0, n)
