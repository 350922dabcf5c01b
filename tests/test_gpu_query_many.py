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
