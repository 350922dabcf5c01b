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


@pytest.mark.parametrize("d,alpha", [(2, 2.0), (6, 1.25), (9, 0.9), (20, 2.0), (40, 3.0)])
@pytest.mark.parametrize("k", [1, 4, 5, 23])
def test_grids_split_over_waves(ctx, d, alpha, k):
    """Signature words that end inside, at and past the grids the four waves
    share, in 32 and 64 bits; a last group of one point."""
    pts = workloads.uniform_points(321, d, seed=d)
    _check(ctx, pts, 0.35 * np.sqrt(d / 2.0), k, alpha, d + k)


@pytest.mark.parametrize("n", [768 * 256 - 256, 768 * 256 - 255])
def test_keys_either_side_of_the_split(ctx, n):
    pts = workloads.uniform_points(n, 3, seed=3)
    _check(ctx, pts, 0.02, 2, 2.0, 1)


def _stars(spokes, contiguous, n=9000, d=8, r=0.1, hubs=3):
    """Hubs with `spokes` points on the sphere around each, just within r (in
    d = 8 most of them are farther than r from one another), among far-away
    points; the spokes' indices together or spread over all."""
    rng = np.random.default_rng(spokes)
    pts = rng.random((n, d)) + 10.0
    at = np.arange(n) if contiguous else rng.permutation(n)
    for h in range(hubs):
        ids = at[h * (spokes + 1):(h + 1) * (spokes + 1)]
        g = rng.standard_normal((spokes, d))
        g *= 0.999 * r / np.linalg.norm(g, axis=1, keepdims=True)
        centre = rng.random(d)
        pts[ids[0]] = centre
        pts[ids[1:]] = centre + g
    return pts.astype(np.float32)


@pytest.mark.parametrize("spokes", [63, 64, 65, 66, 127, 129, 160, 1023, 1025, 1300])
@pytest.mark.parametrize("contiguous", [True, False])
def test_long_rows_in_bins(ctx, spokes, contiguous):
    """Rows either side of the short-row limit, of a crowded bin and of the
    longest row a crowded bucket sorts itself."""
    _check(ctx, _stars(spokes, contiguous), 0.1, 3, 6.0, spokes)


@pytest.mark.parametrize("n", [600, 3000, 40000])
def test_few_entries_in_many_buckets(ctx, n):
    pts = workloads.uniform_points(n, 4, seed=n)
    _check(ctx, pts, (6.0 / n) ** 0.25, 4, 2.0, 2)


def test_batches_around_the_request_loop():
    """Batched calls in several passes before, while and after requests are
    served: their extra streams are kept from call to call and given up to
    the loop."""
    import torch
    from paper_1409_8112_amd import rtg
    with rtg.Context(0, arena_bytes=2 << 30) as c:
        queries, refs = [], []
        for q in range(9):
            n, d = 700 + 301 * q, (2, 3, 6)[q % 3]
            pts = workloads.uniform_points(n, d, seed=q)
            r = {2: 0.05, 3: 0.1, 6: 0.4}[d]
            queries.append(dict(points=torch.from_numpy(pts).cuda(), r=r, k=3, alpha=2.0, seed=q))
            refs.append(oracle.rtg(pts, r, 3, 2.0, q))

        def batch():
            res = c.all_pairs_batched(queries)
            for x, ref in zip(res, refs):
                rp, col = x.to_numpy()
                assert np.array_equal(rp, ref.row_ptr) and np.array_equal(col, ref.col)
            c.release_many(res)

        batch()
        batch()
        tickets = [c.submit(q["points"], q["r"], q["k"], q["alpha"], q["seed"]) for q in queries]
        batch()
        for t, ref in zip(tickets, refs):
            x = c.wait(t)
            rp, col = x.to_numpy()
            assert np.array_equal(rp, ref.row_ptr) and np.array_equal(col, ref.col)
            x.release()
        batch()


@pytest.mark.parametrize("d,k,robots,upper", [(12, 8, 0, False), (12, 12, 0, True), (12, 8, 2, False),
                                              (20, 8, 0, False), (16, 9, 0, False)])
def test_hashed_keys(ctx, d, k, robots, upper):
    """Cells of more than 40 bits in a pass of 2^20 keys: sorted by a 24-bit
    hash, some hundred collisions per grid; one to three signature words."""
    from paper_1409_8112_amd import rtg
    n = 140_000
    pts = workloads.clustered_points(n, d, seed=d, n_clusters=400, sigma=0.01)
    r = {12: 0.028, 16: 0.038, 20: 0.048}[d]
    flags = (rtg.UPPER_ONLY if upper else 0) | (rtg.robots(robots) if robots else 0)
    _check(ctx, pts, r * (1.3 if robots else 1.0), k, 2.0, 3, flags)
    assert ctx.stats()["key_passes"] == 3


@pytest.mark.parametrize("scale", [2.0 ** -40, 2.0 ** 40])
def test_mr_metric_far_from_unit_scale(ctx, scale):
    """Radii below and above where the MR decision starts in FP32."""
    from paper_1409_8112_amd import rtg
    pts = (workloads.uniform_points(5000, 6, seed=3) * scale).astype(np.float32)
    _check(ctx, pts, 0.45 * scale, 4, 2.0, 2, rtg.robots(2))


@pytest.fixture(scope="module")
def small_ctx():
    from paper_1409_8112_amd import rtg
    with rtg.Context(0, arena_bytes=256 << 20) as c:
        yield c


@pytest.mark.parametrize("n", [2, 127, 128, 129, 257, 1000])
@pytest.mark.parametrize("d,k", [(1, 1), (2, 2), (3, 3), (3, 9), (5, 8), (8, 8)])
def test_small_instances(small_ctx, n, d, k):
    """Grids shared by the waves in every way, rows over several workgroups."""
    pts = workloads.uniform_points(n, d, seed=n + d)
    _check(small_ctx, pts, 0.4 * np.sqrt(d) * (4.0 / n) ** (1.0 / d), k, 1.5, k)


@pytest.mark.parametrize("d,cells", [(3, 505), (3, 520), (8, 6), (8, 11), (1, 100_000)])
@pytest.mark.parametrize("sign", [1, -1])
def test_small_instances_far_from_the_first_point(small_ctx, d, cells, sign):
    """Cells within and beyond what a word's field holds beside point 0's
    (the general pipeline then)."""
    rng = np.random.default_rng(cells)
    r, alpha, n = 0.05, 2.0, 400
    pts = rng.random((n, d)) * 0.3
    pts[n // 2:, 0] += sign * cells * alpha * r
    from paper_1409_8112_amd import rtg
    _check(small_ctx, pts.astype(np.float32), r, 4, alpha, 5, rtg.NO_ROTATE)


@pytest.mark.parametrize("n", [2, 1024, 1025, 2049, 8193, 16383, 16384, 16385])
@pytest.mark.parametrize("d", [2, 6])
def test_segments_sorted_one_to_a_block(ctx, n, d):
    """Segments up to and past the largest a block sorts, alone and beside
    shorter ones in a batch; one to four radix passes."""
    import torch
    pts = workloads.uniform_points(n, d, seed=n)
    r = 0.9 * (8.0 / n) ** (1.0 / d)
    _check(ctx, pts, r, 5, 1.3, n)
    small = workloads.uniform_points(37, d, seed=1)
    res = ctx.all_pairs_batched([dict(points=torch.from_numpy(p).cuda(), r=r, k=3, alpha=1.3, seed=7)
                                 for p in (small, pts, small)])
    for x, p in zip(res, (small, pts, small)):
        ref = oracle.rtg(p, r, 3, 1.3, 7)
        rp, col = x.to_numpy()
        assert np.array_equal(rp, ref.row_ptr) and np.array_equal(col, ref.col)
    ctx.release_many(res)


@pytest.mark.parametrize("n,d,cells,k", [(2000, 3, 1000, 4), (200, 3, 700, 20), (400, 8, 40, 1),
                                         (400, 8, 40, 5), (1000, 8, 12, 8), (1500, 6, 40, 6),
                                         (2000, 2, 60000, 3), (64, 3, 500_000, 2)])
@pytest.mark.parametrize("first", ["end", "middle", "stray"])
def test_small_thin_sets(small_ctx, n, d, cells, k, first):
    """Points along one axis, many more cells long than wide, however point 0
    lies: the two launches take them, whatever a field beside point 0 holds."""
    from paper_1409_8112_amd import rtg
    r, alpha = 0.05, 2.0
    rng = np.random.default_rng(n + d)
    pts = rng.random((n, d)) * 0.2
    pts[:, 0] = np.linspace(0.0, cells * alpha * r, n)
    if first == "middle":
        pts[[0, n // 2]] = pts[[n // 2, 0]]
    if first == "stray":
        pts = pts[rng.permutation(n)]
        pts[:, 0] = rng.random(n) * 3.0
        pts[0, 0] = cells * alpha * r
    _check(small_ctx, pts.astype(np.float32), r, k, alpha, 5, rtg.NO_ROTATE)
    assert small_ctx.stats()["kernel_launches"][rtg.KERNELS.index("keys")] == 0


def test_small_cells_beyond_a_word(small_ctx):
    """Cells that take more than 32 bits go through the general pipeline."""
    from paper_1409_8112_amd import rtg
    pts = (workloads.uniform_points(500, 3, seed=1) * 800.0).astype(np.float32)
    _check(small_ctx, pts, 0.05, 4, 2.0, 5)
    assert small_ctx.stats()["kernel_launches"][rtg.KERNELS.index("keys")] == 1


@pytest.mark.parametrize("size", [95, 97, 200, 500, 1000, 1100, 2300])
@pytest.mark.parametrize("places", [1, 2, 5])
def test_rows_crowded_in_a_few_places(ctx, size, places):
    """Clusters whose indices lie in a few runs: a row's columns fill few of
    its bins, with fewer and more entries than a wave sorts."""
    rng = np.random.default_rng(size + places)
    n, d = 9000, 6
    pts = np.concatenate([np.repeat(rng.random((n // size + 1, d)), size, axis=0)[:n],
                          rng.random((9000, d)) + 5.0])
    pts[:n] += 0.002 * rng.standard_normal((n, d))
    pts = np.concatenate([pts[i::places] for i in range(places)]).astype(np.float32)
    _check(ctx, pts, 0.02, 3, 2.5, size)
