"""sdf_build at the edges of its inputs: samples and weights that are not finite,
and calls past the size of one launch."""

import numpy as np
import pytest
from scipy.spatial import cKDTree

from helpers import flush_print
from workloads import configs as C
from workloads import shapes

pytestmark = pytest.mark.gpu

PARAMS = C.SDFParams(xi_floor=0.25)
GRID = C.GridSpec((14, 13, 12), (-6.5, -6.0, -5.5), 1.0)


@pytest.fixture(scope="module")
def ctxs():
    from paper_1712_00238_amd.api import Context
    c32, c64 = Context(0, "f32"), Context(0, "f64")
    yield {"f32": c32, "f64": c64}
    c32.close()
    c64.close()


def sphere(count, radius=4.0, seed=2):
    v = np.random.default_rng(seed).normal(size=(count, 3))
    v /= np.linalg.norm(v, axis=1, keepdims=True)
    return shapes.PointSamples(radius * v + 0.3, v.copy(), np.full(count, 4 * np.pi * radius ** 2 / count))


def join(s, q, n=(1.0, 0.0, 0.0), w=1.0):
    q = np.asarray(q, dtype=np.float64).reshape(-1, 3)
    return shapes.PointSamples(np.concatenate([s.q, q]), np.concatenate([s.n, np.tile(n, (len(q), 1))]),
                               np.concatenate([s.w, np.full(len(q), w)]))


def build(ctx, s, grid=GRID, params=PARAMS, phi=None):
    return ctx.sdf_build(s.q, s.n, s.w, grid, params, phi=phi).cpu().numpy().reshape(-1)


INF, NAN = np.inf, np.nan
# samples that fill a leaf of their own: NaN points share the first place
# of the order and (+inf, NaN, NaN) has the last: 64 and more of the first, and
# one of the last where it falls alone into the last leaf
ALL_BAD = [(640, [[NAN, NAN, NAN]] * 64), (576, [[INF, NAN, NAN]]), (700, [[NAN, NAN, NAN]] * 200),
           (64, [[INF, NAN, NAN]] * 3)]


@pytest.mark.parametrize("phi", [None, "inverse_square"])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("count,bad", ALL_BAD)
def test_leaf_without_a_finite_sample_counts_nowhere(ctxs, dtype, phi, count, bad):
    """The sums are those without the bad samples, in another order."""
    s = sphere(count)
    flush_print("bad leaf", dtype, phi, count, len(bad))
    a, b = build(ctxs[dtype], s, phi=phi), build(ctxs[dtype], join(s, bad), phi=phi)
    tol = 1e-12 if dtype == "f64" else 1e-5
    assert np.max(np.abs(a - b)) <= tol * np.abs(a).max()


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_leaf_of_a_node_and_samples_that_are_not_finite(ctxs, dtype):
    """63 NaN samples and one finite sample, four cells below the grid's corner and
    so of the lowest key, fill the first leaf, whose centre it is."""
    s = join(sphere(640), [[x - 4.0 * GRID.h for x in GRID.origin]], n=(-1.0, 0.0, 0.0), w=0.5)
    flush_print("node and NaNs", dtype)
    a, b = build(ctxs[dtype], s), build(ctxs[dtype], join(s, [[NAN, NAN, NAN]] * 63))
    tol = 1e-12 if dtype == "f64" else 1e-5
    assert np.max(np.abs(a - b)) <= tol * np.abs(a).max()


def ball_edges(s, grid, j):
    """For every node: is sample j inside its ball, and the ball's relative margin."""
    pts = grid.node_positions()
    xi = cKDTree(s.q).query(pts)[0]
    return np.linalg.norm(pts - s.q[j], axis=1) / ((1 + PARAMS.eps) * xi) - 1.0


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("bad", [NAN, INF, 1e300])
@pytest.mark.parametrize("count,grid", [(640, GRID), (30000, C.GridSpec((18, 17, 16), (-8.5, -8.0, -7.5), 1.0))])
def test_weight_that_is_not_finite_reaches_its_own_nodes_only(ctxs, dtype, bad, count, grid):
    """Nodes with the sample outside their ball have the sums of the part without
    it, those with it inside are not finite (1e300 is infinite in 32 bits).  30000
    samples on 4900 nodes are enough pairs for interpolated clusters."""
    s = sphere(count)
    j = count // 3
    w = s.w.copy()
    w[j] = 0.0
    ref = build(ctxs[dtype], shapes.PointSamples(s.q, s.n, w), grid)
    w[j] = bad
    flush_print("bad weight", dtype, bad, count)
    got = build(ctxs[dtype], shapes.PointSamples(s.q, s.n, w), grid)
    margin = ball_edges(s, grid, j)
    out, inside = margin > 1e-9, margin < -1e-9
    assert out.sum() > 100 and inside.sum() > 100
    tol = 1e-12 if dtype == "f64" else 1e-5
    assert np.max(np.abs(got - ref)[out]) <= tol * np.abs(ref).max()
    if dtype == "f32" or not np.isfinite(bad):
        live = inside & (ref != 0)
        assert not np.isfinite(got[live]).any()


@pytest.mark.parametrize("n", [(1024, 1024, 1024), (32768, 32768, 1)])
def test_grid_past_one_launch(ctxs, n):
    """2^30 and more threads' worth of 16-node bricks: the nodes of both ends and of
    the middle are those of a small grid there."""
    import torch
    s = sphere(50, 30.0)
    h = 0.5
    centre = [0.5 * h * m if m > 3 else 0.0 for m in n]
    s = shapes.PointSamples(s.q + np.array(centre), s.n, s.w)
    flush_print("large grid", n)
    out = ctxs["f32"].sdf_build(s.q, s.n, s.w, C.GridSpec(n, (0.0, 0.0, 0.0), h), PARAMS)
    for share in (0.0, 0.5, 1.0):
        m = tuple(min(x, 24) for x in n)
        at = [int(share * (x - y)) for x, y in zip(n, m)]
        part = C.GridSpec(m, tuple(h * a for a in at), h)
        ref = ctxs["f64"].sdf_build(s.q, s.n, s.w, part, PARAMS)
        got = out[at[2]:at[2] + m[2], at[1]:at[1] + m[1], at[0]:at[0] + m[0]].to(torch.complex128)
        # far from the part its terms cancel some hundredfold
        assert float((got - ref).abs().max()) <= 1e-4 * float(ref.abs().max())
    del out
    torch.cuda.empty_cache()


def test_samples_past_one_launch_of_the_interpolation_sums(ctxs):
    """1.4e8 samples: more than 2^32 threads in the sums of all interpolation points
    (without the last of them the field is off by its own size).  A ball of radius
    10 holds 1.4e6 samples, a quarter of them to a lane: sqrt(3.5e5) roundings of
    6e-8, and terms that cancel threefold."""
    import torch
    torch.cuda.empty_cache()
    count, radius = 140_000_000, 50.0
    gen = torch.Generator(device="cuda").manual_seed(1)
    n = torch.randn((count, 3), generator=gen, device="cuda", dtype=torch.float64)
    n /= n.norm(dim=1, keepdim=True)
    q = radius * n
    w = torch.full((count,), 4 * np.pi * radius ** 2 / count, dtype=torch.float64, device="cuda")
    # nodes 1 to 4 above the surface, whose balls reach up to 10
    grid = C.GridSpec((4, 3, 4), (0.0, 0.0, radius + 1.0), 1.0)
    flush_print("samples", count)
    got = ctxs["f32"].sdf_build(q, n, w, grid, PARAMS)
    ref = ctxs["f64"].sdf_build(q, n, w, grid, PARAMS)
    err = float((got.to(torch.complex128) - ref).abs().max()) / float(ref.abs().max())
    flush_print("relative error", err)
    assert err <= 1e-4
    del q, n, w
    torch.cuda.empty_cache()


def test_build_where_memory_holds_only_the_least_workspace():
    """With 1.5 GiB left on the device 1e7 samples have room for their order (0.7 GB)
    but not for the FP32 sum's records (2.6 GB): the build runs pair by pair."""
    import torch
    from paper_1712_00238_amd.api import Context
    torch.cuda.empty_cache()
    count, radius = 10_000_000, 20.0
    gen = torch.Generator(device="cuda").manual_seed(3)
    n = torch.randn((count, 3), generator=gen, device="cuda", dtype=torch.float64)
    n /= n.norm(dim=1, keepdim=True)
    q = radius * n
    w = torch.full((count,), 4 * np.pi * radius ** 2 / count, dtype=torch.float64, device="cuda")
    grid = C.GridSpec((4, 3, 4), (0.0, 0.0, radius + 1.0), 1.0)
    torch.cuda.empty_cache()
    with Context(0, "f64") as ctx:
        ref = ctx.sdf_build(q, n, w, grid, PARAMS).clone()
    left, held = 3 << 29, []
    with Context(0, "f32") as ctx:
        ctx.sdf_build(q[:100], n[:100], w[:100], grid, PARAMS)
        torch.cuda.synchronize()
        flush_print("free before", torch.cuda.mem_get_info()[0])
        while torch.cuda.mem_get_info()[0] > left + (16 << 20):
            size = min(torch.cuda.mem_get_info()[0] - left, 16 << 30)
            held.append(torch.empty(size, dtype=torch.uint8, device="cuda"))
        flush_print("free", torch.cuda.mem_get_info()[0])
        try:
            got = ctx.sdf_build(q, n, w, grid, PARAMS)
            again = ctx.sdf_build(q, n, w, grid, PARAMS)
            torch.cuda.synchronize()
        finally:
            held.clear()
            torch.cuda.empty_cache()
    assert torch.equal(got, again)
    # sequential FP32 sums of up to 1.6e5 terms a lane
    assert float((got.to(torch.complex128) - ref).abs().max()) <= 1e-3 * float(ref.abs().max())


def test_window_of_a_much_larger_part(ctxs):
    """Samples off the grid share a few keys, so their leaves are as wide as the part
    (8000 cells about a 64-cell window).  FP32 terms carry up to 3e-5 each, the
    sums of a node's terms cancel some threefold."""
    near, far = sphere(2000, 30.0, 5), sphere(2000, 8000.0, 6)
    mix = np.random.default_rng(1).permutation(4000)
    s = shapes.PointSamples(np.concatenate([near.q, far.q])[mix], np.concatenate([near.n, far.n])[mix],
                            np.concatenate([near.w, far.w])[mix])
    grid = C.GridSpec((33, 32, 31), (-8.0, -8.0, -7.5), 0.5)
    a, b = build(ctxs["f32"], s, grid), build(ctxs["f64"], s, grid)
    err = np.abs(a - b)
    flush_print("window: max rel", (err / np.abs(b)).max(), "2-norm", np.linalg.norm(err) / np.linalg.norm(b))
    assert np.all(err <= 1e-4 * np.abs(b) + 1e-6 * np.abs(b).max())


@pytest.mark.parametrize("outlier", [50.0, 2000.0, 8000.0, 80000.0])
def test_ball_edges_in_a_wide_leaf(ctxs, outlier):
    """Three samples in one leaf: the nearest (of next to no weight), one that some
    balls hold and some do not, and an outlier.  Whether the second counts is
    decided in FP64."""
    s = shapes.PointSamples(np.array([[0.3, 0.2, -0.1], [7.9, 0.4, 0.7], [outlier, 0.5 * outlier, 0.3 * outlier]]),
                            np.array([[1.0, 0.0, 0.0], [0.6, 0.0, 0.8], [1.0, 0.0, 0.0]]),
                            np.array([1e-12, 1.0, 1e-12]))
    grid = C.GridSpec((96, 96, 96), (-4.03, -4.01, -4.02), 0.0837)
    a, b = (np.abs(build(ctxs[d], s, grid)) for d in ("f32", "f64"))
    in_a, in_b = a > 1e-6 * a.max(), b > 1e-6 * b.max()
    flush_print("ball edges", outlier, int((in_a != in_b).sum()), int(in_b.sum()))
    assert 1000 < in_b.sum() < in_b.size - 1000
    assert np.array_equal(in_a, in_b)
