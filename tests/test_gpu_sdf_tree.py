"""sdf_build over its sample tree: leaves, sibling groups and record groups at
their edges, grids on both sides of the one-wave / four-wave rule, far clusters
replaced by interpolation points, and the same sums with the workspace capped
below them."""

import numpy as np
import pytest

from helpers import flush_print, sdf_compare
from oracle import sdf as osdf
from workloads import configs as C
from workloads import shapes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctxs():
    from paper_1712_00238_amd.api import Context
    c32, c64 = Context(0, "f32"), Context(0, "f64")
    yield {"f32": c32, "f64": c64}
    c32.close()
    c64.close()


def sphere(count, radius, seed, flat=False):
    rng = np.random.default_rng(seed)
    v = rng.normal(size=(count, 3))
    v /= np.linalg.norm(v, axis=1, keepdims=True)
    if not flat:
        return shapes.PointSamples(radius * v + 0.3, v.copy(), np.full(count, 4 * np.pi * radius ** 2 / count))
    q = rng.uniform(-radius, radius, size=(count, 3))
    q[:, 2] = np.where(np.arange(count) % 2, 1.5, -1.5)
    n = np.zeros((count, 3))
    n[:, 2] = np.sign(q[:, 2])
    return shapes.PointSamples(q, n, np.full(count, 8 * radius ** 2 / count))


def build(ctx, s, grid, params):
    return ctx.sdf_build(s.q, s.n, s.w, grid, params).cpu().numpy().reshape(-1)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("count", [15, 16, 17, 63, 64, 65, 1023, 1025, 4096, 4097])
def test_tree_and_sort_edges(ctxs, dtype, count):
    """One record group short and over, one leaf, one sibling group, and the
    largest count of the one-block sort."""
    s = sphere(count, 4.0, count)
    grid = C.GridSpec((11, 10, 9), (-5.2, -4.6, -4.1), 1.0)
    params = C.SDFParams(xi_floor=0.25)
    flush_print("sdf tree", dtype, count)
    rel, band = (1e-10, 1e-10) if dtype == "f64" else (2e-5, 2e-5)
    rep = sdf_compare(build(ctxs[dtype], s, grid, params), s, grid, params, rel, band, max_ambiguous_frac=0.03)
    flush_print(rep)
    assert rep["ok"], rep


# (samples, radius, two flat faces, grid, spacing): pairs from 1e8 on, so far clusters are interpolated
FAR = [(2900, 6.0, False, (33, 34, 35), 1.5), (20000, 7.0, False, (40, 37, 30), 1.0),
       (20000, 20.0, True, (41, 40, 39), 1.0), (1300, 5.0, True, (66, 65, 64), 0.7)]


@pytest.mark.parametrize("count,radius,flat,n,h", FAR)
def test_interpolated_clusters_against_fp64(ctxs, count, radius, flat, n, h):
    """FP32 builds against the FP64 ones, which sum every pair.  Interpolation
    leaves up to 1e-6 of a cluster's terms and FP32 sums 6e-8 per operation, and
    the sum of a node's terms may cancel some fifty-fold: 1e-4 of the value,
    plus 1e-6 of the largest one."""
    s = sphere(count, radius, 7 + count, flat)
    grid = C.GridSpec(n, tuple(-0.5 * h * (m - 1) for m in n), h)
    params = C.SDFParams()
    flush_print("sdf interpolation", count, flat, n)
    a, b = build(ctxs["f32"], s, grid, params), build(ctxs["f64"], s, grid, params)
    err = np.abs(a - b)
    flush_print("rel 2-norm", np.linalg.norm(err) / np.linalg.norm(b))
    # ball-edge decisions are FP64 in both: no node is exempt
    assert np.all(err <= 1e-4 * np.abs(b) + 1e-6 * np.abs(b).max())
    assert np.array_equal(a == 0, b == 0)
    # and the FP64 build against the oracle on sampled nodes
    pick = np.random.default_rng(3).choice(len(b), 300, replace=False)
    ref = osdf.sdf_points(s, grid.node_positions()[pick], params)
    assert np.max(np.abs(b[pick] - ref)) <= 1e-10 * np.abs(b).max()


def test_capped_workspace_sums_pair_by_pair(ctxs):
    """A cap that holds the sorted samples but not the FP32 sum's records: the
    build runs all the same."""
    from paper_1712_00238_amd.api import Context
    s = sphere(20000, 7.0, 5)
    grid = C.GridSpec((40, 37, 30), (-19.5, -18.0, -14.5), 1.0)
    ref = build(ctxs["f64"], s, grid, C.SDFParams())
    with Context(0, "f32", workspace_cap=2 << 20) as ctx:
        got = build(ctx, s, grid, C.SDFParams())
    assert np.all(np.abs(got - ref) <= 1e-4 * np.abs(ref) + 1e-6 * np.abs(ref).max())


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_sample_that_is_not_finite_counts_nowhere(ctxs, dtype):
    """A sample with a NaN or infinite coordinate is nobody's nearest and in no
    ball: the build equals the one without it."""
    s = sphere(700, 4.0, 2)
    grid = C.GridSpec((14, 13, 12), (-6.5, -6.0, -5.5), 1.0)
    params = C.SDFParams(xi_floor=0.25)
    bad = shapes.PointSamples(np.concatenate([s.q, [[np.nan, 0, 0], [1.0, np.inf, 2.0]]]),
                              np.concatenate([s.n, [[1.0, 0, 0], [0, 1.0, 0]]]), np.concatenate([s.w, [1.0, 1.0]]))
    a, b = build(ctxs[dtype], s, grid, params), build(ctxs[dtype], bad, grid, params)
    tol = 1e-12 if dtype == "f64" else 1e-5
    assert np.max(np.abs(a - b)) <= tol * np.abs(a).max()
