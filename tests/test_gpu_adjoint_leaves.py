"""sdf_build_adjoint leaf by leaf: sample counts round the 64-sample leaves,
ragged grids of one and of several bricks (leaves split over blocks), planar
grids, and a sample that is not finite."""

import numpy as np
import pytest

from helpers import flush_print
from oracle import sdf_adjoint as oadj
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


def samples(count, seed, planar):
    rng = np.random.default_rng(seed)
    v = rng.normal(size=(count, 3))
    if planar:
        v[:, 2] = 0.0
    v /= np.linalg.norm(v, axis=1, keepdims=True)
    r = 3.0 + 0.4 * np.sin(5 * v[:, :1])
    return shapes.PointSamples(r * v + (np.array([0.3, 0.2, 0.0 if planar else 0.1])), v.copy(),
                               rng.uniform(0.5, 1.5, count) * 4 * np.pi * 9 / count)


GRIDS = [((7, 5, 3), False), ((13, 9, 6), False), ((19, 17, 1), True)]


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n,planar", GRIDS)
@pytest.mark.parametrize("count", [1, 63, 64, 65, 321])
def test_against_oracle(ctxs, dtype, n, planar, count):
    s = samples(count, count + n[0], planar)
    grid = C.GridSpec(n, tuple(-0.5 * (m - 1) + 0.013 * (m > 1) for m in n), 1.0)
    params = C.SDFParams(xi_floor=0.25)
    rng = np.random.default_rng(5)
    cot = rng.normal(size=n[::-1]) + 1j * rng.normal(size=n[::-1])
    if dtype == "f32":
        cot = cot.astype(np.complex64)
    flush_print("adjoint leaves", dtype, n, count)
    got = [a.cpu().numpy() for a in ctxs[dtype].sdf_build_adjoint(s.q, s.n, s.w, grid, params, cot)]
    ref = oadj.sdf_adjoint_grid(s, grid, params, cot.astype(np.complex128))
    # FP64 in both contexts: hundreds of terms of a few roundings, cancelling a thousandfold at worst
    for a, b in zip(got, ref):
        assert np.max(np.abs(a - b)) <= 1e-10 * np.abs(b).max()


def test_sample_that_is_not_finite_gets_and_gives_nothing(ctxs):
    s = samples(130, 4, False)
    grid = C.GridSpec((13, 9, 6), (-6.0, -4.0, -2.5), 1.0)
    params = C.SDFParams(xi_floor=0.25)
    cot = np.random.default_rng(1).normal(size=(6, 9, 13)) + 0j
    a = [x.cpu().numpy() for x in ctxs["f64"].sdf_build_adjoint(s.q, s.n, s.w, grid, params, cot)]
    bad = shapes.PointSamples(np.concatenate([s.q, [[np.nan, 0, 0]]]), np.concatenate([s.n, [[1.0, 0, 0]]]),
                              np.concatenate([s.w, [1.0]]))
    b = [x.cpu().numpy() for x in ctxs["f64"].sdf_build_adjoint(bad.q, bad.n, bad.w, grid, params, cot)]
    for x, y in zip(a, b):
        assert np.max(np.abs(x - y[:130])) <= 1e-12 * np.abs(x).max()
        assert np.all(y[130] == 0)


@pytest.mark.parametrize("n,count", [((40, 37, 33), 1000), ((24, 8, 4), 257), ((70, 45, 1), 700)])
def test_nearest_samples_found_once_or_per_brick(ctxs, n, count):
    """Grids of few bricks find the nearest samples in a pass of their own where
    the workspace allows; under a cap below it a block does both for its brick."""
    from paper_1712_00238_amd.api import Context
    s = samples(count, count, n[2] == 1)
    grid = C.GridSpec(n, tuple(-0.1 * (m - 1) + 0.013 * (m > 1) for m in n), 0.2)
    params = C.SDFParams(xi_floor=0.05)
    cot = np.random.default_rng(6).normal(size=n[::-1]) + 1j
    bricks = -(-n[0] // 16) * -(-n[1] // 16) if n[2] == 1 else -(-n[0] // 8) * -(-n[1] // 8) * -(-n[2] // 4)
    flush_print("adjoint, nearest pass", n, count)
    a = [x.cpu().numpy() for x in ctxs["f64"].sdf_build_adjoint(s.q, s.n, s.w, grid, params, cot)]
    with Context(0, "f64", workspace_cap=max(bricks * 5120, 150 * count)) as capped:
        b = [x.cpu().numpy() for x in capped.sdf_build_adjoint(s.q, s.n, s.w, grid, params, cot)]
    # FP64 sums in another order, cancelling a thousandfold at worst
    for x, y in zip(a, b):
        assert np.max(np.abs(x - y)) <= 1e-11 * np.abs(y).max()
