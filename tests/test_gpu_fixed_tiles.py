"""score_grad_fixed tile by tile: grids that tiles divide unevenly, boxes that
wrap round the torus (several images of a tile), pose ranges with partial grids,
the FP64 sums' flush, and values that are not finite."""

import numpy as np
import pytest

from helpers import flush_print
from oracle import correlate as oc
from oracle import grad as og
from oracle import spread as osp
from workloads import configs as C
from workloads import rotations as wr

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctxs():
    from paper_1712_00238_amd.api import Context
    c32, c64 = Context(0, "f32"), Context(0, "f64")
    yield {"f32": c32, "f64": c64}
    c32.close()
    c64.close()


def case(n, nm, planar, count, seed):
    rng = np.random.default_rng(seed)
    gf = C.GridSpec((n, n, 1 if planar else n), (0, 0, 0), 1.0)
    gm = C.GridSpec((nm, nm, 1 if planar else nm), (0, 0, 0), 1.0)
    rho_m = rng.normal(size=gm.n[::-1]) + 1j * rng.normal(size=gm.n[::-1])
    w = rng.uniform(0.5, 1.5, size=gm.n[::-1])
    t = rng.uniform(-3 * n, 4 * n, size=(count, 3))
    q = wr.planar_rotations(41.0, count) if planar else wr.uniform_quaternions(count, seed)
    if planar:
        t[:, 2] = 0.0
    return gf, gm, rho_m, w, np.concatenate([t, q], axis=1), rng.normal(size=count)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n,nm,planar,count", [(4, 4, False, 3), (9, 7, False, 35), (17, 17, False, 5),
                                               (37, 11, False, 2), (40, 40, True, 33), (33, 5, True, 1),
                                               (65, 21, True, 4)])
def test_against_oracle(ctxs, dtype, n, nm, planar, count):
    gf, gm, rho_m, w, poses, s = case(n, nm, planar, count, n + nm)
    flush_print("fixed tiles", dtype, n, nm, planar, count)
    got = ctxs[dtype].score_grad_fixed(gf, rho_m, w, gm, poses, grad_scale=s).cpu().numpy()
    c = oc.moving_coefficients(rho_m, w)
    ref = og.fixed_cotangent(c, osp.body_positions(nm, planar), poses, s, got.shape)
    # positions of up to 30 cells and weights rounded once each: 1e-5 of the largest sum in 32 bits
    tol = 1e-12 if dtype == "f64" else 1e-5
    assert np.max(np.abs(got - ref)) <= tol * np.abs(ref).max()


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_repeats_bit_for_bit_and_without_partial_grids(ctxs, dtype):
    """Integer sums: two calls are equal; a cap below the partial grids gives the
    same to rounding."""
    import torch
    from paper_1712_00238_amd.api import Context
    gf, gm, rho_m, w, poses, s = case(24, 9, False, 40, 2)
    a, b = (ctxs[dtype].score_grad_fixed(gf, rho_m, w, gm, poses, grad_scale=s) for _ in range(2))
    with Context(0, dtype, workspace_cap=4096) as ctx:
        c = ctx.score_grad_fixed(gf, rho_m, w, gm, poses, grad_scale=s)
    torch.cuda.synchronize()
    assert torch.equal(a, b)
    assert float((a - c).abs().max()) <= (1e-13 if dtype == "f64" else 1e-6) * float(a.abs().max())


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_values_that_are_not_finite(ctxs, dtype):
    """A NaN coefficient leaves NaN at its own nodes only; a zero scale drops its pose."""
    gf, gm, rho_m, w, poses, s = case(24, 9, False, 2, 3)
    ref = ctxs[dtype].score_grad_fixed(gf, rho_m, w, gm, poses, grad_scale=np.array([1.0, 0.0])).cpu().numpy()
    one = ctxs[dtype].score_grad_fixed(gf, rho_m, w, gm, poses[:1]).cpu().numpy()
    assert np.max(np.abs(ref - one)) <= 1e-6 * np.abs(one).max()
    rho_m[4, 5, 6] = np.nan
    got = ctxs[dtype].score_grad_fixed(gf, rho_m, w, gm, poses[:1]).cpu().numpy()
    bad = np.isnan(got)
    assert 1 <= bad.sum() <= 64
    assert np.max(np.abs(got - one)[~bad]) <= 1e-6 * np.abs(one).max()
