"""score_grad_fixed at the edges of its inputs: poses and terms that are not
finite, long body lines almost along the grid's axes, scales and coefficients of
uneven size."""

import numpy as np
import pytest

from helpers import flush_print
from oracle import correlate as oc
from oracle import grad as og
from oracle import rotation
from oracle import spread as osp
from workloads import configs as C
from workloads import rotations as wr

pytestmark = pytest.mark.gpu

INF, NAN = np.inf, np.nan


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


def fixed(ctx, gf, rho_m, w, gm, poses, s):
    return ctx.score_grad_fixed(gf, rho_m, w, gm, poses, grad_scale=s).cpu().numpy()


def reached(shape, nm, planar, pose):
    """Nodes of the samples' stencils; a coordinate that is not a number has floor 0."""
    with np.errstate(invalid="ignore"):
        ti = np.floor(pose[:3])
        y = (pose[:3] - ti) + osp.body_positions(nm, planar) @ rotation.quat_to_matrix(pose[3:]).T
    base = (np.nan_to_num(np.floor(y), nan=0.0) + np.nan_to_num(ti, nan=0.0) - 1).astype(int)
    mask = np.zeros(shape, dtype=bool)
    for cz in range(1 if planar else 4):
        for cy in range(4):
            for cx in range(4):
                mask[(base[:, 2] + cz) % shape[0] if not planar else 0, (base[:, 1] + cy) % shape[1],
                     (base[:, 0] + cx) % shape[2]] = True
    return mask


# the entries of a pose that are not finite: one translation, the rotation, both
BAD_POSES = [{0: NAN}, {1: NAN}, {3: NAN, 4: NAN, 5: NAN, 6: NAN}, {a: NAN for a in range(7)}, {3: INF}]


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n,nm,planar", [(37, 7, False), (20, 9, False), (70, 21, True)])
@pytest.mark.parametrize("bad", BAD_POSES)
def test_pose_that_is_not_finite_reaches_its_stencils_only(ctxs, dtype, n, nm, planar, bad):
    """NaN at the nodes of its samples' stencils, the other poses' sums elsewhere;
    with a scale of zero it adds nothing."""
    gf, gm, rho_m, w, poses, s = case(n, nm, planar, 5, n + nm)
    c = oc.moving_coefficients(rho_m, w)
    for a, v in bad.items():
        poses[2, a] = v
    flush_print("bad pose", dtype, n, nm, planar, bad)
    keep = [0, 1, 3, 4]
    shape = gf.n[::-1]
    ref = og.fixed_cotangent(c, osp.body_positions(nm, planar), poses[keep], s[keep], shape)
    tol = (1e-12 if dtype == "f64" else 1e-5) * np.abs(ref).max()
    hit = reached(shape, nm, planar, poses[2])
    got = fixed(ctxs[dtype], gf, rho_m, w, gm, poses, s).reshape(shape)
    assert np.array_equal(np.isnan(got.real), hit) and np.array_equal(np.isnan(got.imag), hit)
    assert np.max(np.abs(got - ref)[~hit]) <= tol
    s[2] = 0.0
    got = fixed(ctxs[dtype], gf, rho_m, w, gm, poses, s).reshape(shape)
    assert np.max(np.abs(got - ref)) <= tol


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_masked_pose_in_the_backward_call(ctxs, dtype):
    """score_grad_backward's rho_fixed cotangent with a NaN pose of cotangent zero."""
    gf, gm, rho_m, w, poses, s = case(20, 9, False, 4, 5)
    poses[1] = NAN
    s[1] = 0.0
    flush_print("masked pose", dtype)
    got = ctxs[dtype].score_grad_backward(None, gf, rho_m, w, gm, poses, s, want_pose=False, want_fixed=True)[3]
    keep = [0, 2, 3]
    ref = og.fixed_cotangent(oc.moving_coefficients(rho_m, w), osp.body_positions(9, False), poses[keep], s[keep],
                             gf.n[::-1])
    assert np.max(np.abs(got.cpu().numpy() - ref)) <= (1e-12 if dtype == "f64" else 1e-5) * np.abs(ref).max()


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("planar", [False, True])
def test_infinite_terms_add_as_numbers_do(ctxs, dtype, planar):
    """An infinite part leaves its infinity at its sample's nodes, infinities of
    opposite signs NaN where they meet, and the other part is as without them."""
    n, nm = (30, 9) if not planar else (50, 13)
    gf, gm, rho_m, w, poses, s = case(n, nm, planar, 3, n)
    s[:] = [1.0, -0.5, 2.0]
    at = [(0, 3, 4), (0, 5, 6)] if planar else [(2, 3, 4), (3, 5, 4)]
    zeroed = rho_m.copy()
    for j in at:
        zeroed[j] = 1j * rho_m[j].imag
    c = oc.moving_coefficients(zeroed, w)
    shape = gf.n[::-1]
    ref = og.fixed_cotangent(c, osp.body_positions(nm, planar), poses, s, shape)
    up, down = np.zeros(shape, dtype=bool), np.zeros(shape, dtype=bool)
    for j, sign in zip(at, (1.0, -1.0)):
        one = np.zeros(rho_m.shape)
        one[j] = 1.0
        for b in range(3):
            hit = np.abs(og.fixed_cotangent(one.ravel(), osp.body_positions(nm, planar), poses[b:b + 1], np.ones(1),
                                            shape)) > 0
            (up if sign * s[b] > 0 else down)[hit] = True
        rho_m[j] = complex(sign * INF, rho_m[j].imag)
    expect = np.where(up & down, NAN, np.where(up, INF, np.where(down, -INF, ref.real)))
    flush_print("infinite terms", dtype, planar)
    got = fixed(ctxs[dtype], gf, rho_m, w, gm, poses, s).reshape(shape)
    tol = (1e-12 if dtype == "f64" else 1e-5) * np.abs(ref).max()
    plain = np.isfinite(expect)
    assert np.array_equal(got.real[~plain], expect[~plain], equal_nan=True)
    assert (up & down).any() and up.any() and down.any()
    assert np.max(np.abs(got.real[plain] - expect[plain])) <= tol
    assert np.max(np.abs(got.imag - ref.imag)) <= tol
    # an infinite scale: every node of its pose
    s[2] = INF
    got = fixed(ctxs[dtype], gf, zeroed, w, gm, poses, s).reshape(shape)
    hit = reached(shape, nm, planar, poses[2])
    assert not np.isfinite(got.imag[hit]).any()
    two = og.fixed_cotangent(c, osp.body_positions(nm, planar), poses[:2], s[:2], shape)
    assert np.max(np.abs(got - two)[~hit]) <= tol


@pytest.mark.parametrize("n,nm,angle,t", [(1100, 1024, 9e-5, (3.3, 40.0)), (1600, 1500, -9.9e-5, (0.7, 2.026)),
                                          (520, 500, 9.9e-5, (5.25, 7.98))])
def test_long_lines_almost_along_an_axis(ctxs, n, nm, angle, t):
    """Lines of a wide planar body that drift across a tile's edge over their length."""
    gf, gm, rho_m, w, poses, s = case(n, nm, True, 1, n)
    poses[0] = [t[0], t[1], 0.0, np.cos(0.5 * angle), 0.0, 0.0, np.sin(0.5 * angle)]
    flush_print("long lines", n, nm, angle)
    got = fixed(ctxs["f64"], gf, rho_m, w, gm, poses, s).reshape(gf.n[::-1])
    ref = og.fixed_cotangent(oc.moving_coefficients(rho_m, w), osp.body_positions(nm, True), poses, s, gf.n[::-1])
    assert np.max(np.abs(got - ref)) <= 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("small", [1e-3, 1e-6, 1e-12, 1e-24])
@pytest.mark.parametrize("nm,planar", [(9, False), (13, True)])
def test_poses_of_small_scale_keep_their_digits(ctxs, dtype, small, nm, planar):
    """Softmax-like scales on poses that do not meet: each pose's nodes are as
    accurate as if it were alone (positions of 40 cells and weights rounded once
    each: 1e-5 and 1e-13 of the pose's largest sum)."""
    gf, gm, rho_m, w, poses, s = case(80, nm, planar, 20, nm)
    poses[:, :3] = [10.3, 20.6, 0.0 if planar else 30.2]
    poses[1::2, 0] += 40.0  # 0 and 40 apart, 9 sqrt 3 + 4 and 13 sqrt 2 + 4 reach 20
    s = np.where(np.arange(20) % 2, small * s, s)
    xb, shape = osp.body_positions(nm, planar), gf.n[::-1]
    flush_print("small scales", dtype, small, nm, planar)
    got = fixed(ctxs[dtype], gf, rho_m, w, gm, poses, s).reshape(shape)
    c = oc.moving_coefficients(rho_m, w)
    for part in (0, 1):
        ref = og.fixed_cotangent(c, xb, poses[part::2], s[part::2], shape)
        on = np.zeros(shape, dtype=bool)
        on[..., 40 * part:40 * part + 40] = True
        assert np.max(np.abs(got - ref)[on]) <= (1e-13 if dtype == "f64" else 1e-5) * np.abs(ref).max()


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_one_large_coefficient_leaves_the_others_theirs(ctxs, dtype):
    """A coefficient 1e4 (FP64: 1e2) times the rest: nodes away from it are as accurate
    as without it."""
    gf, gm, rho_m, w, poses, s = case(40, 15, False, 6, 4)
    poses[:, :3] = 20.0
    large = 1e4 if dtype == "f32" else 1e2
    rho_m[0, 0, 0] = large * (1 + 1j)
    one = np.zeros(rho_m.shape)
    one[0, 0, 0] = 1.0
    xb, shape = osp.body_positions(15, False), gf.n[::-1]
    away = og.fixed_cotangent(one.ravel(), xb, poses, np.ones(6), shape) == 0
    ref = og.fixed_cotangent(oc.moving_coefficients(rho_m, w), xb, poses, s, shape)
    flush_print("one large coefficient", dtype)
    err = np.abs(fixed(ctxs[dtype], gf, rho_m, w, gm, poses, s).reshape(shape) - ref)[away].max()
    flush_print("error", err / np.abs(ref[away]).max())
    assert err <= (1e-13 if dtype == "f64" else 1e-5) * np.abs(ref[away]).max()


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n,nm,planar,count", [(4, 3, False, 70), (8, 8, False, 1), (20, 20, False, 9),
                                               (21, 21, False, 9), (48, 48, True, 9), (49, 49, True, 9),
                                               (5, 5, True, 2), (30, 30, False, 1), (64, 64, True, 3)])
def test_small_tori(ctxs, dtype, n, nm, planar, count):
    """Fields on either side of the rule that walks all samples for every tile, with
    the largest boxes, against the oracle (positions and weights rounded once each)."""
    gf, gm, rho_m, w, poses, s = case(n, nm, planar, count, n + count)
    flush_print("small torus", dtype, n, nm, planar, count)
    got = fixed(ctxs[dtype], gf, rho_m, w, gm, poses, s).reshape(gf.n[::-1])
    ref = og.fixed_cotangent(oc.moving_coefficients(rho_m, w), osp.body_positions(nm, planar), poses, s, gf.n[::-1])
    assert np.max(np.abs(got - ref)) <= (1e-12 if dtype == "f64" else 1e-5) * np.abs(ref).max()
