"""score_grad where few blocks would run: fewer poses a block, one sample a
thread, at the line between that split and the full one, with and without the
workspace for it."""

import numpy as np
import pytest

from helpers import flush_print
from oracle import correlate as oc
from oracle import grad as og
from oracle import spread as osp
from workloads import configs as C
from workloads import rotations as wr

pytestmark = pytest.mark.gpu


def case(n, nm, planar, count, seed):
    rng = np.random.default_rng(seed)
    gf = C.GridSpec((n, n, 1 if planar else n), (0, 0, 0), 1.0)
    gm = C.GridSpec((nm, nm, 1 if planar else nm), (0, 0, 0), 1.0)
    rho_f = rng.normal(size=gf.n[::-1]) + 1j * rng.normal(size=gf.n[::-1])
    rho_m = rng.normal(size=gm.n[::-1]) + 1j * rng.normal(size=gm.n[::-1])
    w = rng.uniform(0.5, 1.5, size=gm.n[::-1])
    t = rng.uniform(-n, 2 * n, size=(count, 3))
    q = wr.planar_rotations(41.0, count) if planar else wr.uniform_quaternions(count, seed)
    if planar:
        t[:, 2] = 0.0
    return gf, gm, rho_f, rho_m, w, np.concatenate([t, q], axis=1), rng.normal(size=count)


def full_split_bytes(n, nm, planar, count, dtype, weights):
    """Workspace of sixteen poses a block and four samples a thread (or the 8^3 tiles)."""
    K = nm * nm if planar else nm ** 3
    box = dtype == "f32" and not planar and n >= 17
    tiles = -(-nm // 8) ** 3 if box else -(-K // 1024)
    b = -(-(count * tiles * 56) // 256) * 256
    if weights:
        b += -(-(-(-count // 16) * K * (4 if dtype == "f32" else 8)) // 256) * 256
    return b + (96 * count if box else 0) + 256


# one pose; 8 blocks of old; a tile of one sample over; more than 64 pose groups; the line where blocks are enough
@pytest.mark.parametrize("dtype,n,nm,planar,count", [
    ("f64", 40, 16, True, 1), ("f64", 96, 64, True, 25), ("f64", 24, 11, False, 3), ("f32", 48, 33, True, 70),
    ("f64", 12, 4, True, 1100), ("f64", 70, 33, True, 511), ("f64", 70, 33, True, 513), ("f32", 17, 9, False, 1),
    ("f32", 34, 16, False, 130), ("f32", 20, 8, False, 1030), ("f32", 40, 24, False, 38)])
def test_fine_split_against_oracle_and_full_split(dtype, n, nm, planar, count):
    from paper_1712_00238_amd.api import Context
    gf, gm, rho_f, rho_m, w, poses, s = case(n, nm, planar, count, n + nm)
    out = {}
    for weights in (False, True):
        cap = full_split_bytes(n, nm, planar, count, dtype, weights)
        for name, ctx in (("fine", Context(0, dtype)), ("full", Context(0, dtype, workspace_cap=cap))):
            flush_print("pose split", dtype, n, nm, planar, count, weights, name)
            with ctx:
                got = ctx.score_grad(rho_f, gf, rho_m, w, gm, poses, want_pose=True, want_w=weights, grad_scale=s)
                out[name, weights] = [None if x is None else x.cpu().numpy() for x in got]
    # FP64 sums in another order; the FP32 score is rounded once, the FP32 weight sums up to 64 times
    for weights in (False, True):
        for k, tol in ((0, 1e-12 if dtype == "f64" else 2e-7), (1, 1e-12),
                       (2, 1e-12 if dtype == "f64" else 64 * 6e-8)):
            a, b = out["fine", weights][k], out["full", weights][k]
            assert (a is None) == (b is None)
            if a is not None:
                assert np.max(np.abs(a - b)) <= tol * np.max(np.abs(b)), (k, weights)
    c = oc.moving_coefficients(rho_m, w)
    xb = osp.body_positions(nm, planar)
    score, gp, _ = out["fine", True]
    # positions of up to 60 cells round to 4e-6 cells in 32 bits, sums of up to 14 thousand terms of either sign
    tol = 1e-10 if dtype == "f64" else 2e-4
    for b in sorted({0, count // 2, count - 1}):
        f, dt, dq, _ = og.pose_value_and_grad(rho_f, c, rho_m, xb, poses[b, :3], poses[b, 3:])
        ref = np.concatenate([dt, dq])
        assert abs(score[b] - f) <= tol * max(1.0, abs(f))
        assert np.max(np.abs(gp[b] - ref)) <= tol * np.max(np.abs(ref))
