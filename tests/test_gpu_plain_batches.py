"""The multi-pass search in batches of rotations: the tile spread and the fused
transform passes at every grid size, odd boxes and tiles partly outside the
body, several batches under a workspace cap, and fields that are not finite."""

import numpy as np
import pytest

from helpers import flush_print
from oracle import correlate as oc
from workloads import configs as C
from workloads import rotations as wr

pytestmark = pytest.mark.gpu


def case(n, nm, planar, seed):
    rng = np.random.default_rng(seed)
    gf = C.GridSpec((n, n, 1 if planar else n), (0, 0, 0), 1.0)
    gm = C.GridSpec((nm, nm, 1 if planar else nm), (0, 0, 0), 1.0)
    f = [rng.normal(size=g.n[::-1]) + 1j * rng.normal(size=g.n[::-1]) for g in (gf, gm)]
    return gf, gm, f[0], f[1], rng.uniform(0.5, 1.5, size=gm.n[::-1])


def quats(planar, count, seed):
    return wr.planar_rotations(23.0, count) if planar else wr.uniform_quaternions(count, seed)


SIZES = [(8, 2, False), (8, 2, True), (16, 6, False), (16, 5, True), (32, 15, False), (32, 19, True), (64, 33, False),
         (64, 41, True), (96, 21, False), (96, 64, True), (128, 87, True)]


@pytest.mark.parametrize("n,nm,planar", SIZES)
def test_fp64_peaks_and_volumes(n, nm, planar):
    """FP64 against the oracle: transforms and sums of n^d terms keep 1e-11 of the largest score."""
    from paper_1712_00238_amd.api import Context
    gf, gm, rho_f, rho_m, w = case(n, nm, planar, n + nm)
    q = quats(planar, 3, n)
    flush_print("plain batch", n, nm, planar)
    with Context(0, "f64") as ctx:
        spec = ctx.spectrum(rho_f, gf)
        out = ctx.score_rotations(spec, gf, rho_m, w, gm, q)
        vol = ctx.score_volume(spec, gf, rho_m, w, gm, q).cpu().numpy()
    c = oc.moving_coefficients(rho_m, w)
    for r in range(len(q)):
        ref = oc.score_volume(rho_f, c, q[r], nm, planar)
        tol = 1e-11 * np.abs(ref).max()
        assert np.max(np.abs(vol[r] - ref)) <= tol
        t = out["t"][r].cpu().numpy()
        assert abs(float(out["score"][r]) - ref.max()) <= tol
        assert abs(ref[t[2], t[1], t[0]] - ref.max()) <= tol
        offs = [(dx, dy, dz) for dz in (-1, 0, 1) for dy in (-1, 0, 1) for dx in (-1, 0, 1)]
        nb = [ref[(t[2] + dz) % ref.shape[0], (t[1] + dy) % n, (t[0] + dx) % n] for dx, dy, dz in offs]
        assert np.max(np.abs(out["nbhd"][r].cpu().numpy() - nb)) <= tol


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_batches_under_a_cap_equal_one_batch(dtype):
    """Integer sums: the batch a rotation falls in changes nothing, bit for bit."""
    import torch
    from paper_1712_00238_amd.api import Context
    gf, gm, rho_f, rho_m, w = case(32, 15, False, 3)
    q = quats(False, 11, 5)
    elem = 8 if dtype == "f64" else 4
    with Context(0, dtype) as a, Context(0, dtype, workspace_cap=2 * elem * (32 ** 3 * 4 + 15 ** 3) + 8192) as b:
        a.set_option("path", 1)
        b.set_option("path", 1)
        spec = a.spectrum(rho_f, gf)
        x, y = (c.score_rotations(spec, gf, rho_m, w, gm, q) for c in (a, b))
        torch.cuda.synchronize()
        assert all(torch.equal(x[k], y[k]) for k in x)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_field_that_is_not_finite_gives_nan_volumes(dtype, bad):
    from paper_1712_00238_amd.api import Context
    gf, gm, rho_f, rho_m, w = case(16, 6, False, 4)
    rho_m[2, 3, 1] = bad
    with Context(0, dtype) as ctx:
        vol = ctx.score_volume(ctx.spectrum(rho_f, gf), gf, rho_m, w, gm, quats(False, 2, 1))
        assert bool(vol.isnan().all())


def test_zero_field_scores_zero():
    from paper_1712_00238_amd.api import Context
    gf, gm, rho_f, rho_m, w = case(16, 6, False, 4)
    with Context(0, "f64") as ctx:
        out = ctx.score_rotations(ctx.spectrum(rho_f, gf), gf, 0 * rho_m, w, gm, quats(False, 2, 1))
        assert bool((out["score"] == 0).all()) and bool((out["t"] == 0).all())


@pytest.mark.parametrize("count", [8, 9])
def test_tiles_of_few_and_of_many_rotations(count):
    """Up to 8192 tiles (eight rotations of 128^3) take eight waves each, more
    take four: the integer sums are the same either way."""
    from paper_1712_00238_amd.api import Context
    gf, gm, rho_f, rho_m, w = case(128, 13, False, 3)
    q = quats(False, count, 8)
    flush_print("plain tiles", count)
    with Context(0, "f64") as ctx:
        spec = ctx.spectrum(rho_f, gf)
        many = ctx.score_rotations(spec, gf, rho_m, w, gm, q)
        for r in (0, count - 1):
            one = ctx.score_rotations(spec, gf, rho_m, w, gm, q[r:r + 1])
            for k in ("score", "t", "nbhd", "refined"):
                assert np.array_equal(many[k][r].cpu().numpy(), one[k][0].cpu().numpy()), (r, k)
