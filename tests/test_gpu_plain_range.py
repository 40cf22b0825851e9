"""The multi-pass search on coefficients of uneven size: what a few large ones
leave of the others."""

import numpy as np
import pytest

from helpers import flush_print
from oracle import correlate as oc
from workloads import configs as C
from workloads import rotations as wr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n,nm,planar", [(128, 70, False), (128, 87, True)])
def test_one_large_coefficient(dtype, n, nm, planar):
    """One coefficient holds half of the field's square sum.  Positions of up to 60
    cells are rounded to 6e-8 (1.1e-16), which moves the weights by 1e-6 (2e-15) at
    the 2-norm, and the transforms by less; the oracle's own in 64 bits likewise."""
    from paper_1712_00238_amd.api import Context
    rng = np.random.default_rng(n + nm)
    gf = C.GridSpec((n, n, 1 if planar else n), (0, 0, 0), 1.0)
    gm = C.GridSpec((nm, nm, 1 if planar else nm), (0, 0, 0), 1.0)
    rho_f, rho_m = (rng.normal(size=g.n[::-1]) + 1j * rng.normal(size=g.n[::-1]) for g in (gf, gm))
    rho_m = rho_m.astype(np.complex64).astype(np.complex128)
    rho_f = rho_f.astype(np.complex64).astype(np.complex128)
    rho_m[0, nm // 2, nm // 2 + 1] = np.round(np.linalg.norm(rho_m))
    w = np.ones(gm.n[::-1])
    q = wr.planar_rotations(23.0, 1) if planar else wr.uniform_quaternions(1, 5)
    ref = oc.score_volume(rho_f, oc.moving_coefficients(rho_m, w), q[0], nm, planar)
    with Context(0, dtype) as ctx:
        vol = ctx.score_volume(ctx.spectrum(rho_f, gf), gf, rho_m, w, gm, q).cpu().numpy()[0]
    err = np.linalg.norm(vol - ref.reshape(vol.shape)) / np.linalg.norm(ref)
    flush_print("one large coefficient", dtype, n, nm, planar, "2-norm", err)
    assert err <= (8e-15 if dtype == "f64" else 2e-6)
