"""sdf_build of few samples, a thread per node: against the tree walk (which the
counting builds keep) at the edges of the rule, and against the oracle."""

import numpy as np
import pytest

from helpers import flush_print
from oracle import phi as ophi
from workloads import configs as C
from workloads import shapes

pytestmark = pytest.mark.gpu

PARAMS = C.SDFParams(xi_floor=0.25)


@pytest.fixture(scope="module")
def ctxs():
    from paper_1712_00238_amd.api import Context
    c32, c64 = Context(0, "f32"), Context(0, "f64")
    yield {"f32": c32, "f64": c64}
    c32.close()
    c64.close()


def sphere(count, radius=4.0):
    v = np.random.default_rng(count).normal(size=(count, 3))
    v /= np.linalg.norm(v, axis=1, keepdims=True)
    s = shapes.PointSamples(radius * v + 0.3, v.copy(), np.full(count, 4 * np.pi * radius ** 2 / count))
    if count > 5:  # exact ties of opposite sides (and other weight): the lower index decides
        s.q[4], s.n[4], s.w[4] = s.q[1], -s.n[1], 3.0 * s.w[1]
    return s


def grid(n, extent=14.0):
    h = extent / max(n)
    return C.GridSpec(n, tuple(-0.5 * h * (m - 1) + 0.01 for m in n), h)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n", [(9, 10, 11), (33, 1, 1), (1, 1, 70), (30, 31, 1), (64, 64, 64), (128, 90, 91),
                               (1024, 1024, 1)])
@pytest.mark.parametrize("count", [1, 32, 33, 64, 65, 300, 301, 576, 577])
def test_against_the_tree(ctxs, dtype, n, count):
    """The decisions are the same FP64 ones; sums differ by their order and form (3e-5
    a term in FP32, cancelling threefold)."""
    s, g = sphere(count), grid(n)
    flush_print("few", dtype, n, count)
    ctx = ctxs[dtype]
    few = ctx.sdf_build(s.q, s.n, s.w, g, PARAMS)
    ctx.set_option("sdf_stats", 1)
    tree = ctx.sdf_build(s.q, s.n, s.w, g, PARAMS)
    ctx.set_option("sdf_stats", 0)
    assert bool(((few == 0) == (tree == 0)).all())
    assert float((few - tree).abs().max()) <= (1e-12 if dtype == "f64" else 1e-4) * float(tree.abs().max())


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("phi", ["skeletal", "inverse_square", "dsl"])
def test_against_the_oracle(ctxs, dtype, phi):
    """With samples that are not finite, which count nowhere."""
    s, g = sphere(60), grid((17, 16, 15))
    bad = shapes.PointSamples(np.concatenate([s.q, [[np.nan, 0.0, 0.0], [0.0, np.inf, 1.0]]]),
                              np.concatenate([s.n, [[1.0, 0.0, 0.0]] * 2]), np.concatenate([s.w, [1.0, 1.0]]))
    flush_print("few, oracle", dtype, phi)
    got = ctxs[dtype].sdf_build(bad.q, bad.n, bad.w, g, PARAMS, phi=phi, radius=1.5).cpu().numpy().reshape(-1)
    ref = ophi.phi_points(s, g.node_positions(), PARAMS, phi, radius=1.5)
    assert np.max(np.abs(got - ref)) <= (1e-11 if dtype == "f64" else 1e-5) * np.abs(ref).max()
