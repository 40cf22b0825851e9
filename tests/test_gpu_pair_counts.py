"""score_pairs at the edges of its preparing launches (sixteen pairs each), with
reordered and plain spectra, shared and own, in one call."""

import numpy as np
import pytest

from helpers import flush_print
from workloads import configs as C
from workloads import rotations as wr

pytestmark = pytest.mark.gpu


def rand_job(ctx, n, nm, seed, spec=None):
    rng = np.random.default_rng(seed)
    gf, gm = C.GridSpec((n, n, n), (0, 0, 0), 1.0), C.GridSpec((nm, nm, nm), (0, 0, 0), 1.0)
    if spec is None:
        spec = ctx.spectrum(rng.normal(size=(n, n, n)) + 1j * rng.normal(size=(n, n, n)), gf)
    return {"spec": spec, "g_fixed": gf, "g_moving": gm, "quats": wr.uniform_quaternions(2, seed),
            "rho_moving": rng.normal(size=(nm, nm, nm)) + 1j * rng.normal(size=(nm, nm, nm)),
            "w_moving": rng.uniform(0.5, 1.5, size=(nm, nm, nm))}


@pytest.mark.parametrize("count", [1, 15, 16, 17, 33])
def test_each_pair_as_alone(count):
    from paper_1712_00238_amd.api import Context
    sizes = [(8, 2), (64, 20), (16, 6), (64, 9), (32, 14)]
    with Context(0, "f32") as ctx:
        jobs = [rand_job(ctx, *sizes[j % 5], seed=j) for j in range(count)]
        if count > 15:  # pairs that share a fixed part across two launches
            jobs[-1] = rand_job(ctx, 64, 7, 99, spec=jobs[1]["spec"])
        flush_print("pair counts", count)
        outs = ctx.score_pairs(jobs)
        for j, (job, out) in enumerate(zip(jobs, outs)):
            one = ctx.score_rotations(job["spec"], job["g_fixed"], job["rho_moving"], job["w_moving"],
                                      job["g_moving"], job["quats"])
            s, r = out["score"].cpu().numpy(), one["score"].cpu().numpy()
            # the same two rotations share a transform either way; FP32 sums of 64^3 terms otherwise
            assert np.max(np.abs(s - r)) <= 2e-6 * np.max(np.abs(r)), j
            assert np.array_equal(out["t"].cpu().numpy(), one["t"].cpu().numpy()), j
