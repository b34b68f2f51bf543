"""Frame updates below and above the angle (1/4) and the length error (2^-18)
up to which the update takes power series instead of roots, sines and
divisions, in all kernels that update frames: one Euler and one RK4 step from
frames of slightly wrong length against the FP64 oracle.

Tolerance.  A frame turns by dt Omega; the velocities agree to 1e-12 of each
other, so at angles up to 3 the frames agree to 3e-12, and 1e-11 with the
rounding of the update (about 30 operations on numbers of size one, 1e-14) and
of the four RK4 stages."""
import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import rod_of, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mrs():
    import paper_2604_12083_amd as m

    return m


@pytest.fixture(scope="module")
def ctx(mrs):
    c = mrs.mrs_context_create(0)
    yield c
    mrs.mrs_context_destroy(c)


@pytest.mark.parametrize("F,M", [(1, 64), (3, 50)])  # whole steps in one workgroup, stages
@pytest.mark.parametrize("angle", [1e-7, 0.2, 0.3, 3.0])  # the largest of the ensemble
@pytest.mark.parametrize("stretch", [0.0, 2.0 ** -19, 2.0 ** -17, 1e-3])
def test_frames_after_one_step(mrs, ctx, F, M, angle, stretch):
    e = synth.filaments(F, M, 3.0, 7)
    D = np.asarray(e.D).reshape(-1, 3, 3) * (1.0 + stretch)
    _, W = oracle.velocities(e.offsets, e.X, D, e.rod(), e.f, e.n, e.eps, e.mu, False)
    dt = angle / np.linalg.norm(W, axis=1).max()
    for integ in ("EULER", "RK4") if angle <= 0.3 else ("EULER",):
        say("frames", F, M, angle, stretch, integ)
        _, Do, _, _ = oracle.step(e.offsets, e.X, D, e.rod(), e.f, e.n, e.eps, e.mu, getattr(oracle, integ), dt, 1, False)
        h = mrs.mrs_ensemble_create(ctx, e.offsets, e.X, D, e.f, e.n, e.eps, e.mu, rod_of(mrs, e.rod()))
        mrs.mrs_ensemble_step(ctx, h, getattr(mrs, "MRS_" + integ), dt, 1, mrs.MRS_FP64, False)
        D1 = mrs.mrs_ensemble_get(ctx, h)[1]
        mrs.mrs_ensemble_destroy(h)
        d = np.abs(np.asarray(D1).reshape(-1) - np.asarray(Do).reshape(-1)).max()
        say(f"  {d:.2e}")
        assert d <= 1e-11
