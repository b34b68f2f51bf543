"""Ensembles of at most 64 points step in one launch (k_small_steps); with the
profiler on, and above 64 points, they step stage by stage.  The sums and
operations are the same in the same order, so states, velocities and clocks
have to be equal bit for bit: no tolerance."""
import numpy as np
import pytest

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


def _make(mrs, ctx, F, M, ext=True):
    e = synth.swimmers(F, M=M, box=0.85 * F ** 0.5 + 1.0, seed=F + M)
    rng = np.random.default_rng(F * M)
    f, n = rng.normal(scale=1e-3, size=e.X.shape), rng.normal(scale=1e-4, size=e.X.shape)
    sw = synth.swim_params(e)
    h = mrs.mrs_ensemble_create(ctx, e.offsets, e.X, e.D, f if ext else None, n if ext else None, e.eps, e.mu,
                                rod_of(mrs, sw.rod))
    mrs.mrs_ensemble_set_swimming(ctx, h, sw.wave, None)
    return h


def _same(a, b):
    return all(np.array_equal(np.asarray(x), np.asarray(y)) and np.isfinite(np.asarray(x)).all() for x, y in zip(a, b))


@pytest.mark.parametrize("F,M", [(1, 2), (20, 3), (1, 17), (1, 63), (1, 64), (2, 32), (1, 65)])
def test_whole_steps_equal_stages(mrs, ctx, F, M):
    for prec in (mrs.MRS_FP64, mrs.MRS_FP32C):
        got = []
        for staged in (False, True):
            h = _make(mrs, ctx, F, M, ext=M != 17)
            mrs.mrs_ensemble_set_time(ctx, h, 0.25)
            mrs.mrs_profile_enable(ctx, staged)
            r = []
            for integ in (mrs.MRS_EULER, mrs.MRS_RK2, mrs.MRS_RK4):
                for steps, elastic in ((33, True), (1, False), (0, True)):
                    say("steps", F, M, prec, staged, integ, steps, elastic)
                    mrs.mrs_ensemble_step(ctx, h, integ, 1e-6, steps, prec, elastic)
                    r += [*mrs.mrs_ensemble_get(ctx, h), mrs.mrs_ensemble_get_time(ctx, h)]
            mrs.mrs_ensemble_eval(ctx, h, prec)
            r += mrs.mrs_ensemble_get(ctx, h)
            mrs.mrs_profile_enable(ctx, False)
            mrs.mrs_profile_reset(ctx)
            mrs.mrs_ensemble_destroy(h)
            got.append(r)
        assert _same(*got), (F, M, prec)


@pytest.mark.parametrize("graph", [False, True])
def test_batches_equal_single_ensembles(mrs, ctx, graph):
    sizes = [(1, 64), (3, 9), (1, 5), (2, 32)]
    for extra in ([], [(1, 70)]):  # the second batch steps by stages
        hs = [_make(mrs, ctx, *s) for s in sizes + extra]
        one = [_make(mrs, ctx, *s) for s in sizes + extra]
        for _ in range(3):
            say("batch", graph, len(hs))
            mrs.mrs_batch_step(ctx, hs, mrs.MRS_RK2, 1e-6, 55, mrs.MRS_FP64, True, graph)
        mrs.mrs_batch_eval(ctx, hs, mrs.MRS_FP64)
        for h, o in zip(hs, one):
            mrs.mrs_ensemble_step(ctx, o, mrs.MRS_RK2, 1e-6, 165, mrs.MRS_FP64)
            mrs.mrs_ensemble_eval(ctx, o, mrs.MRS_FP64)
            assert _same(mrs.mrs_ensemble_get(ctx, h), mrs.mrs_ensemble_get(ctx, o))
            mrs.mrs_ensemble_destroy(h)
            mrs.mrs_ensemble_destroy(o)


def test_non_finite_velocities_are_reported(mrs, ctx):
    h = _make(mrs, ctx, 1, 40)
    f = np.zeros((40, 3))
    f[7] = 1e308
    mrs.mrs_ensemble_set_external(ctx, h, f, np.zeros((40, 3)))
    with pytest.raises(mrs.MrsError) as ex:
        mrs.mrs_ensemble_step(ctx, h, mrs.MRS_EULER, 1e-6, 3, mrs.MRS_FP64)
    assert ex.value.status == mrs.MRS_ENUMERIC
    mrs.mrs_ensemble_destroy(h)
