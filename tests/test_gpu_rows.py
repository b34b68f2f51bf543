"""State, loads and time in and out of resident ensembles: every value comes
back bit for bit in the caller's order, at sizes around the 32,768-row pinned
slots, and calls that return before the device has the new values are seen by
every later call (evaluation, Parareal, another stream)."""
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


def _ens(mrs, ctx, n, loads=True, seed=3):
    """n points in filaments of 50 (the last one shorter)."""
    e = synth.filaments(-(-n // 50), 50, 20.0, seed)
    off = np.append(np.arange(0, n, 50), n).astype(np.int32)
    X, D, f, t = (a[:n].copy() for a in (e.X, e.D, e.f, e.n))
    h = mrs.mrs_ensemble_create(ctx, off, X, D, f if loads else None, t if loads else None, e.eps, e.mu,
                                rod_of(mrs, e.rod()))
    return h, off, X, D, f, t


@pytest.mark.parametrize("n", [1, 85, 86, 32767, 32768, 32769, 70001])
def test_state_round_trip(mrs, ctx, n):
    h, _, X, D, _, _ = _ens(mrs, ctx, n)
    try:
        say(f"rows n={n}")
        for k in range(3):
            Xg, Dg, U, W = mrs.mrs_ensemble_get(ctx, h)
            assert np.array_equal(Xg, X) and np.array_equal(Dg, D) and not U.any() and not W.any()
            if k == 0:
                X = X + 1.0
                mrs.mrs_ensemble_set_state(ctx, h, X, None)
            else:
                D = -D
                mrs.mrs_ensemble_set_state(ctx, h, None, D)
    finally:
        mrs.mrs_ensemble_destroy(h)


@pytest.mark.parametrize("n", [300, 33000])
def test_new_loads_in_the_callers_order(mrs, ctx, n):
    """Loads set later give the velocities of an ensemble created with them;
    absent ones are zero."""
    h, off, X, D, f, t = _ens(mrs, ctx, n, loads=False)
    e = synth.filaments(2, 50, 1.0, 1)
    try:
        for fe, te in ((f, t), (f, None), (None, None), (None, t)):
            mrs.mrs_ensemble_set_external(ctx, h, fe, te)
            mrs.mrs_ensemble_eval(ctx, h, mrs.MRS_FP64, False)
            got = mrs.mrs_ensemble_get(ctx, h)[2:]
            g = mrs.mrs_ensemble_create(ctx, off, X, D, np.zeros_like(X) if fe is None else fe, te, e.eps, e.mu,
                                        rod_of(mrs, e.rod()))
            try:
                mrs.mrs_ensemble_eval(ctx, g, mrs.MRS_FP64, False)
                ref = mrs.mrs_ensemble_get(ctx, g)[2:]
            finally:
                mrs.mrs_ensemble_destroy(g)
            assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1])
    finally:
        mrs.mrs_ensemble_destroy(h)


def test_later_calls_see_queued_values(mrs):
    """set_state and set_time directly before Parareal, and before a change
    of stream, give what they give when the context is synchronised between."""
    import torch

    c = mrs.mrs_context_create(0)
    e = synth.swimmers(8, box=3.0, seed=5)
    sw = synth.swim_params(e)
    other = torch.cuda.Stream()
    res = []
    try:
        for wait in (True, False, False):
            h = mrs.mrs_ensemble_create(c, e.offsets, e.X, e.D, None, None, e.eps, e.mu, rod_of(mrs, sw.rod))
            mrs.mrs_ensemble_set_swimming(c, h, sw.wave, sw.lj)
            out = []
            for t in (0.3, 0.7):
                mrs.mrs_ensemble_set_state(c, h, e.X + t, e.D)
                mrs.mrs_ensemble_set_time(c, h, t)
                if wait:
                    mrs.mrs_context_synchronize(c)
                mrs.mrs_parareal(c, h, 3, mrs.MRS_RK2, 1e-6, 2, 1, 1, 0.0, mrs.MRS_FP64)
                out += list(mrs.mrs_ensemble_get(c, h)) + [mrs.mrs_ensemble_get_time(c, h)]
            mrs.mrs_ensemble_set_state(c, h, e.X, e.D)
            mrs.mrs_ensemble_set_time(c, h, 0.1)
            if wait:
                mrs.mrs_context_synchronize(c)
            mrs.mrs_context_set_stream(c, other)
            mrs.mrs_ensemble_step(c, h, mrs.MRS_RK4, 1e-6, 2, mrs.MRS_FP32C, True)
            out += list(mrs.mrs_ensemble_get(c, h)) + [mrs.mrs_ensemble_get_time(c, h)]
            mrs.mrs_context_set_stream(c, None)
            mrs.mrs_ensemble_destroy(h)
            res.append(out)
        for r in res[1:]:
            assert all(np.array_equal(a, b) for a, b in zip(r, res[0]))
    finally:
        mrs.mrs_context_destroy(c)
