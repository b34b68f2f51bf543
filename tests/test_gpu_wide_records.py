"""FP32C ensembles whose pair sum runs on FP64-kind records (wave-split sizes,
and contact forces up to 3,200 points): both sides of each limit against the
FP64 oracle, overflowing loads still reported, and a batch that mixes the
forms equal to each ensemble alone, bit for bit.

Tolerance.  Contact forces cancel, so a target's error is held against the sum
S_i of the sizes of its terms, not against |U_i|.  With FP64-kind records only
the loads are rounded (each component by at most 2^-24 of itself), so |dU_i| <=
2^-24 S_i, doubled here for the FP64 rounding of records, sums and oracle.
The FP32 path adds the rounding of its pair arithmetic (the relative error of
r, 7 x 2^-24, enters up to the fifth power, plus about ten operations) and of
plain sums of up to 64 terms: below (35 + 10 + 64) 2^-24 < 2^-17."""
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


def _make(mrs, ctx, F, M=51, lj=True):
    e = synth.swimmers(F, M=M, box=0.85 * F ** 0.5 + 1.0, seed=F)
    rng = np.random.default_rng(F)
    f, n = rng.normal(scale=1e-3, size=e.X.shape), rng.normal(scale=1e-4, size=e.X.shape)
    sw = synth.swim_params(e)
    h = mrs.mrs_ensemble_create(ctx, e.offsets, e.X, e.D, f, n, e.eps, e.mu, rod_of(mrs, sw.rod))
    mrs.mrs_ensemble_set_swimming(ctx, h, sw.wave, sw.lj if lj else None)
    return h, e, f, n, sw


def _term_sizes(X, f, n, eps, mu=1.0):
    """Per target the sums of the sizes of its terms of U and Omega."""
    fs, ns = np.linalg.norm(f, axis=1), np.linalg.norm(n, axis=1)
    SU, SW = np.empty(len(X)), np.empty(len(X))
    for i, x in enumerate(X):
        r2 = ((x - X) ** 2).sum(1)
        r, R = np.sqrt(r2), np.sqrt(r2 + eps * eps)
        h1, h2 = (r2 + 2 * eps ** 2) / R ** 3, 1 / R ** 3
        h3 = (2 * r2 + 5 * eps ** 2) / (2 * R ** 5)
        h4 = np.abs(10 * eps ** 4 - 7 * eps ** 2 * r2 - 2 * r2 ** 2) / (4 * R ** 7)
        h5 = 3 * (2 * r2 + 7 * eps ** 2) / (4 * R ** 7)
        SU[i] = ((h1 + h2 * r2) * fs + h3 * r * ns).sum()
        SW[i] = (h3 * r * fs + (h4 + h5 * r2) * ns).sum()
    return SU / (8 * np.pi * mu), SW / (8 * np.pi * mu)


@pytest.mark.parametrize("F,M,lj", [(20, 51, True), (21, 51, True), (64, 50, True), (66, 50, True), (20, 51, False),
                                    (21, 51, False)])
def test_both_sides_of_the_limits(mrs, ctx, F, M, lj):
    """1,020 / 1,071 points (wave-split limit) and 3,200 / 3,300 (contact)."""
    h, e, f, n, sw = _make(mrs, ctx, F, M, lj)
    try:
        mrs.mrs_ensemble_eval(ctx, h, mrs.MRS_FP32C, False)
        U, W = mrs.mrs_ensemble_get(ctx, h)[2:]
    finally:
        mrs.mrs_ensemble_destroy(h)
    g = f + oracle.lj_forces(e.offsets, e.X, sw.lj) if lj else f
    Uo, Wo = oracle.mrs_eval(e.X, g, n, e.eps, e.mu)
    wide = e.N <= 1024 or (lj and e.N <= 3200)
    tol = 2.0 ** -23 if wide else 2.0 ** -17
    SU, SW = _term_sizes(e.X, g, n, e.eps, e.mu)
    eu, ew = ((np.linalg.norm(a - b, axis=1) / s).max() for a, b, s in ((U, Uo, SU), (W, Wo, SW)))
    say(f"N={e.N} lj={lj}: U {eu:.2e} W {ew:.2e} of the terms (tolerance {tol:.2e})")
    assert eu <= tol and ew <= tol


@pytest.mark.parametrize("F", [2, 30])
def test_overflowing_loads_are_reported(mrs, ctx, F):
    h, e, f, n, _ = _make(mrs, ctx, F)
    try:
        mrs.mrs_ensemble_set_external(ctx, h, 1e44 * f, n)  # about 1e42: beyond FP32 in units of eps
        with pytest.raises(mrs.MrsError) as ei:
            mrs.mrs_ensemble_eval(ctx, h, mrs.MRS_FP32C, False)
        assert ei.value.status == mrs.MRS_ENUMERIC
    finally:
        mrs.mrs_ensemble_destroy(h)


def test_mixed_batch_equals_alone(mrs, ctx):
    mk = lambda: [_make(mrs, ctx, F, lj=lj)[0] for F, lj in ((3, True), (25, True), (30, False), (70, True), (10, False))]
    a, b = mk(), mk()
    try:
        for k in range(3):
            mrs.mrs_batch_step(ctx, a, mrs.MRS_RK2, 1e-6, 2, mrs.MRS_FP32C, True, use_graph=True)
            for h in b:
                mrs.mrs_ensemble_step(ctx, h, mrs.MRS_RK2, 1e-6, 2, mrs.MRS_FP32C, True)
            for x, y in zip(a, b):
                assert all(np.array_equal(p, q) for p, q in zip(mrs.mrs_ensemble_get(ctx, x), mrs.mrs_ensemble_get(ctx, y)))
    finally:
        for h in a + b:
            mrs.mrs_ensemble_destroy(h)
