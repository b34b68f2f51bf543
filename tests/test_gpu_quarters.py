"""FP64 sums at one target per lane in quarters of the work items (1,025 to
3,200 points): sizes that fill the last tile to one, two and four quarters and
leave the last source block short, against the FP64 oracle, in both schedules
and with stored chunk counts; and the first size that runs whole items.

Tolerance.  A target's velocity is a sum of N <= 3,300 terms of total size S_i;
N + 110 roundings per side (the sum, the pair term with the split cross
products' factor 1.5) stay below 2^-40 S_i, both sides together 2^-39 S_i."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import eval_dev, say
from tests.test_gpu_wide_records import _term_sizes

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


def _cloud(n):
    """Clusters of 64 points, some of them far apart (both block forms)."""
    rng = np.random.default_rng(n)
    at = rng.uniform(0, 40, (n // 64 + 1, 3))
    X = np.repeat(at, 64, axis=0)[:n] + rng.uniform(0, 1, (n, 3))
    return X, rng.normal(size=(n, 3)), rng.normal(scale=0.1, size=(n, 3))


@pytest.mark.parametrize("n", [1025, 1087, 1088, 1281, 1344, 2047, 3199, 3200, 3201, 3300])
def test_quarters_against_the_oracle(mrs, ctx, n):
    X, f, t = _cloud(n)
    eps = 0.05
    Uo, Wo = oracle.mrs_eval(X, f, t, eps, 1.0)
    SU, SW = _term_sizes(X, f, t, eps)
    was = mrs.mrs_tune_get(ctx, n, mrs.MRS_FP64)
    try:
        for chunks, sched in ((0, 0), (0, 1), (7, 0), (1, 0), (1, 1)):
            say("quarters", n, chunks, sched)
            mrs.mrs_tune_set(ctx, n, mrs.MRS_FP64, 0, 1, chunks, sched)
            for _ in range(2):
                U, W = eval_dev(mrs, ctx, X, f, t, eps, 1.0, mrs.MRS_FP64)
                assert (np.linalg.norm(U - Uo, axis=1) <= 2.0 ** -39 * SU).all()
                assert (np.linalg.norm(W - Wo, axis=1) <= 2.0 ** -39 * SW).all()
    finally:
        mrs.mrs_tune_set(ctx, n, mrs.MRS_FP64, was["mode"], was["targets_per_lane"], was["chunks"], was["schedule"])
