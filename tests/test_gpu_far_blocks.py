"""The block paths of the FP32C tiled pair kernels: source blocks near, far
and remote (beyond 128 eps, where part of H4 rounds away) of the targets,
against the FP64 oracle.  Tolerance: 1e-5 per target in the form max |a - b| /
|b| (Eq. true_err), the bar of MRS_FP32C."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import eval_dev, say

pytestmark = pytest.mark.gpu

EPS = 0.02
# (mode, targets per lane, chunks, schedule)
CFGS = [(0, 1, 0, 0), (0, 2, 0, 0), (2, 1, 0, 0), (0, 1, 0, 1)]


@pytest.fixture(scope="module")
def mrs():
    import paper_2604_12083_amd as m

    return m


def _clusters(gap, seed):
    """Two clouds of 1,090 points each in cubes of side 8 eps whose boxes are
    `gap` eps apart along x (ragged last blocks, every block compact)."""
    rng = np.random.default_rng(seed)
    X = rng.uniform(0, 8 * EPS, (2180, 3))
    X[1090:, 0] += (8 + gap) * EPS
    return X, rng.normal(size=X.shape), rng.normal(size=X.shape)


@pytest.mark.parametrize("gap", [0.0, 3.0, 5.0, 20.0, 127.9, 128.1, 1000.0])
def test_block_paths_match_oracle(mrs, gap):
    X, f, n = _clusters(gap, int(10 * gap))
    c = mrs.mrs_context_create(0)
    try:
        Uo, Wo = oracle.mrs_eval(X, f, n, EPS, 1.0)
        for cfg in CFGS:
            mrs.mrs_tune_set(c, len(X), 1, *cfg)
            U, W = eval_dev(mrs, c, X, f, n, EPS, 1.0, 1)
            eu, ew = oracle.rel_err(U, Uo), oracle.rel_err(W, Wo)
            say(f"gap {gap} cfg {cfg}: U {eu:.2e} W {ew:.2e}")
            assert eu <= 1e-5 and ew <= 1e-5, cfg
    finally:
        mrs.mrs_context_destroy(c)



@pytest.mark.parametrize("gap", [0.0, 20.0, 30.0, 500.0])
def test_fp64_block_paths_match_oracle(mrs, gap):
    """FP64 (1e-12): blocks nearer and farther than four half-diagonals (about
    7 eps each here), one and two targets per lane, both schedules; also at a
    large offset from the origin."""
    c = mrs.mrs_context_create(0)
    try:
        for shift in (0.0, 100.0):
            X, f, n = _clusters(gap, 50 + int(gap))
            X = X + shift
            Uo, Wo = oracle.mrs_eval(X, f, n, EPS, 1.0)
            for cfg in [(0, 1, 0, 0), (0, 2, 0, 0), (0, 2, 0, 1), (0, 1, 7, 0)]:
                mrs.mrs_tune_set(c, len(X), 0, *cfg)
                U, W = eval_dev(mrs, c, X, f, n, EPS, 1.0, 0)
                eu, ew = oracle.rel_err(U, Uo), oracle.rel_err(W, Wo)
                say(f"fp64 gap {gap} shift {shift} cfg {cfg}: U {eu:.2e} W {ew:.2e}")
                assert eu <= 1e-12 and ew <= 1e-12, cfg
    finally:
        mrs.mrs_context_destroy(c)
