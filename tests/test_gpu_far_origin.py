"""FP64 split cross products far from the origin: a cloud of loads seen by another
one, both moved by up to 10^6 (5 10^7 eps), against the FP64 oracle on the same
(moved) positions.  Sources and targets have to be taken from the same block
centre: a centre rounded for one of them only puts half an ulp of the coordinate
into every r of the block, 6e-11 of distances from 2 to 10 here.

Tolerance.  Only the first cloud carries loads, so a target's velocity is a sum
of n <= 1,700 terms of total size S_i; n + 110 roundings per side (the sum, the
pair term with the split's factor 1.5) stay below 2^-42 S_i, both sides together
2^-41 S_i."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import eval_dev, say
from tests.test_gpu_wide_records import _term_sizes

pytestmark = pytest.mark.gpu

EPS = 0.02


@pytest.mark.parametrize("n", [1090, 1700])  # quarters of the work items, whole items
@pytest.mark.parametrize("gap", [100, 500])
def test_moved_clouds_against_the_oracle(n, gap):
    import paper_2604_12083_amd as mrs

    rng = np.random.default_rng(n + gap)
    X = rng.uniform(0, 8 * EPS, (2 * n, 3))
    X[n:, 0] += (8 + gap) * EPS
    f, t = rng.normal(size=X.shape), rng.normal(scale=0.1, size=X.shape)
    f[n:], t[n:] = 0.0, 0.0
    c = mrs.mrs_context_create(0)
    try:
        mrs.mrs_profile_enable(c, True)
        for shift in (0.0, 1e4, 1e6):
            Y = X + shift
            Uo, Wo = oracle.mrs_field(Y[n:], Y, f, t, EPS, 1.0)
            SU, SW = (s[n:] for s in _term_sizes(Y, f, t, EPS))
            for cfg in ((0, 1, 7, 0), (0, 2, 7, 0), (0, 2, 7, 1)):
                mrs.mrs_tune_set(c, 2 * n, mrs.MRS_FP64, *cfg)
                mrs.mrs_profile_reset(c)
                U, W = (a[n:] for a in eval_dev(mrs, c, Y, f, t, EPS, 1.0, mrs.MRS_FP64))
                assert mrs.mrs_profile_query(c, "pairs_tile_f64")[0] == 1
                eu, ew = np.linalg.norm(U - Uo, axis=1) / SU, np.linalg.norm(W - Wo, axis=1) / SW
                say(f"n {n} gap {gap} shift {shift:g} cfg {cfg}: U {eu.max():.1e} W {ew.max():.1e}")
                assert eu.max() <= 2.0 ** -41 and ew.max() <= 2.0 ** -41, (shift, cfg)
    finally:
        mrs.mrs_context_destroy(c)
