"""The tiled pair kernels at sizes whose one-shot evaluations run in one launch:
every comparison here first asserts, from the profile, that the kernel it is about
was launched.  Evaluations reach it through stored chunk counts that differ from
the automatic ones, the automatic ones through a resident ensemble.

Tolerance.  A target's velocity is a sum of N < 3,400 terms of total size S_i; N +
110 roundings per side stay below 2^-40 S_i in FP64, both sides together 2^-39
S_i.  FP32C adds the rounding of positions, loads and pair arithmetic and of
plain sums of up to 64 terms, below 2^-17 S_i (as in test_gpu_wide_records)."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import dev, say
from tests.test_gpu_far_blocks import EPS, _clusters
from tests.test_gpu_quarters import _cloud
from tests.test_gpu_wide_records import _term_sizes

pytestmark = pytest.mark.gpu

TOL = {0: 2.0 ** -39, 1: 2.0 ** -17}
NAME = {(0, 0): "pairs_tile_f64", (1, 0): "pairs_tile_f32c", (1, 2): "pairs_tile_f32c_quad"}


@pytest.fixture()
def mrs():
    import paper_2604_12083_amd as m

    return m


@pytest.fixture()
def ctx(mrs):
    c = mrs.mrs_context_create(0)
    mrs.mrs_profile_enable(c, True)
    yield c
    mrs.mrs_context_destroy(c)


def _launches(mrs, ctx, call):
    """What call returns, and the pair kernels that it launched."""
    mrs.mrs_profile_reset(ctx)
    got = call()
    total = mrs.mrs_profile_query(ctx, "pairs")[0]
    return got, {k for k in ("pairs_split", *NAME.values()) if mrs.mrs_profile_query(ctx, k)[0] == total > 0}


def _eval(mrs, ctx, entry, X, f, n, eps, prec):
    import torch

    dX, df, dn = dev(X), dev(f), dev(n)
    U, W = torch.empty_like(dX), torch.empty_like(dX)
    getattr(mrs, entry)(ctx, len(X), dX, df, dn, eps, 1.0, prec, U, W, torch.cuda.current_stream())
    torch.cuda.synchronize()
    mrs.mrs_context_synchronize(ctx)
    return U.cpu().numpy(), W.cpu().numpy()


def _check(got, X, f, n, eps, prec, tag, ref={}):
    key = (X.tobytes(), eps)
    if key not in ref:
        ref.clear()
        ref[key] = (*oracle.mrs_eval(X, f, n, eps, 1.0), *_term_sizes(X, f, n, eps))
    Uo, Wo, SU, SW = ref[key]
    eu, ew = (np.linalg.norm(a - b, axis=1) / s for a, b, s in ((got[0], Uo, SU), (got[1], Wo, SW)))
    say(f"{tag}: U {eu.max():.1e} W {ew.max():.1e}")
    assert eu.max() <= TOL[prec] and ew.max() <= TOL[prec], tag


def _is(names, prec, mode=0):
    return NAME[prec, mode if prec else 0] in names and "pairs_split" not in names


@pytest.mark.parametrize("gap", [0.0, 3.0, 5.0, 20.0, 127.9, 128.1, 1000.0])
def test_block_paths_of_the_tiled_kernels(mrs, ctx, gap):
    X, f, n = _clusters(gap, 900 + int(10 * gap))
    for prec in (1, 0):
        for cfg in ((0, 1, 9, 0), (0, 1, 9, 1), (0, 2, 9, 0), (0, 2, 9, 1), (2, 1, 9, 0), (2, 1, 9, 1)):
            mrs.mrs_tune_set(ctx, len(X), prec, *cfg)
            got, names = _launches(mrs, ctx, lambda: _eval(mrs, ctx, "mrs_eval_device", X, f, n, EPS, prec))
            assert _is(names, prec, cfg[0]), (cfg, names)
            _check(got, X, f, n, EPS, prec, f"gap {gap} prec {prec} cfg {cfg}")


@pytest.mark.parametrize("prec", [1, 0])
@pytest.mark.parametrize("N", [2560, 3001, 3300])
def test_schedules_give_identical_sums(mrs, ctx, prec, N):
    """Grid and persistent schedule of the same items, allocating and not: bit for
    bit, and the second call of each as the first (the work-queue counters)."""
    X, f, n = _cloud(N)
    for mode, tpl in ((0, 1), (0, 2), (2, 1)):
        got = []
        for sched in (0, 1):
            mrs.mrs_tune_set(ctx, N, prec, mode, tpl, 9, sched)
            for entry in ("mrs_eval_device", "mrs_eval_device_noalloc") * 2:
                g, names = _launches(mrs, ctx, lambda: _eval(mrs, ctx, entry, X, f, n, 0.05, prec))
                assert _is(names, prec, mode), (mode, tpl, sched, names)
                got.append(g)
        _check(got[0], X, f, n, 0.05, prec, f"N {N} prec {prec} mode {mode} tpl {tpl}")
        assert all(np.array_equal(got[0][k], g[k]) for g in got[1:] for k in (0, 1)), (mode, tpl)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("N", [1025, 1281, 2180, 3200, 3201, 3300])
def test_automatic_items_of_ensembles(mrs, ctx, prec, N):
    """The automatic decomposition (FP64: quarters of the items up to 3,200 points,
    whole items beyond), without an entry and stored on both schedules."""
    X, f, n = _cloud(N)
    D = np.tile(np.eye(3).ravel(), (N, 1))
    rod = mrs.rod_params()
    got = []

    def run():
        h = mrs.mrs_ensemble_create(ctx, [0, N], X, D, f, n, 0.05, 1.0, rod)
        try:
            mrs.mrs_ensemble_eval(ctx, h, prec, False)
            return mrs.mrs_ensemble_get(ctx, h)[2:]
        finally:
            mrs.mrs_ensemble_destroy(h)

    auto = mrs.mrs_tune_get(ctx, N, prec)
    for sched in (None, 0, 1):
        if sched is not None:
            mrs.mrs_tune_set(ctx, N, prec, auto["mode"], auto["targets_per_lane"], 0, sched)
        g, names = _launches(mrs, ctx, run)
        assert _is(names, prec), (sched, names)
        got.append(g)
    _check(got[0], X, f, n, 0.05, prec, f"ensemble N {N} prec {prec} {auto}")
    assert all(np.array_equal(got[0][k], g[k]) for g in got[1:] for k in (0, 1))


@pytest.mark.parametrize("offset", [0.0, 1e4, 1e6])
def test_filaments_far_from_the_origin(mrs, ctx, offset):
    """Straight filaments at separations from contact to a few hundred eps,
    crossing ones among them, `offset` eps from the origin (beyond 2^16 eps the hi
    parts of the FP32C positions round by more than a hundredth of eps, and the
    boxes are widened by it): masked, exact and anchored blocks on every form."""
    rng = np.random.default_rng(41)
    M, ds = 64, 1.0 / 64
    eps = 1.5 * ds
    X = []
    for k in range(48):
        d = rng.normal(size=3)
        at = rng.uniform(0.0, 200.0 * eps, 3) if k % 3 else rng.normal(scale=0.5 * eps, size=3) - 0.5 * d / np.linalg.norm(d)
        X.append(at + (np.arange(M) * ds)[:, None] * d / np.linalg.norm(d))
    X = np.concatenate(X) + offset * eps * np.array([0.6, -0.64, 0.48])
    f, n = rng.normal(size=X.shape), rng.normal(size=X.shape)
    for prec in (1, 0):
        for cfg in ((0, 1, 9, 0), (0, 2, 9, 0), (2, 1, 9, 0)):
            mrs.mrs_tune_set(ctx, len(X), prec, *cfg)
            got, names = _launches(mrs, ctx, lambda: _eval(mrs, ctx, "mrs_eval_device", X, f, n, eps, prec))
            assert _is(names, prec, cfg[0]), (cfg, names)
            _check(got, X, f, n, eps, prec, f"offset {offset:g} prec {prec} cfg {cfg}")
