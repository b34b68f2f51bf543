"""Lennard-Jones forces by both routes: one launch with the rod forces (up to
3,200 points in 64 source blocks, pair kernels without a mask) and the general
kernels, at the limits of each: 64 and 65 source blocks, filaments of several
blocks, filaments longer than the 127 nodes of a rod pass, blocks of 64 targets
with more than four filaments, the last target block not full.

Tolerance.  A pair force is a difference, 24 e (2 s^12 - s^6)/r with s =
sigma/r, of about 20 roundings entering at most to the 12th power: below 64 x
2^-53 of t = 24 e (4 s^12 + s^6)/r on either side.  With T_j = |f_j| + sum of t
over the neighbours as the size of a point's force, the velocity of a target is
a sum of N <= 4,000 terms of total size S_i(T); N + 64 + 70 roundings (the sum,
the force, the pair term) on either side stay below 2^-40 S_i.  FP32C adds its
own: 2^-23 S_i on FP64-kind records, 2^-17 S_i on the FP32 path."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import dev, rod_of, say
from tests.test_gpu_wide_records import _term_sizes

pytestmark = pytest.mark.gpu
SIG, EN, EPS, DS = 0.24, 1e-4, 0.08, 0.02


@pytest.fixture(scope="module")
def mrs():
    import paper_2604_12083_amd as m

    return m


@pytest.fixture(scope="module")
def ctx(mrs):
    c = mrs.mrs_context_create(0)
    yield c
    mrs.mrs_context_destroy(c)


class _Rod:
    a, b, omega0, ds = (1e-3, 1e-3, 1e-3), (0.5, 0.5, 0.5), (0.0, 0.3, 0.1), DS


def _scene(F, M, seed):
    """F nearly straight, nearly parallel rods of M points, in contact with their neighbours."""
    rng = np.random.default_rng(seed)
    X, D = np.empty((F, M, 3)), np.empty((F, M, 3, 3))
    w = int(np.ceil(F ** 0.5))
    place = rng.permutation(w * w)[:F]  # a square lattice, in any order
    place[:2] = (0, 1) if F == 2 else place[:2]
    s = (np.arange(M) - 0.5 * M) * DS
    for f in range(F):
        tilt, turn = rng.uniform(-0.05, 0.05, 2) / max(1.0, M * DS), rng.uniform(0, 2 * np.pi)
        d3 = np.array([*tilt, 1.0]) / np.sqrt(1 + tilt @ tilt)
        d1 = np.array([np.cos(turn), np.sin(turn), 0.0])
        d1 -= (d1 @ d3) * d3
        d1 /= np.linalg.norm(d1)
        q = np.array([d1, np.cross(d3, d1), d3])
        at = SIG * np.array([place[f] % w, place[f] // w, 0.0]) + rng.uniform(-0.01, 0.01, 3)
        X[f] = at + s[:, None] * d3 + 0.01 * np.sin(7 * s)[:, None] * d1
        D[f] = q
    f, n = rng.normal(scale=1e-3, size=(F * M, 3)), rng.normal(scale=1e-4, size=(F * M, 3))
    return np.arange(F + 1, dtype=np.int32) * M, X.reshape(-1, 3), D.reshape(-1, 3, 3), f, n


def _force_sizes(off, X):
    fil = np.repeat(np.arange(len(off) - 1), np.diff(off))
    T = np.zeros(len(X))
    for i, x in enumerate(X):
        r = np.linalg.norm(x - X, axis=1)
        k = (fil != fil[i]) & (r < 2 ** (1 / 6) * SIG)
        s6 = (SIG / r[k]) ** 6
        T[i] = (24 * EN * (4 * s6 * s6 + s6) / r[k]).sum()
    return T


@pytest.mark.parametrize("F,M", [(2, 51), (25, 51), (64, 49), (65, 49), (32, 100), (10, 130), (2, 700), (100, 3),
                                 (40, 90), (24, 128), (20, 129)])
def test_lj_velocities(mrs, ctx, F, M):
    import torch

    off, X, D, f, n = _scene(F, M, F * M)
    flj = oracle.lj_forces(off, X, (SIG, EN))
    T = _force_sizes(off, X)
    assert T.any()
    Uo, Wo = oracle.mrs_eval(X, f + flj, n, EPS, 1.0)
    SU, SW = _term_sizes(X, np.linalg.norm(f, axis=1)[:, None] + T[:, None], n, EPS)
    h = mrs.mrs_ensemble_create(ctx, off, X, D, f, n, EPS, 1.0, rod_of(mrs, _Rod))
    mrs.mrs_ensemble_set_swimming(ctx, h, None, (SIG, EN))
    wide = F * M <= 3200
    for prec, tol in ((mrs.MRS_FP64, 2.0 ** -40), (mrs.MRS_FP32C, 2.0 ** -23 if wide else 2.0 ** -17)):
        say("lj", F, M, prec)
        mrs.mrs_ensemble_eval(ctx, h, prec, False)
        U, W = mrs.mrs_ensemble_get(ctx, h)[2:]
        eu, ew = ((np.linalg.norm(a - b, axis=1) / s).max() for a, b, s in ((U, Uo, SU), (W, Wo, SW)))
        say(f"  U {eu:.2e} W {ew:.2e} of the terms (tolerance {tol:.2e})")
        assert eu <= tol and ew <= tol
    # with the rod forces: as if they were external loads, but for the order
    # of the sums
    mrs.mrs_ensemble_eval(ctx, h, mrs.MRS_FP64, True)
    U, W = mrs.mrs_ensemble_get(ctx, h)[2:]
    g, m = torch.empty_like(dev(X)), torch.empty_like(dev(X))
    mrs.mrs_rod_forces_device(ctx, off, dev(X), dev(D), rod_of(mrs, _Rod), dev(f), dev(n), g, m,
                              torch.cuda.current_stream())
    torch.cuda.synchronize()
    g, m = g.cpu().numpy(), m.cpu().numpy()
    mrs.mrs_ensemble_set_external(ctx, h, g, m)
    mrs.mrs_ensemble_eval(ctx, h, mrs.MRS_FP64, False)
    U1, W1 = mrs.mrs_ensemble_get(ctx, h)[2:]
    SU, SW = _term_sizes(X, np.linalg.norm(g, axis=1)[:, None] + np.linalg.norm(f, axis=1)[:, None] + T[:, None], m, EPS)
    assert (np.linalg.norm(U - U1, axis=1) <= 2.0 ** -40 * SU).all()
    assert (np.linalg.norm(W - W1, axis=1) <= 2.0 ** -40 * SW).all()
    mrs.mrs_ensemble_destroy(h)


@pytest.mark.parametrize("mode,tpl,sched", [(0, 1, 0), (0, 1, 1), (0, 2, 0), (0, 2, 1), (2, 1, 0), (2, 1, 1)])
def test_contact_sources_in_every_fp32_form(mrs, mode, tpl, sched):
    """The FP32 path above 3,200 points: tiles, two targets per lane and the
    four-wave split, in both schedules."""
    off, X, D, f, n = _scene(40, 90, 3600)
    flj = oracle.lj_forces(off, X, (SIG, EN))
    Uo, Wo = oracle.mrs_eval(X, f + flj, n, EPS, 1.0)
    SU, SW = _term_sizes(X, f + flj, n, EPS)
    c = mrs.mrs_context_create(0)
    try:
        mrs.mrs_tune_set(c, len(X), mrs.MRS_FP32C, mode, tpl, 0, sched)
        h = mrs.mrs_ensemble_create(c, off, X, D, f, n, EPS, 1.0, rod_of(mrs, _Rod))
        mrs.mrs_ensemble_set_swimming(c, h, None, (SIG, EN))
        say("contact", mode, tpl, sched)
        mrs.mrs_ensemble_eval(c, h, mrs.MRS_FP32C, False)
        U, W = mrs.mrs_ensemble_get(c, h)[2:]
        mrs.mrs_ensemble_destroy(h)
    finally:
        mrs.mrs_context_destroy(c)
    assert (np.linalg.norm(U - Uo, axis=1) <= 2.0 ** -17 * SU).all()
    assert (np.linalg.norm(W - Wo, axis=1) <= 2.0 ** -17 * SW).all()
