"""Small one-shot evaluations run in one launch; with an output over an input,
or beyond the size limit, they take the pack, pair and reduction kernels.
Both do the same operations in the same order, so the velocities are equal
bit for bit, also through mrs_eval_device_noalloc and in a HIP graph."""
import numpy as np
import pytest

from tests.gpu_util import dev, say

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


def _inputs(n):
    rng = np.random.default_rng(n)
    return [dev(a) for a in (rng.uniform(0, 1, (n, 3)), rng.normal(size=(n, 3)), rng.normal(size=(n, 3)))]


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n", [1, 3, 4, 5, 64, 255, 257, 1023, 1024])
@pytest.mark.parametrize("entry", ["mrs_eval_device", "mrs_eval_device_noalloc"])
def test_one_launch_equals_general_path(mrs, ctx, n, prec, entry):
    import torch

    ev = getattr(mrs, entry)
    X, f, t = _inputs(n)
    s = torch.cuda.Stream()
    U, W = torch.empty_like(X), torch.empty_like(X)
    Uo, Wo = f.clone(), t.clone()  # outputs over the loads: the general path
    torch.cuda.synchronize()
    ev(ctx, n, X, f, t, 0.02, 0.7, prec, U, W, s)
    ev(ctx, n, X, Uo, Wo, 0.02, 0.7, prec, Uo, Wo, s)
    torch.cuda.synchronize()
    say(f"{entry} n={n} prec={prec}")
    assert torch.equal(U, Uo) and torch.equal(W, Wo)


@pytest.mark.parametrize("n", [2048, 2049])
def test_stored_split_configuration_at_the_limit(mrs, n):
    import torch

    c = mrs.mrs_context_create(0)
    try:
        for prec in (0, 1):
            mrs.mrs_tune_set(c, n, prec, 1)  # wave-split
            X, f, t = _inputs(n)
            U, W = torch.empty_like(X), torch.empty_like(X)
            Uo, Wo = f.clone(), t.clone()
            torch.cuda.synchronize()
            mrs.mrs_eval_device(c, n, X, f, t, 0.02, 1.0, prec, U, W, torch.cuda.current_stream())
            mrs.mrs_eval_device(c, n, X, Uo, Wo, 0.02, 1.0, prec, Uo, Wo, torch.cuda.current_stream())
            torch.cuda.synchronize()
            assert torch.equal(U, Uo) and torch.equal(W, Wo)
    finally:
        mrs.mrs_context_destroy(c)


def test_one_launch_in_a_graph(mrs, ctx):
    """Captured once, replayed on changed inputs with eager work between."""
    import torch

    n = 300
    X, f, t = _inputs(n)
    U, W, U1, W1 = (torch.zeros_like(X) for _ in range(4))
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    mrs.mrs_eval_device_noalloc(ctx, n, X, f, t, 0.02, 1.0, 0, U, W, s)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    fresh = mrs.mrs_context_create(0)  # no evaluation outside the capture to wait for
    try:
        with torch.cuda.graph(g, stream=s):
            mrs.mrs_eval_device_noalloc(fresh, n, X, f, t, 0.02, 1.0, 0, U, W, s)
        for k in range(3):
            f.mul_(1.5)
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            mrs.mrs_eval_device(ctx, n, X, f, t, 0.02, 1.0, 0, U1, W1, s)
            torch.cuda.synchronize()
            assert torch.equal(U, U1) and torch.equal(W, W1), k
    finally:
        mrs.mrs_context_destroy(fresh)
