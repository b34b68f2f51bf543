"""Evaluations beyond the one-launch sizes in a HIP graph: the work list is part of
the graph, so replays on changed inputs, with other evaluations, allocations and
synchronisations between them, equal the eager call bit for bit."""
import numpy as np
import pytest

from tests.gpu_util import dev, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,n", [(0, 6145), (0, 12800), (1, 3073), (1, 5003), (1, 12800)])
def test_replays_equal_eager_calls(prec, n):
    import torch

    import paper_2604_12083_amd as mrs

    rng = np.random.default_rng(n)
    X, f, t = (dev(a) for a in (rng.uniform(0, 1, (n, 3)), rng.normal(size=(n, 3)), rng.normal(size=(n, 3))))
    U, W, U1, W1 = (torch.zeros_like(X) for _ in range(4))
    Y, V = torch.rand((3 * n, 3), dtype=torch.float64, device=X.device), torch.empty((3 * n, 3), dtype=torch.float64,
                                                                                    device=X.device)
    s = torch.cuda.Stream()
    captured, eager = mrs.mrs_context_create(0), mrs.mrs_context_create(0)
    try:
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            mrs.mrs_eval_device_noalloc(captured, n, X, f, t, 0.02, 1.0, prec, U, W, s)
        for k in range(3):
            f.mul_(1.5)
            mrs.mrs_eval_device_noalloc(eager, 3 * n, Y, Y, Y, 0.02, 1.0, prec, V, torch.empty_like(V))
            mrs.mrs_context_synchronize(eager)
            say(f"replay {k} n={n} prec={prec}")
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            mrs.mrs_eval_device(eager, n, X, f, t, 0.02, 1.0, prec, U1, W1, s)
            torch.cuda.synchronize()
            assert torch.equal(U, U1) and torch.equal(W, W1), k
    finally:
        mrs.mrs_context_destroy(captured)
        mrs.mrs_context_destroy(eager)
