"""mrs_rod_forces_device on every form of its offsets (equal lengths, a short
list in the kernel's arguments, a long list on the device) and of its arrays
(loads absent, outputs over inputs, two streams), against the FP64 oracle.

Tolerance: 1e-12 of the largest load (FP64; a point's load is a sum of a few
terms of that size)."""
import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import dev, rod_of, say

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


def _case(lengths, seed):
    rng = np.random.default_rng(seed)
    n = int(np.sum(lengths))
    e = synth.filaments(-(-n // 50), 50, 2.0, seed)
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    X = e.X[:n] + rng.normal(scale=1e-3, size=(n, 3))
    return off, X, e.D[:n].copy(), e.f[:n], e.n[:n], synth.RodParams((0.3, 0.2, 0.1), (1.0, 1.5, 2.0), (0.1, -0.2, 0.3), e.ds)


LENGTHS = {"one": [64], "equal": [51] * 40, "points": [1] * 300, "pairs": [2] * 130, "long": [255, 256, 257, 600],
           "args": [1 + (7 * k) % 90 for k in range(799)], "list": [1 + (5 * k) % 30 for k in range(801)]}


def _check(mrs, off, X, D, rod, f, n, g, m):
    go, mo = oracle.rod_forces(off, X, D, rod, f if f is not None else np.zeros_like(X),
                               n if n is not None else np.zeros_like(X))
    for got, ref in ((g, go), (m, mo)):
        assert np.abs(got.cpu().numpy() - ref).max() <= 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("name", list(LENGTHS))
@pytest.mark.parametrize("loads", ["both", "force", "none"])
def test_offsets_and_loads(mrs, ctx, name, loads):
    import torch

    off, X, D, f, n, rod = _case(LENGTHS[name], 11)
    f, n = (f if loads != "none" else None), (n if loads == "both" else None)
    say(f"rod_forces {name} n={len(X)} loads={loads}")
    dX, dD = dev(X), dev(D)
    g, m = torch.full_like(dX, 7.0), torch.full_like(dX, 7.0)
    args = (dX, dD, rod_of(mrs, rod), None if f is None else dev(f), None if n is None else dev(n))
    s, t = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    mrs.mrs_rod_forces_device(ctx, off, *args, g, m, s)
    g2, m2 = torch.empty_like(g), torch.empty_like(g)
    torch.cuda.synchronize()
    for st in (s, t, s):  # calls on two streams, no wait between them
        mrs.mrs_rod_forces_device(ctx, off, *args, g2, m2, st)
    torch.cuda.synchronize()
    _check(mrs, off, X, D, rod, f, n, g, m)
    assert torch.equal(g, g2) and torch.equal(m, m2)


@pytest.mark.parametrize("over", ["loads", "swapped", "state", "frames"])
def test_outputs_over_inputs(mrs, ctx, over):
    import torch

    off, X, D, f, n, rod = _case([40] * 30, 12)
    dX, dD, df, dn = dev(X), dev(D), dev(f), dev(n)
    g, m = {"loads": (df, dn), "swapped": (dn, df), "state": (dX, torch.empty_like(dX)),
            "frames": (torch.empty_like(dX), dD.view(-1)[1000:1000 + 3 * len(X)].view(-1, 3))}[over]
    torch.cuda.synchronize()
    mrs.mrs_rod_forces_device(ctx, off, dX, dD, rod_of(mrs, rod), df, dn, g, m, torch.cuda.current_stream())
    torch.cuda.synchronize()
    _check(mrs, off, X, D, rod, f, n, g, m)
