"""GPU: the pair-symmetric evaluation of one self-gravitating set against the
general kernel in the default launch shape.

Both form the same float32 partial sums over the same j-tiles; only the sums
over tiles differ (compensated float32 there, float64 here).  A two-sum's low
word is a float32 sum: over k tiles it is off by at most about k 2^-48 of the
tiles' magnitudes.  k is at most 1100 here, so 1e-11 of the largest row value
bounds the difference with room for cancellation between tiles (a factor of
two or three in a Plummer sphere).
"""
import numpy as np
import pytest

from gpu_util import dev, host

pytestmark = pytest.mark.gpu
TOL = 1e-11


def setup_module(module):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"


def _set(n, seed=3):
    import nbody_inputs
    p = nbody_inputs.plummer(n, seed, "salpeter")
    return dev(p.pos), dev(p.vel), dev(p.mass)


def _general(ctx, n):
    """Pin the general kernel to the shape it takes by default."""
    t = ctx.get_tile(n, n)
    t["split"] = 0
    ctx.set_tile("ds", **t)


def _close(a, b):
    for x, y in zip(a, b):
        x, y = host(x), host(y)
        assert np.max(np.abs(x - y)) <= TOL * np.max(np.abs(y))


# smallest size; odd sizes; even and odd numbers of blocks; the last block
# full, one particle, one short; both fold intervals
@pytest.mark.parametrize("n", [24576, 24577, 25600, 26623, 40001, 65535, 65536, 66561, 70001])
def test_pair_symmetric_equals_general(n):
    import torch
    import paper_0707_0438_amd as nb
    x, v, m = _set(n)
    idx = torch.arange(n, dtype=torch.int32, device="cuda")
    with nb.Context(0) as c, nb.Context(0) as g:
        _general(g, n)
        full = c.force(x, v, x, v, m, 1e-3, G=1.5, i_self=idx)
        again = c.force(x, v, x, v, m, 1e-3, G=1.5, i_self=idx)
        acc = c.force_acc(x, x, m, 1e-3, G=1.5, i_self=idx)
        ref = g.force(x, v, x, v, m, 1e-3, G=1.5, i_self=idx)
        refa = g.force_acc(x, x, m, 1e-3, G=1.5, i_self=idx)
        for a, b in zip(full, again):
            assert torch.equal(a, b)
        _close(full, ref)
        _close(acc, refa)


def test_other_i_self_takes_the_general_kernel():
    """i_self is checked on the device: not the identity, absent, and back."""
    import torch
    import paper_0707_0438_amd as nb
    n = 25000
    x, v, m = _set(n)
    idx = torch.arange(n, dtype=torch.int32, device="cuda")
    none = idx.clone()
    none[n - 1] = -1
    with nb.Context(0) as c, nb.Context(0) as g:
        _general(g, n)
        for s in (none, idx.flip(0).contiguous(), None):
            for a, b in zip(c.force(x, v, x, v, m, 1e-2, i_self=s), g.force(x, v, x, v, m, 1e-2, i_self=s)):
                assert torch.equal(a, b)
        _close(c.force(x, v, x, v, m, 1e-2, i_self=idx), g.force(x, v, x, v, m, 1e-2, i_self=idx))


def test_bands_of_distances():
    """2^18 + 1 bodies against sampled rows of the general kernel: several
    launches whose rows are added up."""
    import torch
    import paper_0707_0438_amd as nb
    n = (1 << 18) + 1
    x, v, m = _set(n)
    idx = torch.arange(n, dtype=torch.int32, device="cuda")
    rows = torch.arange(0, n, 257, device="cuda")
    with nb.Context(0) as c:
        full = c.force(x, v, x, v, m, 1e-3, i_self=idx)
        # a small i-list takes the same 256-record tiles when pinned to them
        t = c.get_tile(n, n)
        t["split"] = 0
        c.set_tile("ds", **t)
        sub = c.force(x[:, rows].contiguous(), v[:, rows].contiguous(), x, v, m, 1e-3,
                      i_self=rows.to(torch.int32))
        _close([a[..., rows] for a in full], sub)
