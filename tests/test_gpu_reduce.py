"""GPU: the split reduce over many j-ranges of many i.

The same evaluation in one range and in S: the float32 partial sums of the
64-record tiles are the same, their sum is a two-sum in one range and a
float64 sum over ranges else.  A two-sum's low word is a float32 sum, off by
at most about k 2^-48 over k tiles of the tiles' magnitudes; k is 65 here, so
1e-12 of the largest value has room for a factor of four of cancellation."""
import numpy as np
import pytest

from gpu_util import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ni", [512, 577])
@pytest.mark.parametrize("split", [32, 33, 65])
def test_many_ranges_equal_one(ni, split):
    import torch
    import nbody_inputs
    import paper_0707_0438_amd as nb
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    p = nbody_inputs.plummer(4160, 11)
    x, v, m = dev(p.pos), dev(p.vel), dev(p.mass)
    xi, vi = x[:, :ni].contiguous(), v[:, :ni].contiguous()
    own = torch.arange(ni, dtype=torch.int32, device="cuda")
    with nb.Context(0) as c:
        c.set_tile("ds", 64, 1, 128, split=1)
        ref = c.force(xi, vi, x, v, m, 1e-2, i_self=own)
        refa = c.force_acc(xi, x, m, 1e-2, i_self=own)
        c.set_tile("ds", 64, 1, 128, split=split)
        got = c.force(xi, vi, x, v, m, 1e-2, i_self=own)
        gota = c.force_acc(xi, x, m, 1e-2, i_self=own)
    for a, b in list(zip(got, ref)) + list(zip(gota, refa)):
        a, b = host(a), host(b)
        assert np.max(np.abs(a - b)) <= 1e-12 * np.max(np.abs(b))
