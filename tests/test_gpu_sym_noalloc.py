"""GPU: nbody_force_noalloc of a self-gravitating set that nbody_force
evaluates pair by pair."""
import numpy as np
import pytest

import nbody_inputs as ics
from gpu_util import dev, host

pytestmark = pytest.mark.gpu


def test_noalloc_keeps_the_general_kernel():
    """The general kernel's bits in its default shape (whose partials fit the
    64 MiB), and nbody_force's values to the rounding of the sums over tiles:
    4 k 2^-48 of the largest over k tiles, the low word of a two-sum being a
    float32 sum."""
    import torch
    import paper_0707_0438_amd as nb
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    n = 30000
    p = ics.plummer(n, 34, "salpeter")
    x, v, m = dev(p.pos), dev(p.vel), dev(p.mass)
    own = torch.arange(n, dtype=torch.int32, device="cuda")
    with nb.Context(0) as c:
        got = c.force(x, v, x, v, m, 1e-3, i_self=own, noalloc=True)
        full = c.force(x, v, x, v, m, 1e-3, i_self=own)
        t = c.get_tile(n, n)
        t["split"] = 0
        c.set_tile("ds", **t)
        ref = c.force(x, v, x, v, m, 1e-3, i_self=own)
    for a, b, f in zip(got, ref, full):
        assert torch.equal(a, b)
        a, f = host(a), host(f)
        assert np.max(np.abs(a - f)) <= 4 * -(-n // t["tile_j"]) * 2.0 ** -48 * np.max(np.abs(f))
