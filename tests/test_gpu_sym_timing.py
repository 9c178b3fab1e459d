"""GPU: kernel timing of a self-gravitating set that the general kernel
evaluates after all, since the device finds i_self not to be the identity."""
import pytest

import nbody_inputs as ics
from gpu_util import dev

pytestmark = pytest.mark.gpu


def test_timing_covers_the_kernel_that_did_the_work():
    """The set's evaluation with i_self[n - 1] = -1 does the pinned general
    kernel's work: more than half its time is reported.  With the identity
    each pair is evaluated once, a quarter of its time is a safe bound."""
    import torch
    import paper_0707_0438_amd as nb
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    n, calls = 40000, 5
    p = ics.plummer(n, 32)
    x, v, m = dev(p.pos), dev(p.vel), dev(p.mass)
    own = torch.arange(n, dtype=torch.int32, device="cuda")
    other = own.clone()
    other[n - 1] = -1

    def timed(c, i_self):
        c.force(x, v, x, v, m, 1e-3, i_self=i_self)
        c.kernel_timing(True)
        for _ in range(calls):
            c.force(x, v, x, v, m, 1e-3, i_self=i_self)
        ms, launches = c.kernel_time()
        c.kernel_timing(False)
        assert launches == calls
        return ms

    with nb.Context(0) as c, nb.Context(0) as g:
        t = g.get_tile(n, n)
        t["split"] = 0
        g.set_tile("ds", **t)
        general = timed(g, other)
        assert timed(c, other) > 0.5 * general
        assert timed(c, own) > 0.25 * general
