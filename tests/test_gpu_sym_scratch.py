"""GPU: scratch of the pair-symmetric evaluation.  NBODY_DEBUG_FAIL_ALLOC=k
fails the k-th device allocation of a context from the host; where the rows
cannot be had the general kernel runs, whose sums over tiles are formed in
another order, so the bits tell which of the two ran."""
import pytest

import nbody_inputs as ics
from gpu_util import dev

pytestmark = pytest.mark.gpu

EPS = 1e-3


def _set(n):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    p = ics.plummer(n, 31, "salpeter")
    return dev(p.pos), dev(p.vel), dev(p.mass), torch.arange(n, dtype=torch.int32, device="cuda")


def _equal(a, b):
    import torch
    return all(torch.equal(u, w) for u, w in zip(a, b))


@pytest.mark.parametrize("n", [25000, 65535])
def test_reserved_set_allocates_nothing(n, monkeypatch):
    """After nbody_reserve(n, n), with its four allocations (i records, j
    records, rows, flag), no evaluation of n bodies allocates."""
    import paper_0707_0438_amd as nb
    x, v, m, own = _set(n)
    with nb.Context(0) as c:
        ref = c.force(x, v, x, v, m, EPS, i_self=own)
        refa = c.force_acc(x, x, m, EPS, i_self=own)
    monkeypatch.setenv("NBODY_DEBUG_FAIL_ALLOC", "5")
    with nb.Context(0) as c:
        c.reserve(n, n)
        assert _equal(c.force(x, v, x, v, m, EPS, i_self=own), ref)
        assert _equal(c.force_acc(x, x, m, EPS, i_self=own), refa)


def test_destroy_returns_every_allocation():
    """2000 contexts that each made the flag of the identity check (nbody_reserve
    of a set that size): the smallest device allocation is 4 KiB, so one kept
    by each would take 8 MiB of the free memory; 4 MiB are allowed for what
    the runtime keeps."""
    import torch
    import paper_0707_0438_amd as nb

    def once():
        with nb.Context(0) as c:
            for prec in ("ds", "fp32"):   # no rows, no partials: the flag and the records alone
                c.set_tile(prec, 64, 1, 128, split=1)
            c.reserve(24576, 24576)

    for _ in range(50):
        once()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info(0)[0]
    for _ in range(2000):
        once()
    torch.cuda.synchronize()
    assert before - torch.cuda.mem_get_info(0)[0] < 4 << 20


def test_rows_that_cannot_be_had_are_not_asked_for_again(monkeypatch):
    """The rows' allocation (the third: flag, records, rows) fails: this call
    and the later ones of that size take the general kernel, and the error
    text of an earlier call stays."""
    import paper_0707_0438_amd as nb
    n = 25000
    x, v, m, own = _set(n)
    with nb.Context(0) as g:
        sym = g.force(x, v, x, v, m, EPS, i_self=own)
        t = g.get_tile(n, n)
        t["split"] = 0
        g.set_tile("ds", **t)
        ref = g.force(x, v, x, v, m, EPS, i_self=own)
        assert not _equal(sym, ref)
    monkeypatch.setenv("NBODY_DEBUG_FAIL_ALLOC", "3")
    with nb.Context(0) as c:
        with pytest.raises(nb.NBodyError):
            c.force(x, v, x, v, m, -1.0, i_self=own)
        text = c.last_error()
        assert text
        for _ in range(3):
            assert _equal(c.force(x, v, x, v, m, EPS, i_self=own), ref)
        assert c.last_error() == text


@pytest.mark.parametrize("k", [3, 4])
def test_reserve_without_room_for_the_rows(k, monkeypatch):
    """nbody_reserve whose flag or rows (its third and fourth allocation)
    cannot be had succeeds, and the set takes the general kernel; reserved
    again, with room, it is evaluated pair by pair."""
    import paper_0707_0438_amd as nb
    n = 25000
    x, v, m, own = _set(n)
    with nb.Context(0) as g:
        sym = g.force(x, v, x, v, m, EPS, i_self=own)
        t = g.get_tile(n, n)
        t["split"] = 0
        g.set_tile("ds", **t)
        ref = g.force(x, v, x, v, m, EPS, i_self=own)
    monkeypatch.setenv("NBODY_DEBUG_FAIL_ALLOC", str(k))
    with nb.Context(0) as c:
        c.reserve(n, n)
        assert _equal(c.force(x, v, x, v, m, EPS, i_self=own), ref)
        c.reserve(n, n)
        assert _equal(c.force(x, v, x, v, m, EPS, i_self=own), sym)
