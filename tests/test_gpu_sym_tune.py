"""GPU: tuned launch shapes and the pair-symmetric evaluation of one
self-gravitating set: a tuned shape takes its place where the autotuner
measured that to be faster, and not otherwise.  The bits tell which ran."""
import json

import pytest

import nbody_inputs as ics
from gpu_util import dev

pytestmark = pytest.mark.gpu

N, EPS = 25000, 1e-3
SHAPE = dict(tile_j=64, ipt=1, wg=256, split=9, jsrc=0, unroll=0, waves=0)


def _set():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    p = ics.plummer(N, 33, "salpeter")
    return dev(p.pos), dev(p.vel), dev(p.mass), torch.arange(N, dtype=torch.int32, device="cuda")


def _force(s, cache=None, tile=None):
    import paper_0707_0438_amd as nb
    x, v, m, own = s
    with nb.Context(0, tune_cache=cache) as c:
        if tile:
            c.set_tile("ds", **tile)
        return c.force(x, v, x, v, m, EPS, i_self=own)


def _equal(a, b):
    import torch
    return all(torch.equal(u, w) for u, w in zip(a, b))


def test_tuned_shape_and_symmetric_evaluation(tmp_path):
    import paper_0707_0438_amd as nb
    s = _set()
    x, v, m, own = s
    sym, shaped = _force(s), _force(s, tile=SHAPE)
    assert not _equal(sym, shaped)
    cache = tmp_path / "tune.jsonl"
    # not timed (a file without sym_ms); slower; faster
    for sym_ms, want in ((None, sym), (1.5, shaped), (0.5, sym)):
        line = dict(arch="gfx950", prec=1, ni_log2=14, nj_log2=14, **SHAPE, ms=1.0)
        if sym_ms is not None:
            line["sym_ms"] = sym_ms
        cache.write_text(json.dumps(line) + "\n")
        assert _equal(_force(s, str(cache)), want), sym_ms
    # the autotuner's own entry: the set itself, then i and j apart
    cache.unlink()
    with nb.Context(0, tune_cache=str(cache)) as c:
        c.autotune(x, v, x, v, m, EPS, prec="ds", reps=2)
        e = json.loads(cache.read_text())
        assert e["sym_ms"] > 0
        assert _equal(c.force(x, v, x, v, m, EPS, i_self=own), sym) == (e["sym_ms"] <= e["ms"])
        c.autotune(x.clone(), v, x, v, m, EPS, prec="ds", reps=1)
        assert json.loads(cache.read_text())["sym_ms"] == 0


@pytest.mark.parametrize("jsrc,tile_j,wg", [(0, 256, 256), (1, 128, 256)])
def test_tuned_shape_behind_the_symmetric_evaluation(jsrc, tile_j, wg, tmp_path):
    """The kernel launched behind, in a tuned shape with one j-range (so that
    it would write the outputs itself), leaves them as they are; where i_self
    is not the identity it does the work."""
    import torch
    import paper_0707_0438_amd as nb
    s = _set()
    x, v, m, own = s
    shape = dict(tile_j=tile_j, ipt=1, wg=wg, split=1, jsrc=jsrc, unroll=0, waves=0)
    sym, shaped = _force(s), _force(s, tile=shape)
    assert not _equal(sym, shaped)
    cache = tmp_path / "tune.jsonl"
    cache.write_text(json.dumps(dict(arch="gfx950", prec=1, ni_log2=14, nj_log2=14, **shape, ms=1.0, sym_ms=0.5)) + "\n")
    assert _equal(_force(s, str(cache)), sym)
    other = own.clone()
    other[0] = -1
    with nb.Context(0, tune_cache=str(cache)) as c:
        got = c.force(x, v, x, v, m, EPS, i_self=other)
        c.set_tile("ds", **shape)
        assert _equal(got, c.force(x, v, x, v, m, EPS, i_self=other))
        torch.cuda.synchronize()
