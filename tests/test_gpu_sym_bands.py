"""The pair-symmetric evaluation in several bands of block distances (launches
whose sums are added up through the output rows), and the integrators that
take it, against the general kernel.

Both form the same float32 partial sums over the same j-tiles; only the sums
over tiles differ (a two-sum there, float64 here).  A two-sum's low word is a
float32 sum: over k tiles it is off by at most about k 2^-48 of the tiles'
magnitudes, and those are at most a few times the largest row value (a
Plummer sphere's field cancels by a factor of two or three): 4 k 2^-48 of it.
"""
import os
import subprocess

import numpy as np
import pytest

from gpu_util import dev, host

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_0707_0438_amd", "csrc")

# two bands of an odd number of blocks; five of an even one (the half distance
# closes the last); more than 2^20; force-only: two bands of longer blocks
FORCE = [300007, 524288, (1 << 20) + 1]
ACC = [500000]
EPS = 1e-3


@pytest.mark.timeout(300)
def test_sizes_take_several_bands(tmp_path):
    """The sizes below are of the forms named (no GPU): a host program built
    against the library's internal header prints their shapes."""
    from paper_0707_0438_amd import build
    exe = str(tmp_path / "sym_bands")
    cmd = [build.hipcc(), "-O2", "-std=c++17", "-x", "hip", f"--offload-arch={build.ARCH}",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-Wno-unused-command-line-argument", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           os.path.join(ROOT, "tests", "host", "sym_bands.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    args = [str(a) for n in FORCE for a in (n, 0)] + [str(a) for n in ACC for a in (n, 1)]
    out = subprocess.run([exe] + args, capture_output=True, text=True, timeout=60).stdout
    shapes = [[int(w) for w in ln.split()] for ln in out.splitlines()]
    assert len(shapes) == len(FORCE) + len(ACC)
    for n, kind, dists, a_band, block, blocks in shapes:
        assert a_band < dists, (n, kind)
    assert any(b[5] % 2 == 0 for b in shapes) and any(b[5] % 2 == 1 for b in shapes)
    assert any(b[1] == 1 and b[4] > 1024 for b in shapes)


def _set(n, seed=5):
    import torch
    import nbody_inputs
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    p = nbody_inputs.plummer(n, seed, "salpeter")
    return dev(p.pos), dev(p.vel), dev(p.mass)


def _general(ctx, n):
    """Pin the general kernel to the shape it takes by default."""
    t = ctx.get_tile(n, n)
    t["split"] = 0
    ctx.set_tile("ds", **t)
    return t["tile_j"]


def _close(a, b, tol):
    for x, y in zip(a, b):
        x, y = host(x), host(y)
        assert np.max(np.abs(x - y)) <= tol * np.max(np.abs(y))


@pytest.mark.gpu
@pytest.mark.parametrize("n,jerk", [(n, True) for n in FORCE] + [(n, False) for n in ACC])
def test_bands_equal_general(n, jerk):
    """Rows spread over all blocks (every 509th, the first and the last)."""
    import torch
    import paper_0707_0438_amd as nb
    x, v, m = _set(n)
    own = torch.arange(n, dtype=torch.int32, device="cuda")
    rows = torch.cat([torch.arange(0, n - 1, 509, device="cuda"), torch.tensor([n - 1], device="cuda")])
    xr, vr, own_r = x[:, rows].contiguous(), v[:, rows].contiguous(), rows.to(torch.int32)
    with nb.Context(0) as c:
        full = c.force(x, v, x, v, m, EPS, G=1.5, i_self=own) if jerk else c.force_acc(x, x, m, EPS, G=1.5, i_self=own)
        tile = _general(c, n)
        ref = c.force(xr, vr, x, v, m, EPS, G=1.5, i_self=own_r) if jerk else \
            c.force_acc(xr, x, m, EPS, G=1.5, i_self=own_r)
    _close([a[..., rows] for a in full], ref, 4 * -(-n // tile) * 2.0 ** -48)


@pytest.mark.gpu
@pytest.mark.parametrize("n", [24577, 70001])
def test_integrators_equal_general(n):
    """Leapfrog's and the Hermite integrator's evaluations of a whole set.  The
    shared step is so short (2^-20) that the two contexts' predicted states
    are the same but for the last bits of a few, and its forces compare as an
    evaluation's do."""
    import paper_0707_0438_amd as nb
    x, v, m = _set(n)

    def run(c):
        acc, pot = c.leapfrog(x.clone(), v.clone(), m, EPS, 2.0 ** -20, 1)
        h = c.hermite(n, eps=EPS, eta=0.02, prec="ds")
        h.set_state(x, v, m)
        block = h.get_state()
        epot = h.energy()[1]
        h.close()
        h = c.hermite(n, eps=EPS, shared_dt_log2=-20, prec="ds")
        h.set_state(x, v, m)
        h.step()
        shared = h.get_state()
        h.close()
        return [acc, pot, block["a"], block["jerk"], shared["a"], shared["jerk"]], epot

    with nb.Context(0) as c, nb.Context(0) as g:
        tile = _general(g, n)
        got, epot = run(c)
        ref, epot_ref = run(g)
        assert not all((a == b).all() for a, b in zip(got, ref))   # the other order of sums ran
        tol = 4 * -(-n // tile) * 2.0 ** -48
        _close(got, ref, tol)
        assert abs(epot - epot_ref) <= tol * abs(epot_ref)
