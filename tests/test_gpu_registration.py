"""Registering scan strategies one after another on one context: every build reuses
the device memory of earlier ones of other sizes, so what it writes may not depend on
what that memory held.  Whole-number outputs equal the oracle's; P and P^T are compared
bit by bit with a fresh context's, and with the oracle (sums of at most a few thousand
terms of order one: 1e-12)."""
import numpy as np
import pytest

import oracle as O
from gpu_util import dev, host, maxrel

pytestmark = pytest.mark.gpu


def _strategy(n, side, seed):
    rng = np.random.default_rng(seed)
    t = np.arange(n)
    u = t % side
    a, b = np.where((t // side) % 2 == 0, u, side - 1 - u), (t // side) % side
    pix = np.where((t // (side * side)) % 2 == 0, b * side + a, a * side + b).astype(np.int32)
    pix[rng.random(n) < 0.2] = -1
    return pix, rng.uniform(0.0, np.pi, n)


def _build(ctx, pix, psi, side, min_hits, stokes, grid):
    lp = ctx.pointing(dev(pix), None if stokes == "I" else dev(psi), side * side, min_hits, 0,
                      stokes=stokes)
    for width in grid:
        lp.set_grid(width)
    return lp


@pytest.mark.parametrize("stokes", ["IQU", "QU", "I"])
def test_builds_on_one_context(stokes):
    import torch
    from paper_1801_08937_amd import mapmaker as mm
    ctx = mm.Context(0)
    # large, small, large again; pixels below min_hits, single samples, a layout
    # rebuilt for another width, and one dropped again
    for k, (n, side, mh, grid) in enumerate([(300007, 32, 3, (32,)), (1, 1, 1, ()), (65, 5, 3, (5,)),
                                             (70001, 64, 14, (64, 16)), (2, 1, 3, (1,)),
                                             (300007, 96, 27, (96,)), (4097, 32, 4, (32, 0)),
                                             (150001, 32, 1, (7, 32))]):
        pix, psi = _strategy(n, side, k)
        if n < 3:
            pix[:] = 0
        op = O.pointing_build(pix, None if stokes == "I" else psi, side * side, mh, stokes)
        lp = _build(ctx, pix, psi, side, mh, stokes, grid)
        hits, obs = lp.hits()
        j, perm, off = lp.export()
        for got, want in ((hits, op.hits), (obs, op.obs_pix), (j, op.j), (perm, op.perm),
                          (off, op.off)):
            np.testing.assert_array_equal(host(got), want)
        if op.n == 0:
            continue
        rng = np.random.default_rng(100 + k)
        x, y = rng.standard_normal(op.n), rng.standard_normal(n)
        px, pty = ctx.apply_P(lp, dev(x)), ctx.apply_PT(lp, dev(y))
        assert maxrel(host(px), O.apply_P(op, x)) <= 1e-12
        assert maxrel(host(pty), O.apply_PT(op, y)) <= 1e-12
        other = mm.Context(0)
        lo = _build(other, pix, psi, side, mh, stokes, grid[-1:])
        assert lo.pt_layout() == lp.pt_layout() and lo.p_copies() == lp.p_copies()
        assert torch.equal(px, other.apply_P(lo, dev(x)))
        assert torch.equal(pty, other.apply_PT(lo, dev(y)))
        # refused as before, and the context still works
        for bad in (-2, side * side):
            wrong = pix.copy()
            wrong[n // 2] = bad
            with pytest.raises(mm.MapmakerError):
                _build(ctx, wrong, psi, side, mh, stokes, ())
        assert torch.equal(px, ctx.apply_P(lp, dev(x)))
        lo.close()
        other.close()
        lp.close()
    ctx.close()


def test_kept_memory_is_bounded():
    """Strategies of many sizes, made and dropped: what stays allocated is at most the
    1 GiB that the library keeps per device and one context's own workspaces (0.5 GiB)."""
    import torch
    from paper_1801_08937_amd import mapmaker as mm
    ctx = mm.Context(0)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    before = torch.cuda.mem_get_info()[0]
    for k in range(8):
        n = (1 << 21) + 400000 * k
        pix, psi = _strategy(n, 64, k)
        lp = _build(ctx, pix, psi, 64, 3, "IQU", (64,))
        lp.close()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    assert before - torch.cuda.mem_get_info()[0] <= 3 << 29
    ctx.close()
