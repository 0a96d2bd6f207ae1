"""Strategies long enough for P's map copies and the sliced P^T (2^22 samples, 256 per
pixel and 2,048 slice waves), registered one after another on one context, whose builds
reuse the device memory of earlier ones: P and P^T bit by bit those of a fresh context,
and the oracle's (sums of at most 600 terms of order one: 1e-12).  The grid is set for
another width, dropped and set again, with shorter builds in between."""
import numpy as np
import pytest

import oracle as O
from gpu_util import dev, host, maxrel

pytestmark = pytest.mark.gpu


def _strategy(n, side, seed):
    """Row and column scans in turn: two scan directions."""
    rng = np.random.default_rng(seed)
    t = np.arange(n)
    u, b = t % side, (t // side) % side
    a = np.where((t // side) % 2 == 0, u, side - 1 - u)
    pix = np.where((t // (side * side)) % 2 == 0, b * side + a, a * side + b).astype(np.int32)
    pix[rng.random(n) < 0.1] = -1
    return pix, rng.uniform(0.0, np.pi, n)


@pytest.mark.parametrize("stokes,prec", [("IQU", 0), ("IQU", 1), ("QU", 0), ("I", 1)])
def test_layouts_on_reused_memory(stokes, prec):
    import torch
    from paper_1801_08937_amd import mapmaker as mm
    dt = torch.float32 if prec else torch.float64
    tol = 2e-5 if prec else 1e-12
    ctx = mm.Context(0)

    def build(c, pix, psi, side, grids):
        lp = c.pointing(dev(pix), None if stokes == "I" else dev(psi), side * side, 3, prec,
                        stokes=stokes)
        for w in grids:
            lp.set_grid(w)
        return lp

    for k, (n, side, grids) in enumerate([(1 << 23, 128, (128,)), (300007, 32, (32,)),
                                          (5500003, 110, (55, 110)), (4097, 32, (32, 0)),
                                          (1 << 23, 128, (128, 0)),
                                          (6000011, 110, (110, 0, 110))]):
        pix, psi = _strategy(n, side, k)
        lp = build(ctx, pix, psi, side, grids)
        if n > 1 << 22:
            assert lp.pt_layout()[0] > 0
            assert lp.p_copies() == (2 if grids[-1] == side else 0)
        g = torch.Generator(device="cuda").manual_seed(k)
        x = torch.randn(lp.n, generator=g, device="cuda", dtype=torch.float64)
        z = torch.randn(n, generator=g, device="cuda", dtype=torch.float64).to(dt)
        y, b = ctx.apply_P(lp, x), ctx.apply_PT(lp, z)
        fresh = mm.Context(0)
        lf = build(fresh, pix, psi, side, grids[-1:])
        assert lf.pt_layout() == lp.pt_layout() and lf.p_copies() == lp.p_copies()
        assert torch.equal(y, fresh.apply_P(lf, x))
        assert torch.equal(b, fresh.apply_PT(lf, z))
        lf.close()
        fresh.close()
        op = O.pointing_build(pix, None if stokes == "I" else psi, side * side, 3, stokes)
        assert maxrel(host(y), O.apply_P(op, host(x))) <= tol
        assert maxrel(host(b), O.apply_PT(op, host(z).astype(np.float64))) <= tol
        lp.close()
    ctx.close()
