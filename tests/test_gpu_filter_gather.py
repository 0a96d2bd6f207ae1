"""A = P^T F P with the template filter gathering the map itself (one column,
orders to 3, subscans to 1,024 samples) against P, F and P^T applied one after the
other, at the edges of the register cache's sizes and past them, for all map
components, with and without ground templates; and the allocation-free apply,
which lays the same buffers out differently, against the plain one (same bits).

P, F and P^T sum at most a few hundred terms of order one; the two ways differ in
the rounding of the gathered value only: 1e-13 in FP64, 1e-5 in FP32."""
import numpy as np
import pytest

from gpu_util import dev, host, maxrel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1801_08937_amd import mapmaker as mm
    return mm.Context(0)


@pytest.mark.parametrize("sub", [5, 64, 65, 129, 256, 257, 385, 512, 513, 1024, 1025])
@pytest.mark.parametrize("stokes,prec,order,ground", [
    ("IQU", 0, 2, True), ("IQU", 1, 3, False), ("QU", 0, 1, True), ("QU", 1, 0, True),
    ("I", 0, 3, False), ("I", 1, 2, True), ("IQU", 0, 4, True)])
def test_filter_gather(ctx, sub, stokes, prec, order, ground):
    import torch
    rng = np.random.default_rng(sub + 7 * order)
    n, side = 30011, 24
    pix = rng.integers(-1, side * side, n).astype(np.int32)
    psi = rng.uniform(0.0, np.pi, n)
    cuts = np.unique(np.concatenate([np.arange(0, n, sub), [n // 3, n]])).astype(np.int64)
    ist = np.array([0, n // 3, n], dtype=np.int64)
    gb = dev(rng.integers(-1, 130, n).astype(np.int32)) if ground else None
    lp = ctx.pointing(dev(pix), None if stokes == "I" else dev(psi), side * side, 3, prec,
                      stokes=stokes)
    for grid in (0, side):
        lp.set_grid(grid)
        nz = ctx.polyfilter(lp, ist, np.array([0.7, 1.9]), cuts, order, gb, 130 if ground else 0)
        x = dev(rng.standard_normal(lp.n))
        a = ctx.apply_A(lp, nz, x)
        b = ctx.apply_PT(lp, ctx.noise_apply(nz, ctx.apply_P(lp, x)))
        assert maxrel(host(a), host(b)) <= (1e-5 if prec else 1e-13)
        c = torch.empty_like(a)
        ctx.apply_A_noalloc(lp, nz, x, c)
        assert torch.equal(a, c)
        x2 = torch.stack([x, 2 * x], 1).reshape(-1).contiguous()
        a2 = ctx.apply_A(lp, nz, x2, nrhs=2)
        c2 = torch.empty_like(a2)
        ctx.apply_A_noalloc(lp, nz, x2, c2, nrhs=2)
        assert torch.equal(a2, c2)
        assert maxrel(host(a2).reshape(-1, 2)[:, 0], host(a)) <= (1e-5 if prec else 1e-13)


@pytest.mark.parametrize("nb", [1, 64, 5000])
def test_uneven_ground_bins(ctx, nb):
    """Most samples in one bin among empty ones: chunk sums of one group only."""
    import oracle as O
    rng = np.random.default_rng(nb)
    n = 40001
    pix = rng.integers(0, 50, n).astype(np.int32)
    psi = rng.uniform(0.0, np.pi, n)
    gb = np.where(rng.random(n) < 0.9, nb // 2, rng.integers(0, nb, n)).astype(np.int32)
    lp = ctx.pointing(dev(pix), dev(psi), 50, 3, 0)
    op = O.pointing_build(pix, psi, 50, 3)
    ist = np.array([0, n], dtype=np.int64)
    sub = np.unique(np.append(np.arange(0, n, 300), n)).astype(np.int64)
    nz = ctx.polyfilter(lp, ist, np.array([1.3]), sub, 1, dev(gb), nb)
    pf = O.polyfilter_build(op, ist, np.array([1.3]), sub, 1, gb, nb)
    y = rng.standard_normal(n)
    assert maxrel(host(ctx.noise_apply(nz, dev(y))), O.polyfilter_apply(pf, y)) <= 1e-12
