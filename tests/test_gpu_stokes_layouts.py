"""The sliced P^T and the map copies of P on I and QU pointings: a cross-linked
scan large enough for both, and small ragged ones (one observed pixel, fewer
samples than eight per thread, low hit counts) that must stay on the general
forms or go through the copies' remainder loop."""
import numpy as np
import pytest

import oracle as O
import synth
from gpu_util import dev, host, maxrel

pytestmark = pytest.mark.gpu

# sums of at most 2^9 terms of order one per pixel in FP64; FP32 rounds each
# of them (6e-8) and their weights
TOL = {0: 1e-12, 1: 2e-5}


@pytest.fixture(scope="module")
def ctx():
    from paper_1801_08937_amd import mapmaker as mm
    return mm.Context(0)


def _handles(ctx, p, stokes, prec, min_hits=3):
    psi = None if stokes == "I" else p.psi
    lp = ctx.pointing(dev(p.pix), None if psi is None else dev(psi), p.n_pix_total, min_hits,
                      prec, stokes=stokes)
    return lp, O.pointing_build(p.pix, psi, p.n_pix_total, min_hits, stokes)


def _check(ctx, lp, op, prec, rng):
    import torch
    dt = torch.float32 if prec else torch.float64
    x, z = rng.standard_normal(op.n), dev(rng.standard_normal(op.n_samp), dt)
    y = ctx.apply_P(lp, dev(x))
    assert maxrel(host(y), O.apply_P(op, x)) <= TOL[prec]
    m = ctx.apply_PT(lp, z)
    assert maxrel(host(m), O.apply_PT(op, host(z).astype(np.float64))) <= TOL[prec]
    assert torch.equal(m, ctx.apply_PT(lp, z))
    return x, y


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("stokes", ["I", "QU"])
def test_sliced_and_copies(ctx, stokes, prec):
    import torch
    p = synth.config2(n_side=128, grid=(4, 4), samp_per_det=1 << 19, L=1 << 15, half_bw=64,
                      noiseless=True)
    lp, op = _handles(ctx, p, stokes, prec)
    rng = np.random.default_rng(3)
    G, S = lp.pt_layout()
    assert G * S >= 2048 and lp.p_copies() == 0
    x, y = _check(ctx, lp, op, prec, rng)
    lp.set_grid(p.n_side)
    assert lp.p_copies() == 3 and lp.pt_layout()[0] == 3 * G
    assert torch.equal(y, ctx.apply_P(lp, dev(x)))  # the copies hold the same values
    _check(ctx, lp, op, prec, rng)
    # the A apply without allocation: the same bits
    ln = ctx.noise(p.interval_start, p.filter_id, p.band, p.half_bw, prec=prec)
    xa = dev(x)
    a, b = ctx.apply_A(lp, ln, xa), torch.empty_like(xa)
    if prec == 1:  # two FP64 TOD vectors of 2^23 samples fill the static scratch
        ctx.apply_A_noalloc(lp, ln, xa, b)
        assert torch.equal(a, b)


@pytest.mark.parametrize("stokes", ["I", "QU"])
@pytest.mark.parametrize("n_samp,n_side,min_hits", [(2048, 4, 3), (4099, 40, 1), (70001, 12, 3)])
def test_small(ctx, stokes, n_samp, n_side, min_hits):
    import torch
    p = synth.random_problem(n_samp, n_side=n_side, n_samp=n_samp, n_int=3, half_bw=5,
                             flag_frac=0.3)
    for prec in (0, 1):
        lp, op = _handles(ctx, p, stokes, prec, min_hits)
        rng = np.random.default_rng(4)
        x, y = _check(ctx, lp, op, prec, rng)
        lp.set_grid(p.n_side)
        assert torch.equal(y, ctx.apply_P(lp, dev(x)))
        _check(ctx, lp, op, prec, rng)
        ln = ctx.noise(p.interval_start, p.filter_id, p.band, p.half_bw, prec=prec)
        xa = dev(x)
        b = torch.empty_like(xa)
        ctx.apply_A_noalloc(lp, ln, xa, b)
        assert torch.equal(ctx.apply_A(lp, ln, xa), b)
