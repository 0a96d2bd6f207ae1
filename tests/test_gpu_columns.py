"""P and P^T of several columns at the edges of their launches: a wave's run of samples
(256 / R) and one more or less, one sample, pixels with no, one and many samples, few
and many pixels (a block or a wave per pixel), all three Stokes layouts.  FP64: sums
of at most some thousand products of order one, 1e-12 of the largest; FP32: 1e-5."""
import numpy as np
import pytest

import oracle as O
from gpu_util import dev, host, maxrel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1801_08937_amd import mapmaker as mm
    return mm.Context(0)


@pytest.mark.parametrize("stokes", ["IQU", "QU", "I"])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("R", [2, 4, 8, 16, 32, 64])
def test_columns(ctx, R, prec, stokes):
    import torch
    run = 256 // R
    for n, side in [(1, 1), (run - 1, 2), (run, 3), (run + 1, 3), (4 * run + 1, 4), (3001, 9),
                    (20000, 72)]:
        if n < 1:
            continue
        rng = np.random.default_rng(100 * R + n)
        pix = np.sort(rng.integers(0, side * side, n)).astype(np.int32)
        pix[rng.random(n) < 0.3] = 0  # one pixel with many samples
        if n > 2:
            pix[rng.random(n) < 0.1] = -1
        if not (pix >= 0).any():
            pix[0] = 0
        psi = None if stokes == "I" else rng.uniform(0.0, np.pi, n)
        lp = ctx.pointing(dev(pix), None if psi is None else dev(psi), side * side, 1, prec,
                          stokes=stokes)
        op = O.pointing_build(pix, psi, side * side, 1, stokes)
        x, z = rng.standard_normal((op.n, R)), rng.standard_normal((n, R))
        tt = torch.float32 if prec else torch.float64
        # x and the outputs start 8 (FP32: 4) bytes off a 16-byte boundary
        bx = torch.zeros(op.n * R + 1, dtype=torch.float64, device="cuda")
        bx[1:] = dev(x).reshape(-1)
        by = torch.full((n * R + 2,), 7.0, dtype=tt, device="cuda")
        ctx.apply_P(lp, bx[1:], by[1:n * R + 1], nrhs=R)
        tol = 1e-5 if prec else 1e-12
        y = host(by[1:n * R + 1]).reshape(n, R)
        assert float(by[0]) == 7.0 and float(by[n * R + 1]) == 7.0
        zt = dev(z, tt).reshape(-1)
        bz = torch.full((op.n * R + 2,), 7.0, dtype=torch.float64, device="cuda")
        ctx.apply_PT(lp, zt, bz[1:op.n * R + 1], nrhs=R)
        assert float(bz[0]) == 7.0 and float(bz[op.n * R + 1]) == 7.0
        m = host(bz[1:op.n * R + 1]).reshape(op.n, R)
        for r in {0, 1, R // 2, R - 1}:
            assert maxrel(y[:, r], O.apply_P(op, x[:, r].copy())) <= tol
            assert maxrel(m[:, r], O.apply_PT(op, z[:, r].copy())) <= tol


@pytest.mark.parametrize("stokes", ["IQU", "I"])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("R", [2, 4, 8, 16, 32])
def test_A_keeps_the_columns(ctx, R, prec, stokes):
    """A's own TOD may hold its columns one after the other; the values are those of P,
    N^-1 and P^T one by one, bit for bit."""
    import torch
    rng = np.random.default_rng(R)
    lens = [9001, 70, 8191, 12000]
    n, lam, side = sum(lens), 33, 11
    pix = rng.integers(-1, side * side, n).astype(np.int32)
    psi = None if stokes == "I" else dev(rng.uniform(0.0, np.pi, n))
    lp = ctx.pointing(dev(pix), psi, side * side, 1, prec, stokes=stokes)
    istart = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    band = rng.standard_normal((2, lam + 1))
    nz = ctx.noise(istart, np.array([0, 1, 1, 0], dtype=np.int32), band, lam, method=2, prec=prec)
    x = dev(rng.standard_normal(lp.n * R))
    parts = ctx.apply_PT(lp, ctx.noise_apply(nz, ctx.apply_P(lp, x, nrhs=R), nrhs=R), nrhs=R)
    assert torch.equal(ctx.apply_A(lp, nz, x, nrhs=R), parts)


@pytest.mark.parametrize("stokes", ["IQU", "QU", "I"])
@pytest.mark.parametrize("prec,R,lam", [(0, 64, 8), (0, 64, 32), (0, 64, 92), (0, 64, 93),
                                        (0, 32, 33), (0, 16, 60), (0, 8, 12), (0, 8, 150),
                                        (1, 64, 32), (1, 32, 100), (1, 16, 9), (1, 8, 40)])
def test_A_band_in_one_pass(ctx, prec, R, lam, stokes):
    """Direct band of many columns: A gathers P x inside N^-1 (FP64, 64 columns: up to
    lambda 92), with the bits of P, N^-1 and P^T one by one."""
    import torch
    rng = np.random.default_rng(R + lam)
    lens = [2 * lam + 1, 2 * lam + 2, 1000, 64 * 40, 64 * 40 + 1, 127 * 16, (1 << 21) // min(R, 32)]
    n, side = sum(lens), 13
    pix = rng.integers(-1, side * side, n).astype(np.int32)
    psi = None if stokes == "I" else dev(rng.uniform(0.0, np.pi, n))
    lp = ctx.pointing(dev(pix), psi, side * side, 1, prec, stokes=stokes)
    istart = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    fid = rng.integers(0, 3, len(lens)).astype(np.int32)
    nz = ctx.noise(istart, fid, rng.standard_normal((3, lam + 1)), lam, method=1, prec=prec)
    x = dev(rng.standard_normal(lp.n * R))
    parts = ctx.apply_PT(lp, ctx.noise_apply(nz, ctx.apply_P(lp, x, nrhs=R), nrhs=R), nrhs=R)
    assert torch.equal(ctx.apply_A(lp, nz, x, nrhs=R), parts)


@pytest.mark.parametrize("stokes", ["IQU", "QU", "I"])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("big,lam", [(False, 0), (False, 1), (False, 32), (False, 300),
                                     (False, 1023), (False, 1024), (True, 7), (True, 64),
                                     (True, 1700)])
def test_A_band_one_column(ctx, big, lam, prec, stokes):
    """One column: P x gathered as the band's window is staged, on short streams (tiles of
    512) and long ones (2,048; and from map copies); the bits of the three launches."""
    import torch
    rng = np.random.default_rng(lam)
    lens = [2 * lam + 1, 2 * lam + 2, 511 + 2 * lam, 512 + 2 * lam, 513 + 2 * lam, 5000]
    if big:
        lens += [2047 + 2 * lam, 2049 + 2 * lam, (1 << 22) + 3]
    n, side = sum(lens), 13
    u, v = np.arange(n) % side, np.arange(n) // side % side  # back and forth
    pix = (v * side + np.where(np.arange(n) // side % 2 == 0, u, side - 1 - u)).astype(np.int32)
    pix[rng.random(n) < 0.05] = -1
    psi = None if stokes == "I" else dev(rng.uniform(0.0, np.pi, n))
    lp = ctx.pointing(dev(pix), psi, side * side, 1, prec, stokes=stokes)
    istart = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    fid = rng.integers(0, 3, len(lens)).astype(np.int32)
    nz = ctx.noise(istart, fid, rng.standard_normal((3, lam + 1)), lam, method=1, prec=prec)
    x = dev(rng.standard_normal(lp.n))
    for width in (0, side):
        lp.set_grid(width)
        parts = ctx.apply_PT(lp, ctx.noise_apply(nz, ctx.apply_P(lp, x)))
        assert torch.equal(ctx.apply_A(lp, nz, x), parts)


@pytest.mark.parametrize("stokes", ["IQU", "QU", "I"])
@pytest.mark.parametrize("R", [1, 2, 16, 64])
@pytest.mark.parametrize("side", [3, 40])
def test_pcg_mbd_columns(ctx, R, side, stokes):
    """PCG with M_BD (x, r and z = M r in one pass over the pixels): the iterates after
    six steps, and a column that starts converged stays as it is.  Six steps of a
    well-conditioned system amplify rounding by less than 1e4: 1e-10."""
    rng = np.random.default_rng(R + side)
    n = side * side * 40
    pix = rng.permutation(np.arange(n) % (side * side)).astype(np.int32)
    psi = None if stokes == "I" else rng.uniform(0.0, np.pi, n)
    lp = ctx.pointing(dev(pix), None if psi is None else dev(psi), side * side, 3, 0,
                      stokes=stokes)
    op = O.pointing_build(pix, psi, side * side, 3, stokes)
    istart, fid = np.array([0, n // 2, n], dtype=np.int64), np.array([0, 1], dtype=np.int32)
    band = np.array([[1.0, -0.3, 0.1], [1.5, 0.3, -0.1]])
    ln, on = ctx.noise(istart, fid, band, 2), O.noise_build(istart, fid, band, 2)
    M, OM = ctx.mbd(lp, ln), O.mbd_build(op, on)
    b = rng.standard_normal((op.n, R))
    x0 = np.zeros((op.n, R))
    if R > 1:  # this column's first residual is 0
        x0[:, 1] = rng.standard_normal(op.n)
        b[:, 1] = host(ctx.apply_A(lp, ln, dev(x0[:, 1].copy())))
    x, info = ctx.solve(lp, ln, M, dev(b).reshape(-1), dev(x0).reshape(-1), tol=1e-13, max_iter=6,
                        nrhs=R)
    x = host(x).reshape(op.n, R)
    for r in {0, R // 2, R - 1}:
        if r == 1:
            continue
        xo, io = O.pcg(lambda v: O.apply_A(op, on, v), lambda v: O.mbd_apply(OM, v),
                       b[:, r].copy(), 0.0, 6)
        assert maxrel(x[:, r], xo) <= 1e-10
    if R > 1:
        assert maxrel(x[:, 1], x0[:, 1]) <= 1e-10
