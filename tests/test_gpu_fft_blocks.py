"""N^-1 by FFT at the edges of its overlap-save blocks: intervals shorter than
a block, of exactly one or two blocks' valid outputs and one sample more or
less, odd bandwidths, both block sizes, one and several columns.  The band is
random, so every frequency of the spectrum (0 and Nyquist among them) counts.

FP64 tolerance: a transform pair of 2^15 points loses about 30 rounding steps
(3e-15 of the largest output, as the band's symbol and the inputs are of order
one per frequency); 1e-12 leaves two orders.  FP32: the same with 6e-8 steps,
2e-6, times ten."""
import numpy as np
import pytest

import oracle as O
from gpu_util import dev, host, maxrel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1801_08937_amd import mapmaker as mm
    return mm.Context(0)


@pytest.mark.parametrize("n_fft", [16384, 32768])
@pytest.mark.parametrize("lam", [31, 32, 1000, 4095])
@pytest.mark.parametrize("prec,R", [(0, 1), (0, 2), (1, 1), (1, 4)])
def test_fft_block_edges(ctx, n_fft, lam, prec, R):
    import torch
    rng = np.random.default_rng(1000 * lam + n_fft + 10 * prec + R)
    V = n_fft - 2 * lam
    lens = [2 * lam + 1, V - 1, V, V + 1, 2 * V, 2 * lam + 2]
    istart = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    fid = np.array([0, 1, 0, 1, 1, 0], dtype=np.int32)
    band = rng.standard_normal((2, lam + 1)) / np.sqrt(2 * lam + 1)
    nz = ctx.noise(istart, fid, band, lam, method=2, prec=prec)
    nz.set_fft_block(n_fft)
    assert nz.fft_n == n_fft
    y = rng.standard_normal((istart[-1], R)) + 1.0
    t = dev(y, torch.float32 if prec else torch.float64)
    z = host(ctx.noise_apply(nz, t.reshape(-1), nrhs=R)).reshape(-1, R)
    on = O.noise_build(istart, fid, band, lam)
    tol = 2e-5 if prec else 1e-12
    for r in range(R):
        ref = O.noise_apply_fft(on, host(t)[:, r].astype(np.float64))
        assert maxrel(z[:, r], ref) <= tol, (r, maxrel(z[:, r], ref))


@pytest.mark.parametrize("lam", [1, 31, 32, 1000, 2047, 3072])
@pytest.mark.parametrize("prec,R", [(0, 1), (0, 2), (1, 1), (1, 4)])
def test_fft_short_stream(ctx, lam, prec, R):
    """A short stream on its own choice of blocks (8,192 samples, or 16,384 where those
    would be too many): intervals about one and two of their valid stretches."""
    import torch
    rng = np.random.default_rng(77 * lam + 10 * prec + R)
    V = 8192 - 2 * lam
    lens = [max(v, 2 * lam + 1) for v in (0, V - 1, V, V + 1, 2 * V, 2 * lam + 2)]
    istart = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    fid = np.array([0, 1, 0, 1, 1, 0], dtype=np.int32)
    band = rng.standard_normal((2, lam + 1)) / np.sqrt(2 * lam + 1)
    nz = ctx.noise(istart, fid, band, lam, method=2, prec=prec)
    assert nz.fft_n == 16384 and nz.fft_valid == 16384 - 2 * lam
    y = rng.standard_normal((istart[-1], R)) + 1.0
    t = dev(y, torch.float32 if prec else torch.float64)
    z = host(ctx.noise_apply(nz, t.reshape(-1), nrhs=R)).reshape(-1, R)
    on = O.noise_build(istart, fid, band, lam)
    tol = 2e-5 if prec else 1e-12
    for r in range(R):
        ref = O.noise_apply_fft(on, host(t)[:, r].astype(np.float64))
        assert maxrel(z[:, r], ref) <= tol, (r, maxrel(z[:, r], ref))
        one = host(ctx.noise_apply(nz, t[:, r].contiguous()))
        np.testing.assert_array_equal(one, z[:, r])


@pytest.mark.parametrize("n_fft", [16384, 32768])
@pytest.mark.parametrize("lam", [33, 1000])
@pytest.mark.parametrize("prec,R", [(0, 1), (0, 4), (1, 1), (1, 2)])
def test_fft_masked_rhs(ctx, n_fft, lam, prec, R):
    """b = P^T N^-1 (mask . d) with the mask applied as the FFT reads d:
    non-finite values on flagged samples (and on pixels below the hit
    threshold) are ignored, one on a kept sample is an error that leaves b
    untouched."""
    import torch
    from paper_1801_08937_amd import mapmaker as mm
    rng = np.random.default_rng(lam + n_fft + R)
    V = n_fft - 2 * lam
    istart = np.concatenate([[0], np.cumsum([2 * lam + 1, V + 1, 2 * lam + 7, V])]).astype(np.int64)
    n = int(istart[-1])
    pix = rng.integers(-1, 30, n).astype(np.int32)
    pix[17] = 31  # a single hit: dropped
    psi = rng.uniform(0, np.pi, n)
    band = rng.standard_normal((2, lam + 1)) / np.sqrt(2 * lam + 1)
    fid = np.array([0, 1, 1, 0], dtype=np.int32)
    lp = ctx.pointing(dev(pix), dev(psi), 32, 3, prec)
    nz = ctx.noise(istart, fid, band, lam, method=2, prec=prec)
    nz.set_fft_block(n_fft)
    op, on = O.pointing_build(pix, psi, 32, 3), O.noise_build(istart, fid, band, lam)
    d = rng.standard_normal((R, n)).astype(np.float32 if prec else np.float64)
    off = op.j < 0
    dn = d.copy()
    dn[:, off] = np.nan
    dn[0, 17] = np.inf
    b = host(ctx.rhs(lp, nz, dev(dn).reshape(-1), nrhs=R)).reshape(-1, R)
    tol = 2e-5 if prec else 1e-12
    for r in range(R):
        ref = O.rhs(op, on, np.where(off, 0.0, d[r].astype(np.float64)), "fft")
        assert maxrel(b[:, r], ref) <= tol, (r, maxrel(b[:, r], ref))
    for t in (int(np.flatnonzero(~off)[0]), int(np.flatnonzero(~off)[-1])):
        dn2 = d.copy()
        dn2[R - 1, t] = np.nan
        out = torch.full((op.n * R,), 7.0, dtype=torch.float64, device="cuda")
        with pytest.raises(mm.MapmakerError, match="NONFINITE"):
            ctx.rhs(lp, nz, dev(dn2).reshape(-1), out, nrhs=R)
        assert bool((out == 7.0).all())


def test_fft_many_filters(ctx):
    """More filters than the 256 whose spectra are formed at a time, one per interval."""
    rng = np.random.default_rng(4)
    lam, ni = 40, 521
    lens = rng.integers(2 * lam + 1, 200, ni)
    istart = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    band = rng.standard_normal((ni, lam + 1)) / np.sqrt(2 * lam + 1)
    fid = rng.permutation(ni).astype(np.int32)
    nz = ctx.noise(istart, fid, band, lam, method=2, prec=0)
    y = rng.standard_normal(istart[-1])
    ref = O.noise_apply_direct(O.noise_build(istart, fid, band, lam), y)
    assert maxrel(host(ctx.noise_apply(nz, dev(y))), ref) <= 1e-12
