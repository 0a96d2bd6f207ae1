"""Columns of a direct band where N^-1 alone takes tiles in LDS (8 in FP64 with half
bandwidths below 32 on long streams, 32 in FP32 with longer ones on short streams) and A
forms P inside the band by rows, each with its own tile table: A is bit by bit P^T of N^-1 of P, with intervals about both tile lengths (256 and
512 samples), and N^-1 equals that of two columns."""
import numpy as np
import pytest

from gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("lam,R,long", [(8, 8, 1 << 21), (31, 8, 1 << 21), (32, 8, 1 << 21),
                                        (31, 32, 1 << 16), (32, 32, 1 << 16), (90, 32, 1 << 16),
                                        (40, 16, 1 << 17)])
def test_own_tile_tables(lam, R, long, prec):
    import torch
    from paper_1801_08937_amd import mapmaker as mm
    ctx = mm.Context(0)
    rng = np.random.default_rng(lam)
    lens = [255, 256, 257, 511, 512, 513, 2 * lam + 1, long + 77, 1023]
    istart = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    fid = (np.arange(len(lens)) % 2).astype(np.int32)
    n, n_pix = int(istart[-1]), 900
    nz = ctx.noise(istart, fid, rng.standard_normal((2, lam + 1)), lam, method=1, prec=prec)
    pix = (np.arange(n) * 11 // 7 % n_pix).astype(np.int32)
    pix[rng.random(n) < 0.05] = -1
    lp = ctx.pointing(dev(pix), dev(rng.uniform(0, np.pi, n)), n_pix, 1, prec)
    x = dev(rng.standard_normal(lp.n * R))
    y = ctx.apply_P(lp, x, nrhs=R)
    z = ctx.noise_apply(nz, y, nrhs=R)
    assert torch.equal(ctx.apply_A(lp, nz, x, nrhs=R), ctx.apply_PT(lp, z, nrhs=R))
    two = y.reshape(n, R)[:, 2:4].contiguous()
    assert torch.equal(z.reshape(n, R)[:, 2:4],
                       ctx.noise_apply(nz, two.reshape(-1), nrhs=2).reshape(n, 2))
    lp.close()
    nz.close()
    ctx.close()
