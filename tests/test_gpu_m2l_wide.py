"""M_2l on one column around the 32 pixels per block where it goes from several threads
per pixel to one: IQU maps of 8,190 to 8,281 pixels, and of 65,600, with subspaces around
the eight columns a thread takes at a time.  Against the oracle, with Z orthonormal (sums
of at most 64 terms of order one times the conditioning of E: 1e-9), and, with the partial
sums of r.z that a solve asks for, a few iterations of PCG against those of two columns
(the same steps in other kernels: 1e-9 of the solution)."""
import numpy as np
import pytest

import oracle as O
from gpu_util import dev, host, maxrel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1801_08937_amd import mapmaker as mm
    return mm.Context(0)


@pytest.mark.parametrize("n_pix,ks", [(8190, (1, 33)), (8193, (8, 64)), (8281, (7, 9)),
                                      (65600, (32,))])
def test_m2l_one_column_wide(ctx, n_pix, ks):
    rng = np.random.default_rng(n_pix)
    n = n_pix * 12
    pix = rng.permutation(np.arange(n) % n_pix).astype(np.int32)
    psi = rng.uniform(0.0, np.pi, n)
    lp = ctx.pointing(dev(pix), dev(psi), n_pix, 3, 0)
    op = O.pointing_build(pix, psi, n_pix, 3)
    istart, fid = np.array([0, n // 2, n], dtype=np.int64), np.array([0, 1], dtype=np.int32)
    band = np.array([[1.0, -0.2, 0.05], [1.2, 0.1, 0.0]])
    ln, on = ctx.noise(istart, fid, band, 2), O.noise_build(istart, fid, band, 2)
    M, OM = ctx.mbd(lp, ln), O.mbd_build(op, on)
    for k in ks:
        Z = np.linalg.qr(rng.standard_normal((op.n, k)))[0]
        M2 = ctx.defl_from_Z(lp, ln, M, dev(np.ascontiguousarray(Z)))
        v = rng.standard_normal(op.n)
        one = host(ctx.precond_apply(M2, dev(v)))
        assert maxrel(one, O.m2l_apply(O.m2l_from_Z(op, on, OM, Z), v)) <= 1e-9
        x1 = host(ctx.solve(lp, ln, M2, dev(v), tol=0.0, max_iter=4)[0])
        x2 = host(ctx.solve(lp, ln, M2, dev(np.stack([v, -v], axis=1).reshape(-1)), tol=0.0,
                            max_iter=4, nrhs=2)[0]).reshape(-1, 2)[:, 0]
        assert maxrel(x1, x2) <= 1e-9
