"""M_2l on one column (its own kernel) at the edges of its launch: subspaces of 1 to 64
columns, around the 16 and 32 that a wave and a block take at a time, maps of fewer
pixels than a block's 32 and of many blocks, three Stokes layouts.  Against the oracle,
with Z orthonormal; sums of at most 64 terms of order one times the conditioning of E:
1e-9; and against the same vector among two columns."""
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
@pytest.mark.parametrize("side", [5, 33])
@pytest.mark.parametrize("k", [1, 3, 16, 17, 32, 33, 64])
def test_m2l_one_column(ctx, k, side, stokes):
    rng = np.random.default_rng(k + side)
    n = side * side * 24
    pix = rng.permutation(np.arange(n) % (side * side)).astype(np.int32)
    psi = None if stokes == "I" else rng.uniform(0.0, np.pi, n)
    lp = ctx.pointing(dev(pix), None if psi is None else dev(psi), side * side, 3, 0,
                      stokes=stokes)
    op = O.pointing_build(pix, psi, side * side, 3, stokes)
    if k > op.n:
        pytest.skip("more columns than unknowns")
    istart, fid = np.array([0, n // 2, n], dtype=np.int64), np.array([0, 1], dtype=np.int32)
    band = np.array([[1.0, -0.2, 0.05], [1.2, 0.1, 0.0]])
    ln, on = ctx.noise(istart, fid, band, 2), O.noise_build(istart, fid, band, 2)
    M = ctx.mbd(lp, ln)
    Z = np.linalg.qr(rng.standard_normal((op.n, k)))[0]
    M2 = ctx.defl_from_Z(lp, ln, M, dev(np.ascontiguousarray(Z)))
    OM2 = O.m2l_from_Z(op, on, O.mbd_build(op, on), Z)
    v = rng.standard_normal(op.n)
    one = host(ctx.precond_apply(M2, dev(v)))
    assert maxrel(one, O.m2l_apply(OM2, v)) <= 1e-9
    two = host(ctx.precond_apply(M2, dev(np.stack([v, -v], axis=1)).reshape(-1), nrhs=2))
    assert maxrel(two.reshape(-1, 2)[:, 0], one) <= 1e-12
