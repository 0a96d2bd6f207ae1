"""The one-column P at the edges of its launch and of the rule that picks its map:
one sample, odd lengths, one more than a block's samples, and lengths on both
sides of the point from which the map copies are gathered (2^22 samples and 256
per pixel).  Both maps hold the same values, so the outputs are the same bits; the
values are checked against the oracle.  FP64: three products of order one, 1e-14;
FP32: 1e-6 of the largest value."""
import numpy as np
import pytest

import oracle as O
from gpu_util import dev, host, maxrel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1801_08937_amd import mapmaker as mm
    return mm.Context(0)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("stokes", ["IQU", "QU", "I"])
@pytest.mark.parametrize("n", [1, 2, 511, 512, 513, 70001, (1 << 22) - 1, (1 << 22) + 1])
def test_p_one_column(ctx, n, stokes, prec):
    import torch
    side = 32
    rng = np.random.default_rng(n)
    # back-and-forth sweeps with two scan directions and some flagged samples
    t = np.arange(n)
    u = t % side
    a, b = np.where((t // side) % 2 == 0, u, side - 1 - u), (t // side) % side
    pix = np.where((t // (side * side)) % 2 == 0, b * side + a, a * side + b).astype(np.int32)
    pix[rng.random(n) < 0.1] = -1
    if n < 3:
        pix[:] = 5
    psi = rng.uniform(0.0, np.pi, n)
    lp = ctx.pointing(dev(pix), None if stokes == "I" else dev(psi), side * side, 1, prec,
                      stokes=stokes)
    op = O.pointing_build(pix, None if stokes == "I" else psi, side * side, 1, stokes)
    x = rng.standard_normal(op.n)
    y = ctx.apply_P(lp, dev(x))
    assert maxrel(host(y), O.apply_P(op, x)) <= (1e-6 if prec else 1e-14)
    lp.set_grid(side)
    if n > 70000:  # shorter ones: QU and I copies may not fit in a TOD vector, and are left out
        assert lp.p_copies() >= 1
    assert torch.equal(y, ctx.apply_P(lp, dev(x)))
    # an output buffer that starts off a 16-byte boundary
    buf = torch.full((n + 3,), 7.0, dtype=y.dtype, device="cuda")
    ctx.apply_P(lp, dev(x), buf[1:n + 1])
    assert torch.equal(buf[1:n + 1], y) and float(buf[0]) == 7.0 and bool((buf[n + 1:] == 7.0).all())
