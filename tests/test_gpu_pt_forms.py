"""P^T of 8 columns and more in each of its forms (one column per lane, two, and four
waves per pixel): pixels with 1 to 1,300 hits, around the lines between them, in ragged
order with flagged samples.  Against the oracle; sums of at most 1,300 terms of order one:
FP64 1e-12 of the largest, FP32 6e-8 per step of a chain of at most 1,300 / 8: 2e-5."""
import numpy as np
import pytest

import oracle as O
from gpu_util import dev, host, maxrel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1801_08937_amd import mapmaker as mm
    return mm.Context(0)


@pytest.mark.parametrize("stokes,prec", [("IQU", 0), ("IQU", 1), ("QU", 0), ("I", 1)])
@pytest.mark.parametrize("n_pix,hits", [(5, 1), (300, 4), (300, 33), (300, 600), (3, 1300),
                                        (2100, 40), (2100, 3)])
def test_pt_forms(ctx, n_pix, hits, stokes, prec):
    import torch
    rng = np.random.default_rng(n_pix + hits)
    n = n_pix * hits
    pix = rng.permutation(np.arange(n) % n_pix).astype(np.int32)
    pix[rng.random(n) < 0.1] = -1
    pix[:min(n, n_pix)] = np.arange(min(n, n_pix))  # every pixel is hit
    psi = None if stokes == "I" else rng.uniform(0.0, np.pi, n)
    lp = ctx.pointing(dev(pix), None if psi is None else dev(psi), n_pix, 1, prec, stokes=stokes)
    op = O.pointing_build(pix, psi, n_pix, 1, stokes)
    for R in (8, 16, 64):
        z = rng.standard_normal((n, R)).astype(np.float32 if prec else np.float64)
        b = host(ctx.apply_PT(lp, dev(z).reshape(-1), nrhs=R)).reshape(-1, R)
        for r in (0, R // 2 - 1, R - 1):
            ref = O.apply_PT(op, z[:, r].astype(np.float64))
            assert maxrel(b[:, r], ref) <= (2e-5 if prec else 1e-12), (R, r)
