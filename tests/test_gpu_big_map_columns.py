"""P of 32 and 64 columns with a map beyond the L2s, whose waves take longer runs of
samples: ragged lengths, flagged samples; every value is one gather and three products, so
FP64 within 1e-14 of the largest and FP32 within 1e-6, against the same on the device."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("R,n", [(64, (1 << 19) + 13), (32, (1 << 20) + 77), (32, (1 << 20) - 1)])
def test_big_map(R, n, prec):
    import torch
    from paper_1801_08937_amd import mapmaker as mm
    ctx = mm.Context(0)
    n_pix = 40000  # x: 31 and 61 MB
    g = torch.Generator(device="cuda").manual_seed(R)
    pix = (torch.arange(n, device="cuda") * 7 % n_pix).int()
    pix[torch.rand(n, generator=g, device="cuda") < 0.1] = -1
    psi = torch.rand(n, generator=g, device="cuda", dtype=torch.float64) * 3.0
    lp = ctx.pointing(pix, psi, n_pix, 1, prec)
    assert lp.n_obs == n_pix
    x = torch.randn(lp.n * R, generator=g, device="cuda", dtype=torch.float64)
    y = torch.full((n * R + R,), 7.0, device="cuda", dtype=torch.float32 if prec else torch.float64)
    ctx.apply_P(lp, x, y[:n * R], nrhs=R)
    assert bool((y[n * R:] == 7.0).all())
    m, j = x.reshape(n_pix, 3, R), pix.long().clamp(min=0)
    c, s = torch.cos(2 * psi)[:, None], torch.sin(2 * psi)[:, None]
    want = (m[j, 0] + c * m[j, 1] + s * m[j, 2]) * (pix >= 0)[:, None]
    err = float((y[:n * R].reshape(n, R).double() - want).abs().max()) / float(want.abs().max())
    assert err <= (1e-6 if prec else 1e-14)
    lp.close()
    ctx.close()
