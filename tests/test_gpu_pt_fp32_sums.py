"""FP32 P^T of I and QU pointings by time segments: its sums are no further from 64-bit
ones than the weights' own rounding.  I: FP32 samples summed in FP64, so a few rounding
steps of 2^-53 of the sum of magnitudes (512 terms of one to two): 1e-12 of the largest.
QU: weights rounded to FP32 once, at most 2^-25 of each sample's magnitude, 1.001 of it
with the sum's own rounding.  FP32 sums are further off than the first by 1e5."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid", [0, 128])
@pytest.mark.parametrize("stokes", ["I", "QU"])
def test_sums_in_64_bits(stokes, grid):
    import torch
    from paper_1801_08937_amd import mapmaker as mm
    ctx = mm.Context(0)
    n, side = 1 << 23, 128
    g = torch.Generator(device="cuda").manual_seed(11)
    # runs along rows, so that a grid finds one scan direction
    t = torch.arange(n, device="cuda")
    start = torch.randint(0, side * side, (n // 4096 + 1,), generator=g, device="cuda")
    pix = ((start[t // 4096] + t) % (side * side)).int()
    psi = torch.rand(n, generator=g, device="cuda", dtype=torch.float64) * 3.0
    lp = ctx.pointing(pix, None if stokes == "I" else psi, side * side, 1, 1, stokes=stokes)
    assert lp.n_obs == side * side
    lp.set_grid(grid)
    assert lp.pt_layout()[0] > 0
    z = torch.rand(n, generator=g, device="cuda", dtype=torch.float64).add_(1.0).float()
    b = ctx.apply_PT(lp, z).reshape(side * side, -1)
    zero = torch.zeros(side * side, device="cuda", dtype=torch.float64)
    total = zero.index_add(0, pix.long(), z.double())
    if stokes == "I":
        assert float((b[:, 0] - total).abs().max()) <= 1e-12 * float(total.max())
    else:
        for a, w in ((0, torch.cos(2 * psi)), (1, torch.sin(2 * psi))):
            ref = zero.index_add(0, pix.long(), w * z.double())
            assert bool(((b[:, a] - ref).abs() <= 1.001 * 2.0 ** -25 * total).all())
    lp.close()
    ctx.close()
