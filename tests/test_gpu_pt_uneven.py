"""One-column P^T of I and QU pointings whose pixels are hit very unequally (one pixel in
64 takes nearly all samples), with and without a grid: the sums, against FP64 sums on the
device (2^24 samples, up to 65,000 of order one per pixel: 1e-12 of the sum of magnitudes;
FP32 sums of 1,000 per lane 1e-5), and the memory that the pointing takes, which is not
that of the longest lane for all 64."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stokes,prec", [("QU", 0), ("QU", 1), ("I", 0), ("I", 1)])
@pytest.mark.parametrize("grid", [0, 128])
def test_uneven_pixels(stokes, prec, grid):
    import torch
    from paper_1801_08937_amd import mapmaker as mm
    n, side = 1 << 24, 128
    g = torch.Generator(device="cuda").manual_seed(3)
    t = torch.arange(n, device="cuda")
    hot = torch.rand(n, generator=g, device="cuda") < 0.97
    pix = torch.where(hot, (t // 40) % 256 * 64 + 17, t % (side * side)).int()
    psi = torch.rand(n, generator=g, device="cuda", dtype=torch.float64) * 3.0
    z = torch.rand(n, generator=g, device="cuda", dtype=torch.float64).add_(0.5)
    z = z.float() if prec else z
    ctx = mm.Context(0)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free = torch.cuda.mem_get_info()[0]
    lp = ctx.pointing(pix, None if stokes == "I" else psi, side * side, 1, prec, stokes=stokes)
    assert lp.n_obs == side * side
    lp.set_grid(grid)
    # at most 60 bytes per sample, and what the library keeps (1.5 GiB)
    assert free - torch.cuda.mem_get_info()[0] <= 60 * n + (3 << 29)
    b = ctx.apply_PT(lp, z).reshape(side * side, -1)
    zero = torch.zeros(side * side, device="cuda", dtype=torch.float64)
    total = zero.index_add(0, pix.long(), z.double())
    ws = [torch.ones_like(psi)] if stokes == "I" else [torch.cos(2 * psi), torch.sin(2 * psi)]
    for a, w in enumerate(ws):
        ref = zero.index_add(0, pix.long(), w * z.double())
        assert bool(((b[:, a] - ref).abs() <= (1e-5 if prec else 1e-12) * total).all())
    lp.close()
    ctx.close()
