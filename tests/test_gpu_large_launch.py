"""Launches at sizes where one thread per element would pass the 2^32 threads a launch
may have.  Outputs are compared on the device; a gather is exact in FP32."""
import pytest

pytestmark = pytest.mark.gpu


def test_P_of_64_columns():
    """2^28 samples x 64 columns, FP32, intensity only (a 64 GiB output)."""
    import torch
    from paper_1801_08937_amd import mapmaker as mm
    if torch.cuda.mem_get_info()[0] < 100 << 30:
        pytest.skip("100 GiB of device memory")
    ctx = mm.Context(0)
    n, side, R = 1 << 28, 64, 64
    g = torch.Generator(device="cuda").manual_seed(3)
    pix = torch.randint(-1, side * side, (n,), generator=g, device="cuda", dtype=torch.int32)
    lp = ctx.pointing(pix, None, side * side, 1, 1, stokes="I")
    assert lp.n_obs == side * side
    x = torch.randn(side * side * R, generator=g, device="cuda", dtype=torch.float64)
    y = torch.empty(n * R, device="cuda", dtype=torch.float32)
    ctx.apply_P(lp, x, y, nrhs=R)
    rows = x.to(torch.float32).reshape(-1, R)
    for t0 in (0, n // 2 - 777, n - 4096):
        j = pix[t0:t0 + 4096].long()
        want = torch.where((j >= 0)[:, None], rows[j.clamp(min=0)], torch.zeros((), device="cuda"))
        assert torch.equal(y[t0 * R:(t0 + 4096) * R].reshape(-1, R), want)
    lp.close()
    ctx.close()


def test_grid_of_2_26_pixels():
    """A map of more than 2^26 pixels, one sample each (a wave per pixel would be a launch
    of 2^32 threads): the grid hint's layouts, P and P^T."""
    import torch
    from paper_1801_08937_amd import mapmaker as mm
    if torch.cuda.mem_get_info()[0] < 40 << 30:
        pytest.skip("40 GiB of device memory")
    ctx = mm.Context(0)
    width, n = 8192, (1 << 26) + 8192
    # the upper half scanned along rows, the lower one along columns: two directions
    rows = torch.arange(n, device="cuda", dtype=torch.int32).reshape(-1, width)
    pix = torch.cat([rows[:4096].reshape(-1), rows[4096:].t().reshape(-1)])
    lp = ctx.pointing(pix, torch.zeros(n, device="cuda", dtype=torch.float64), n, 1, 0)
    assert lp.n_obs == n
    lp.set_grid(width)
    assert lp.p_copies() == 2 and lp.pt_layout()[0] > 0
    y = torch.randn(n, device="cuda", dtype=torch.float64)
    b = ctx.apply_PT(lp, y).reshape(n, 3)
    # psi = 0: weights 1, 1, 0 and one term per sum
    assert torch.equal(b[pix.long(), 0], y) and torch.equal(b[pix.long(), 1], y)
    assert not bool(b[:, 2].any())
    z = ctx.apply_P(lp, b.reshape(-1).contiguous())
    assert torch.equal(z, y + y)
    lp.close()
    ctx.close()
