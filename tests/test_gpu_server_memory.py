"""The serving engine's byte budget against what it allocates."""
import pytest

import synth
from gpu_util import dev

pytestmark = pytest.mark.gpu

SHAPES = [(32, (4, 2), 1 << 15, 128), (64, (4, 4), 1 << 17, 256)]


def _server(ids, slots=4, budget=8 << 30):
    import torch
    from paper_1801_08937_amd import mapmaker as mm
    assert torch.cuda.is_available()
    srv = mm.Server(0, hbm_budget_bytes=budget, slots=slots, defl_k=0, iters_per_step=3)
    ps = [synth.serve_strategy(s, 0, shapes=SHAPES[s], L=1 << 13) for s in ids]
    for s, p in zip(ids, ps):
        srv.add_strategy(s, dev(p.pix), dev(p.psi), p.n_pix_total, p.interval_start, p.filter_id,
                         p.band, p.half_bw, grid_width=p.n_side)
    return srv, ps


@pytest.mark.parametrize("slots", [1, 8])
def test_session_charge(slots):
    """A session is charged its vectors (x, r, z, p, q and one column), three sets of
    512 partial sums per column (p.q, ||r||^2, r.z), the TOD workspaces, and 64 partial
    maps of P^T."""
    from paper_1801_08937_amd import mapmaker as mm
    srv, (p,) = _server([0], slots)
    ctx = mm.Context(0)
    n = ctx.pointing(dev(p.pix), dev(p.psi), p.n_pix_total, 3, 0).n
    assert srv.memory(0)["session"] == (8 * n * (5 * slots + 1) + 3 * 8 * 512 * slots
                                        + 2 * 8 * p.pix.size * slots + 8 * n * 64)
    srv.close()


def test_registration_leaves_no_more_than_charged():
    """Registering a strategy while another context lives: the memory that its builds
    release goes back to the device, so what is taken is what is charged (64 MiB for
    the runtime's own and for rounding to blocks)."""
    import torch
    from paper_1801_08937_amd import mapmaker as mm
    other = mm.Context(0)
    torch.cuda.synchronize()
    warm, _ = _server([0])  # kernels and libraries are loaded
    warm.close()
    p = synth.serve_strategy(1, 0, shapes=SHAPES[1], L=1 << 13)
    pix, psi = dev(p.pix), dev(p.psi)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    srv = mm.Server(0, hbm_budget_bytes=8 << 30, slots=4, defl_k=0, iters_per_step=3)
    srv.add_strategy(0, pix, psi, p.n_pix_total, p.interval_start, p.filter_id, p.band,
                     p.half_bw, grid_width=p.n_side)
    taken = free - torch.cuda.mem_get_info()[0]
    print("taken", taken, "charged", srv.memory()["used"])
    assert taken <= srv.memory()["used"] + (64 << 20)
    srv.close()
    torch.cuda.synchronize()
    assert free - torch.cuda.mem_get_info()[0] <= 64 << 20
    other.close()
