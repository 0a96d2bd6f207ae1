"""Limits of mm_solve's history."""
import numpy as np
import pytest

import synth
from gpu_util import build_both, dev

pytestmark = pytest.mark.gpu


def test_history_of_2_31_iterations_is_refused():
    """max_iter + 1 does not fit in 32 bits: out of memory, as any history too large, and
    the context works on."""
    import torch
    from paper_1801_08937_amd import mapmaker as mm
    ctx = mm.Context(0)
    lp, ln, op, on = build_both(ctx, synth.config1())
    M = ctx.mbd(lp, ln)
    b = dev(np.random.default_rng(0).standard_normal(op.n))
    x = torch.zeros_like(b)
    with pytest.raises(mm.MapmakerError, match="OOM"):
        ctx.solve(lp, ln, M, b, x, max_iter=2 ** 31 - 1, history=False)
    x, info = ctx.solve(lp, ln, M, b, x, tol=1e-6, max_iter=200)
    assert info["converged"]
    ctx.close()
