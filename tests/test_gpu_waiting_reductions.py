"""Grid-wide steps whose small reductions wait for the pass that uses them
against the same steps with a finalize launch after every pass (as profiling
runs them): every variant and pass fusion, lengths below one tile, cut tiles,
several workgroups, and either side of the longest vector that waits.  The two
sum the same partials in another order; over these iterations the windows'
condition numbers stay below 1e3, so 1e-11 holds a hundred such roundings."""
import numpy as np
import pytest

import aa_workloads as W
from gpu_util import device, rel, to_dev

pytestmark = pytest.mark.gpu
RHS, T_TRANSFORM, DELETE = 1 << 3, 1 << 2, 1 << 5


@pytest.mark.parametrize("variant,flags", [
    ("mgs", 0), ("cgs2", 0), ("cgs2", RHS | DELETE), ("dcgs2", 0), ("dcgs2", RHS),
    ("icwy", 0), ("icwy", DELETE), ("icwy", RHS | DELETE), ("icwy", T_TRANSFORM),
    ("dcgs2_lag", RHS)])
@pytest.mark.parametrize("s,m", [(60, 1), (60, 5), (1025, 3), (70_001, 10), ((1 << 19), 4),
                                 ((1 << 19) + 1, 4)])
def test_waiting_and_finalized_steps_agree(s, m, variant, flags):
    import torch
    device()
    from paper_2110_09667_amd import aa
    prob = W.StencilProblem(d=1, s=s, c=1.0, f=W.uniform(s, 0, s))
    f = to_dev(prob.f)
    got = []
    for finalized in (False, True):
        ctx = aa.AAContext(s, m, variant, flags)
        ctx.set_fused_threshold(0)
        ctx.profile(finalized)
        x = torch.zeros(s, dtype=torch.float64, device="cuda")
        g = torch.empty_like(x)
        for _ in range(m + 5):
            aa.aa_problem_apply(1, s, prob.h, prob.omega, prob.c, f, x, g)
            ctx.step(x, g, x)
        info = ctx.info()
        assert info.status == 0 and info.k == m
        Q = ctx.basis(m).cpu().numpy()
        R, _, _ = ctx.get_qr()
        assert np.all(np.tril(R, -1) == 0.0)
        assert np.linalg.norm(np.eye(m) - Q.T @ Q) <= 1e-9
        got.append((x.cpu().numpy(), info.res_norm, info.step_norm, ctx.sync_counts()))
        ctx.close()
    (x0, r0, d0, c0), (x1, r1, d1, c1) = got
    assert rel(x0, x1) <= 1e-11 and c0 == c1
    assert abs(r0 / r1 - 1) <= 1e-9 and abs(d0 / d1 - 1) <= 1e-9
