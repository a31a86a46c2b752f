"""Per-kind timing of steps whose unprofiled form merges kernels: every kind of
the iteration is recorded as a launch of its own, and the steps compute what
unprofiled ones do (the sums of short vectors in another order: 1e-11 as for the
comparison of the two forms)."""
import numpy as np
import pytest

import aa_workloads as W
from gpu_util import device, rel, to_dev

pytestmark = pytest.mark.gpu
RHS, T_TRANSFORM, DELETE = 1 << 3, 1 << 2, 1 << 5


@pytest.mark.parametrize("variant,flags", [("mgs", 0), ("cgs2", 0), ("dcgs2", RHS | DELETE),
                                           ("icwy", 0), ("icwy", T_TRANSFORM),
                                           ("icwy", RHS | DELETE), ("dcgs2_lag", 0)])
@pytest.mark.parametrize("s", [30_000, (1 << 19) + 3])
def test_every_kind_of_a_step_is_recorded(s, variant, flags):
    import torch
    device()
    from paper_2110_09667_amd import aa
    m, recycled = 5, 4
    prob = W.StencilProblem(d=1, s=s, c=1.0, f=W.uniform(s, 0, s))
    f = to_dev(prob.f)
    got = []
    for profiled in (True, False):
        ctx = aa.AAContext(s, m, variant, flags)
        ctx.set_fused_threshold(0)
        ctx.profile(profiled)
        x = torch.zeros(s, dtype=torch.float64, device="cuda")
        g = torch.empty_like(x)
        for _ in range(m + 1 + recycled):
            aa.aa_problem_apply(1, s, prob.h, prob.omega, prob.c, f, x, g)
            ctx.step(x, g, x)
        if profiled:
            kinds = {k: v[1] for k, v in ctx.profile_read().items()}
        assert ctx.info().status == 0
        got.append(x.cpu().numpy())
        ctx.close()
    assert kinds["givens"] == kinds["rotate"] == recycled
    assert kinds["history"] == m + 1 + recycled and kinds["xupdate"] == m + recycled
    # (the lagged variant divides in its update pass, but for the first column)
    assert kinds["scale"] == (1 if variant == "dcgs2_lag" else m + recycled)
    assert kinds["finalize"] >= 3 * (m + recycled)
    assert rel(got[0], got[1]) <= (1e-11 if s <= 1 << 19 else 0.0)
