"""The end of a multigrid-preconditioned solve at its tolerance: the launches
enqueued past it change nothing, so the solution is bit for bit that of the
same solve with its iteration count fixed, for solves whose test runs in the
one-workgroup kernel of the coarse levels (N = 100) and in a tiled level kernel
of many workgroups (both tile shapes), first solves (too few launches enqueued
at once) and repeated ones."""
import numpy as np
import pytest

import aa_workloads as W
from gpu_util import device, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [100, 256, 512, 1024])
def test_end_at_the_tolerance_is_the_fixed_count(N):
    import torch
    device()
    from paper_2110_09667_amd import aa
    rhs = to_dev(W.normal(N, 8, N * N))
    ctx = aa.PDE2D(N, aa.PDE_BRATU)
    got = []
    for _ in range(4):
        x = torch.full_like(rhs, np.nan)
        ctx.solve(rhs, x)
        got.append((x.cpu().numpy(), ctx.last()))
    iters, conv = got[0][1]
    assert conv and 3 < iters < 200
    ctx.set_iters(iters)
    x = torch.full_like(rhs, np.nan)
    ctx.solve(rhs, x)
    ref = x.cpu().numpy()
    assert np.isfinite(ref).all()
    for v, last in got:
        assert last == (iters, True) and np.array_equal(v, ref)
