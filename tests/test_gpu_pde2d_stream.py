"""A context of the 2D problems set up on one stream and used on another: what
its first cycle reads of the workspace (the matrix of the coarsest levels) is in
place when the set-up call returns, however busy the stream of that call was."""
import numpy as np
import pytest

import aa_workloads as W
from gpu_util import device, rel_inf, to_dev
from oracle import pde2d as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [64, 160])
def test_first_cycle_on_another_stream(N):
    import torch
    device()
    from paper_2110_09667_amd import aa
    r = W.normal(N, 9, N * N)
    ref = P.vcycle(r.reshape(N, N), 1.0 / (N + 1)).reshape(-1)
    rd = to_dev(r)
    z = torch.full_like(rd, np.nan)
    ws = torch.zeros((aa.aa_pde2d_workspace_size(N, 200) + 7) // 8, dtype=torch.float64,
                     device="cuda")
    busy, other = torch.cuda.Stream(), torch.cuda.Stream()
    a = torch.ones(2048, 2048, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(busy):
        for _ in range(20):  # milliseconds of work ahead of the set-up's kernels
            a = a @ a * 0.0 + 1.0
    ctx = aa.aa_pde2d_init(N, aa.PDE_BRATU, 6.7, 1e-10, 200, ws, busy)
    aa.aa_pde2d_set_stream(ctx, other)
    aa.aa_pde2d_vcycle(ctx, rd, z)
    other.synchronize()
    assert rel_inf(z.cpu().numpy(), ref) <= 1e-13
    aa.aa_pde2d_destroy(ctx)
