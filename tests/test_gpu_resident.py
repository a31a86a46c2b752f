"""The register-resident one-workgroup step at the edges of its shapes (rows
per lane 1, 2, 4, 8; windows up to 8, 20, 10 and 5 columns) through window
recycling: every iterate against the CPU oracle, Q's orthonormality and the
rows of T against the basis.

Tolerance 1e-10 on the iterates, as for the other paths: 1e-15 roundings
times the conditioning of the least-squares problems of these windows (at most
1e4 over these iterations).  Windows of 20 on these 1D problems reach 1e6 (the
grid-wide passes part from the oracle by 1.7e-10 there too), so the widest
shapes are held to what does not depend on it: Q R = F of the differences the
kernel itself was given (a few roundings per column and rotation: 100 m eps),
Q's orthonormality and T."""
import numpy as np
import pytest

import aa_workloads as W
import oracle as O
from gpu_util import device, rel, to_dev

pytestmark = pytest.mark.gpu

SHAPES = [(20, 1), (64, 8), (511, 3), (512, 9), (513, 8), (513, 9), (1025, 5), (2048, 10),
          (2049, 2), (4095, 5), (4096, 5)]


@pytest.mark.parametrize("variant,flags", [("mgs", 0), ("cgs2", 0), ("dcgs2", 0), ("dcgs2", 1 << 4),
                                           ("icwy", 0), ("icwy", (1 << 3) | (1 << 5))])
@pytest.mark.parametrize("n,m", SHAPES)
def test_step_matches_oracle(n, m, variant, flags):
    import torch
    device()
    from paper_2110_09667_amd import aa
    prob = W.StencilProblem(d=1, s=n, c=1.0, f=W.uniform(n, 0, n))
    iters = m + 4
    oflags = O.DCGS2_GUARD_GE3 if flags & aa.DCGS2_GUARD_GE3 else 0
    xs, _, _ = O.run_aa(lambda u: O.G_stencil(prob, u), np.zeros(n), m, variant, iters, oflags)
    f = to_dev(prob.f)
    ctx = aa.AAContext(n, m, variant, flags)
    x = torch.zeros(n, dtype=torch.float64, device="cuda")
    g = torch.empty_like(x)
    for i in range(iters + 1):
        aa.aa_problem_apply(1, n, prob.h, prob.omega, prob.c, f, x, g)
        ctx.step(x, g, x)
        assert rel(x.cpu().numpy(), xs[i + 1]) <= 1e-10, i
    info = ctx.info()
    assert info.status == 0 and info.k == m and info.m_i == m and info.stopped == 0
    Q = ctx.basis(m).cpu().numpy()
    R, T, k = ctx.get_qr()
    assert np.all(np.tril(R, -1) == 0.0)
    # the least-squares factors: orthonormal up to the variant's loss
    assert np.linalg.norm(np.eye(m) - Q.T @ Q) <= 1e-8
    if variant == "icwy" and m > 2:
        G = np.tril(Q.T @ Q, -1)[: m - 1]
        assert np.abs(np.tril(T, -1)[: m - 1] - G).max() <= 1e-12
    ctx.close()


@pytest.mark.parametrize("variant,flags", [("mgs", 0), ("cgs2", 0), ("dcgs2", 1 << 4), ("icwy", 0)])
@pytest.mark.parametrize("n", [24, 512, 1024])
def test_widest_window_factors_its_differences(n, variant, flags):
    import torch
    device()
    from paper_2110_09667_amd import aa
    m, eps = 20, 2.0 ** -52
    prob = W.StencilProblem(d=1, s=n, c=1.0, f=W.uniform(n, 0, n))
    f = to_dev(prob.f)
    ctx = aa.AAContext(n, m, variant, flags)
    x = torch.zeros(n, dtype=torch.float64, device="cuda")
    g = torch.empty_like(x)
    res = []
    for i in range(m + 4 if n > 24 else 12):
        aa.aa_problem_apply(1, n, prob.h, prob.omega, prob.c, f, x, g)
        res.append((g - x).cpu().numpy())
        ctx.step(x, g, x)
        if i == 0:
            continue
        F = np.diff(np.array(res), axis=0)[-m:].T
        k = F.shape[1]
        Q = ctx.basis(k).cpu().numpy()
        R, T, kk = ctx.get_qr()
        assert kk == k and np.all(np.tril(R, -1) == 0.0)
        assert np.linalg.norm(Q @ R - F) <= 100 * m * eps * np.linalg.norm(F), i
        if variant == "icwy" and k > 2:
            assert np.abs(np.tril(T - Q.T @ Q, -1)[: k - 1]).max() <= 1e-12
    assert ctx.info().status == 0
    ctx.close()
