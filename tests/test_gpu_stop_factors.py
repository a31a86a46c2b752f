"""The stopping test that a later pass completes for itself (grid-wide steps of
at most 2^19 rows): the factorization of the last iteration that ran is left as
it was.  The step in which the test holds has computed rotations and started
passes over Q, so every workgroup of every pass must take the same end: Q R = F
of the differences the steps were given (a few roundings per column and
rotation: 100 m eps), Q orthonormal (the windows' condition numbers stay below
1e3 here, so 1e-9 holds eps times their square), the iterate unchanged."""
import numpy as np
import pytest

import aa_workloads as W
from gpu_util import device, to_dev

pytestmark = pytest.mark.gpu
RHS, T_TRANSFORM, DELETE = 1 << 3, 1 << 2, 1 << 5
EPS = 2.0 ** -52


@pytest.mark.parametrize("variant,flags", [
    ("mgs", 0), ("cgs2", 0), ("cgs2", RHS | DELETE), ("dcgs2", 0), ("dcgs2", RHS | DELETE),
    ("icwy", 0), ("icwy", RHS), ("icwy", RHS | DELETE), ("icwy", T_TRANSFORM)])
@pytest.mark.parametrize("s", [41, 250, 701])
def test_stop_leaves_the_last_factorization(s, variant, flags):
    import torch
    device()
    from paper_2110_09667_amd import aa
    m, stop = 6, 9  # ||f_8|| = 7.2e-3, ||f_9|| = 5.2e-3 of ||f_0|| (any s): a full window
    n = s * s
    prob = W.StencilProblem(d=2, s=s, c=0.7, f=W.uniform(s, 0, n))
    f = to_dev(prob.f)
    ctx = aa.AAContext(n, m, variant, flags)
    ctx.set_fused_threshold(0)
    ctx.set_stop(6e-3, 0, aa.STOP_RESIDUAL)
    x = to_dev(W.normal(s, 1, n))
    g = torch.empty_like(x)
    res, xs = [], []
    for _ in range(stop + 4):
        aa.aa_problem_apply(2, s, prob.h, prob.omega, prob.c, f, x, g)
        res.append((g - x).cpu().numpy())
        xs.append(x.clone())
        ctx.step(x, g, x)
    info = ctx.info()
    assert info.status == 0 and info.stopped == aa.STOPPED_TEST and info.k == m
    i = info.stop_iter
    assert i == stop
    assert all(torch.equal(v, xs[i]) for v in xs[i:]) and torch.equal(x, xs[i])
    F = np.diff(np.array(res[:i]), axis=0)[-m:].T
    Q = ctx.basis(m).cpu().numpy()
    R, _, k = ctx.get_qr()
    assert k == m
    assert np.linalg.norm(Q @ R - F) <= 100 * m * EPS * np.linalg.norm(F)
    assert np.linalg.norm(np.eye(m) - Q.T @ Q) <= 1e-9
    ctx.close()
