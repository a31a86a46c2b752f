"""The passes with many workgroups per instance against the CPU oracle beyond
what the other batch tests reach: the wide window buckets (17 to 64 columns, with
and without the merged passes), maps in one, two and three dimensions with odd
sides, more chunks than a wave sums at once, windows of different widths in one
batch; a breakdown of an instance that the cost model chose; a candidate of the
learned step taken over by a plain run.

Tolerance: every step's least-squares problem turns roundings into eps times the
condition number of R with its columns scaled to one length, so (steps) eps
max(kappa) relative; kappa is the oracle's, at most 2e5 here (random starts, and
in one dimension a strong cubic term, keep the windows apart: with x_0 = 0 a
window of 63 reaches 1e14)."""
import functools

import numpy as np
import pytest

import aa_workloads as W
import oracle as O
from gpu_util import device, rel, to_dev

pytestmark = pytest.mark.gpu

VARIANTS = ["mgs", "cgs2", "dcgs2", "icwy"]
EPS = 2.0 ** -52
CUBIC = {1: 1e4, 2: 0.7, 3: 0.7}


@functools.lru_cache(maxsize=None)
def instance(d, s):
    n = s ** d
    return (W.StencilProblem(d=d, s=s, c=CUBIC[d], f=W.uniform(s, 0, n)), W.normal(s, 1, n))


@functools.lru_cache(maxsize=None)
def reference(d, s, m, variant, iters):
    """x after `iters` + 1 steps, ||f|| and ||f_0||, the largest scaled kappa."""
    p, x = instance(d, s)
    st, kappa = O.AA(p.n, m, variant), 1.0
    for _ in range(iters + 1):
        x = st.step(x, O.G_stencil(p, x))
        if st.k:
            R = st.Rk()
            kappa = max(kappa, np.linalg.cond(R / np.linalg.norm(R, axis=0)))
    return x, st.res_norm, st.res0_norm, kappa


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("variant", VARIANTS)
@pytest.mark.parametrize("m", [17, 33, 63, 64])
def test_wide_windows_match_oracle(m, variant, fused):
    device()
    from paper_2110_09667_amd import aa
    shapes = [(1, 2049), (2, 47), (3, 13)] + ([(1, 70_001)] if m == 17 else [])
    ms = [m, m, m - 1, m][:len(shapes)]
    iters = m + 6
    probs = [instance(d, s)[0] for d, s in shapes]
    x0 = [to_dev(instance(d, s)[1]) for d, s in shapes]
    b = aa.AABatch(probs, ms, variant, flags=aa.FUSE_RHS | aa.FUSE_DELETE if fused else 0,
                   tol=0.0, max_iter=10 ** 9, x0=x0)
    b.set_split(1, 64)
    b.run(1)
    b.run(2)
    assert b.split_count() == len(shapes)  # every iteration from i = 1 on
    b.run(iters - 2)
    states, active = b.read()
    assert active == len(shapes)
    for j, (d, s) in enumerate(shapes):
        x, res, res0, kappa = reference(d, s, ms[j], variant, iters)
        tol = (iters + 1) * EPS * kappa
        assert kappa <= 2e5
        assert rel(b.x[j].cpu().numpy(), x) <= tol, (d, s)
        assert states[j].iter == iters + 1 and states[j].status == 0
        assert states[j].k == states[j].m_i == ms[j] and states[j].g_evals == iters + 1
        assert abs(states[j].res_norm - res) <= tol * res0


def degenerate(s, jx, jy):
    """A right-hand side that is an eigenvector: every f_i is a multiple of f_0
    to rounding, so the second column lies in the span of the first."""
    i = np.arange(1, s + 1) * np.pi / (s + 1)
    return W.StencilProblem(d=2, s=s, c=0.0, f=np.outer(np.sin(jy * i), np.sin(jx * i)).reshape(-1))


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("variant", VARIANTS)
def test_breakdown_under_the_cost_model(variant, fused):
    """An instance that breaks down in iteration 2 is ended by iteration 3's test,
    as with one workgroup an instance; its neighbours go on.  The split policy
    ends it in iteration 2 with x = G(x_2), the solution to rounding."""
    device()
    from paper_2110_09667_amd import aa
    m, probs = 4, [instance(2, 150)[0], degenerate(151, 60, 80), instance(2, 149)[0]]
    flags = aa.FUSE_RHS | aa.FUSE_DELETE if fused else 0
    got = {}
    for name, split in (("cost", None), ("one workgroup", (0, 0)), ("split", (1, 64))):
        b = aa.AABatch(probs, [m] * 3, variant, flags=flags, tol=0.0, max_iter=10 ** 9)
        if split:
            b.set_split(*split)
        b.run(1)
        b.run(8)
        st, active = b.read()
        assert active == 2
        got[name] = ([(t.iter, t.stop_iter, t.k, t.m_i, t.active, t.status, t.g_evals)
                      for t in st], [x.cpu().numpy() for x in b.x])
    assert not np.array_equal(got["cost"][1][0], got["one workgroup"][1][0])  # another path
    assert got["cost"][0] == got["one workgroup"][0]
    it, stop, k, m_i, alive, status, evals = got["cost"][0][1]
    assert (it, stop, k, m_i, alive, evals) == (3, 3, 2, 2, 0, 4) and status < 0
    it, stop, k, m_i, alive, st, evals = got["split"][0][1]
    assert (it, stop, k, m_i, alive, evals) == (2, 2, 2, 2, 0, 3) and st == status
    p = probs[1]
    lam = sum(4.0 / p.h ** 2 * np.sin(j * np.pi * p.h / 2) ** 2 for j in (60, 80))
    assert rel(got["split"][1][1], p.f / lam) <= 1e-12
    for j in (0, 2):
        assert got["cost"][0][j][:6] == (9, -1, m, m, 1, 0)
        assert rel(got["cost"][1][j], got["one workgroup"][1][j]) <= 1e-11


@pytest.mark.parametrize("variant", VARIANTS)
def test_plain_run_takes_over_a_learned_candidate(variant):
    """After learned iterations whose candidates were accepted G(x_i) is known:
    the plain run that follows uses it instead of evaluating the map, with many
    workgroups an instance as with one."""
    device()
    from paper_2110_09667_amd import aa
    probs = [instance(2, s)[0] for s in (180, 77, 150)]
    net = aa.AAMlp(3)
    p = np.zeros(net.P, dtype=np.float32)
    p[-64 + 20] = 40.0  # beta = 1 in double precision, no correction
    net.set_params(p)
    got = []
    for split in (None, (0, 0)):
        b = aa.AABatch(probs, [10] * 3, variant, flags=aa.BATCH_LEARNED, tol=0.0,
                       max_iter=10 ** 9)
        if split:
            b.set_split(*split)
        b.run_learned(net, 6)
        before, _ = b.read()
        assert any(t.g_valid for t in before)
        b.run(7)
        st, _ = b.read()
        for t, t0 in zip(st, before):
            assert t.iter == 13 and t.status == 0 and not t.g_valid
            assert t.g_evals == t0.g_evals + 7 - (1 if t0.g_valid else 0)
        got.append([x.cpu().numpy() for x in b.x])
    for x, y in zip(*got):
        assert rel(x, y) <= 1e-11 and not np.array_equal(x, y)
