"""aa_batch_set_split(b, 0, 0) leaves every instance with one workgroup, the
cost model's choices too: each is summed in the order of that workgroup, bit for
bit what the learned entry points (which have no other path) compute with a
network that corrects nothing, and what the same instance gives in another
batch of the same windows; a later min_n > 0 brings the choices back."""
import numpy as np
import pytest

import aa_workloads as W
from gpu_util import device

pytestmark = pytest.mark.gpu

VARIANTS = ["mgs", "cgs2", "dcgs2", "icwy"]
M = 10


def problems(sides):
    return [W.StencilProblem(d=2, s=s, c=0.5, f=W.uniform(s, 1, s * s)) for s in sides]


def run(aa, probs, variant, splits=(), flags=0, iters=(5, 8)):
    b = aa.AABatch(probs, [M] * len(probs), variant, flags=flags, tol=0.0, max_iter=10 ** 9)
    for s in splits:
        b.set_split(*s)
    for k in iters:
        b.run(k)
    st, _ = b.read()
    assert all(s.iter == sum(iters) and s.status == 0 for s in st)
    return [x.cpu().numpy() for x in b.x]


@pytest.mark.parametrize("variant", VARIANTS)
def test_off_is_one_workgroup_an_instance(variant):
    device()
    from paper_2110_09667_amd import aa
    # 180: 0.26 MB a vector, wide by the cost model with every variant (no split
    # policy at 13 iterations: n < 65536)
    probs = problems((180, 31, 77, 150))
    wide = run(aa, probs, variant)
    off = run(aa, probs, variant, [(0, 0)])
    back = run(aa, probs, variant, [(0, 0), (65536, 0)])
    alone = run(aa, probs[:1], variant, [(0, 0)])
    assert not np.array_equal(wide[0], off[0])
    assert all(np.array_equal(a, b) for a, b in zip(wide, back))
    assert np.array_equal(alone[0], off[0])
    net = aa.AAMlp(len(probs))
    p = np.zeros(net.P, dtype=np.float32)
    p[-64 + 20] = 40.0  # beta = 1 in double precision, no correction
    net.set_params(p)
    lrn = aa.AABatch(probs, [M] * len(probs), variant, flags=aa.BATCH_LEARNED, tol=0.0,
                     max_iter=10 ** 9)
    lrn.run_learned(net, 13)
    lrn.read()
    for j in range(len(probs)):
        assert np.array_equal(lrn.x[j].cpu().numpy(), off[j]), j


def test_switched_while_a_replay_is_enqueued():
    """Runs replayed as graphs and not waited for, the switch thrown between them:
    each change of the wide set lets the replay end first, and the iterates are
    those of waited-for runs bit for bit."""
    import torch
    device()
    from paper_2110_09667_amd import aa
    probs = problems((180, 31, 77, 150))
    got = []
    for wait in (True, False):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            b = aa.AABatch(probs, [M] * len(probs), "icwy", tol=0.0, max_iter=10 ** 9,
                           stream=stream)
            for min_n in (65536, 0, 65536, 1, 0):
                b.set_split(min_n, 64)
                b.run(6)
                if wait:
                    stream.synchronize()
            st, _ = b.read()
        assert all(s.iter == 30 and s.status == 0 for s in st)
        got.append([x.cpu().numpy() for x in b.x])
    for x, y in zip(*got):
        assert np.isfinite(x).all() and np.array_equal(x, y)
