"""Callers' vectors at the alignment of a double: a slice from an odd element
gives the values of an aligned one, and nothing beside it is touched."""
import numpy as np
import pytest

import aa_workloads as W
from gpu_util import device, to_dev

pytestmark = pytest.mark.gpu


def odd(n):
    """(buffer of NaN, its slice of n doubles that starts 8 bytes off 16)."""
    import torch
    buf = torch.full((n + 3,), np.nan, dtype=torch.float64, device="cuda")
    assert buf.data_ptr() % 16 == 0
    return buf, buf[1:1 + n]


@pytest.mark.parametrize("replicas", [1, 2, 171, 100_003])
def test_em_replicas(replicas):
    import torch
    device()
    from paper_2110_09667_amd import aa
    p = W.em_problem(nsamples=3000, replicas=replicas)
    u, x = to_dev(p.u0()), to_dev(p.samples)
    ref = torch.empty_like(u)
    work = torch.empty(aa.EM_WORK_DOUBLES, dtype=torch.float64, device="cuda")
    aa.aa_em_apply(p.alpha, p.sigma, x, u, ref, work)
    buf, out = odd(p.n)
    aa.aa_em_apply(p.alpha, p.sigma, x, u, out, work)
    assert torch.equal(out, ref)
    assert torch.isnan(buf[0]) and torch.isnan(buf[1 + p.n:]).all()
