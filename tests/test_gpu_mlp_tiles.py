"""The network kernels at the edges of their tiles (16 batch rows per workgroup
in the forward and backward chains, 64-row steps and 32 row slices in the
gradient kernel) against the BF16-emulating oracle.  Tolerance: BF16 rounding
flips of an FP32 sum (2^-9 on single activations, averaged over 256 of them)
stay below 1e-3 of the result's norm, as for the other batch sizes."""
import numpy as np
import pytest

import aa_workloads as W
from gpu_util import device
from oracle import mlp as M
from test_gpu_mlp import packed_random, unpack

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [1, 15, 16, 17, 63, 64, 65, 129])
def test_forward_backward_at_tile_edges(batch):
    import torch
    device()
    from paper_2110_09667_amd import aa
    net = aa.AAMlp(batch + 3)
    flat, params = packed_random(41)
    net.set_params(flat)
    X = W.normal(42, 0, batch * M.NF).reshape(batch, M.NF).astype(np.float32)
    D = W.normal(43, 0, batch * M.NO).reshape(batch, M.NO).astype(np.float32)
    out = torch.full((batch, M.NO), np.nan, dtype=torch.float32, device="cuda")
    net.forward(torch.from_numpy(X).cuda(), out)
    ref, cache = M.forward(params, X.astype(np.float64))
    r = ref[:, :M.NO]
    assert np.linalg.norm(out.cpu().numpy() - r) <= 1e-3 * np.linalg.norm(r)
    dout = np.zeros((batch, M.NOUT))
    dout[:, :M.NO] = D
    gref = M.backward(params, cache, dout)
    for times in (1, 2):  # gradients accumulate; the kept activations are not consumed
        net.backward(torch.from_numpy(D).cuda())
        got = unpack(net.get_grads().astype(np.float64))
        for l in range(4):
            for a, b in ((got[l][0], gref[l][0]), (got[l][1], gref[l][1])):
                assert np.linalg.norm(a - times * b) <= 1e-3 * times * np.linalg.norm(b), (l, times)
