"""The schedule autotuner beside the passes with many workgroups per instance:
it chooses a schedule of the persistent kernel, so it searches only where that
kernel has instances, and over those."""
import numpy as np
import pytest

import aa_workloads as W
from gpu_util import device, rel

pytestmark = pytest.mark.gpu

# side 64 and up, window 10: 1.9 MB an iteration and instance, beyond the size
# up to which a few instances stay with one workgroup each
SIDES, WINDOW = (64, 71, 80), 10


def batch(flags=0):
    from paper_2110_09667_amd import aa
    probs = [W.StencilProblem(d=2, s=s, c=0.5, f=W.uniform(s, 1, s * s)) for s in SIDES]
    return aa.AABatch(probs, [WINDOW] * len(probs), "icwy", flags=flags, tol=0.0,
                      max_iter=10 ** 9)


def old_signature(flags):
    """FNV-1a of format 2: variant, flags, every instance's (n, m, dim)."""
    h = 1469598103934665603
    for v in [2, 3, flags] + [w for s in SIDES for w in (s * s, WINDOW, 2)]:
        for i in range(8):
            h = ((h ^ (v >> (8 * i) & 0xff)) * 1099511628211) % 2 ** 64
    return "%016x" % h


def test_no_instance_in_the_persistent_kernel_nothing_to_tune(tmp_path):
    device()
    cache = tmp_path / "tune.txt"
    bt, bp = batch(), batch()
    bt.set_schedule(grid=7, order=1, use_graph=False)
    bt.run(12)
    bp.run(12)
    best = bt.autotune(2, str(cache))
    assert best.trials == 1 and best.ms_per_iter > 0
    assert (best.grid, best.order, best.pairs) == (7, 1, 4)
    assert not cache.exists()
    bp.run(2)
    st, _ = bt.read()
    bp.read()
    for j in range(len(SIDES)):
        assert st[j].iter == 14 and np.array_equal(bt.x[j].cpu().numpy(), bp.x[j].cpu().numpy())


def test_learned_batch_is_tuned_on_all_its_instances(tmp_path):
    """The trials run the kernel that the learned entry points run: sums in that
    kernel's order (not bit for bit the plain run's, which agrees to rounding),
    and no schedule measured by an earlier format is taken up."""
    device()
    from paper_2110_09667_amd import aa
    cache = tmp_path / "tune.txt"
    bt, bp = batch(aa.BATCH_LEARNED), batch(aa.BATCH_LEARNED)
    bt.run(12)
    bp.run(12)
    bt.read()
    import torch
    arch = torch.cuda.get_device_properties(0).gcnArchName
    cache.write_text(f"{arch} {old_signature(aa.BATCH_LEARNED)} 1 0 2 0.5\n")
    best = bt.autotune(2, str(cache))
    assert best.trials >= 2 and best.grid >= 1
    assert len(cache.read_text().splitlines()) == 2
    done = 12 + 2 * best.trials
    bp.run(done - 12)
    st, _ = bt.read()
    bp.read()
    for j in range(len(SIDES)):
        a, b = bt.x[j].cpu().numpy(), bp.x[j].cpu().numpy()
        assert st[j].iter == done and rel(a, b) <= 1e-9
        assert not np.array_equal(a, b)
    assert bp.autotune(2, str(cache)).trials == 0
