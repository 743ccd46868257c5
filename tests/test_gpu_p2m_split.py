"""P2M by a wave per leaf (plans of up to 8,192 leaves) and by groups of eight leaves (more), with the operator in
LDS (sides up to 16) and in memory: an instance gives the same bits alone and in a forest of more leaves, with
loads in the caller's order and sorted, with sources and targets apart, and is right against the oracle."""
import numpy as np
import pytest

from oracle import direct as od

pytestmark = pytest.mark.gpu


# mean points per cell of the root box: leaf sides 8, 16, 32, 64
@pytest.mark.parametrize("density,side", [(0.4, 8), (0.1, 16), (0.025, 32), (0.006, 64)])
def test_instance_alone_and_in_a_forest(density, side):
    import torch

    import paper_1105_3505_amd as lf
    rng = np.random.default_rng(side)

    def points(n):
        w = int((n / density) ** 0.5)
        c = rng.choice(w * w, size=n, replace=False)
        return np.ascontiguousarray(np.stack([c // w, c % w], 1).astype(np.int32))

    sets = [points(n) for n in (3001, 6000)] + [points(25000) for _ in range(24)]
    tgts = [points(500), None] + [None] * 24
    loads = [rng.standard_normal(len(p)) for p in sets]
    ctx = lf.Context(0)
    dev = [torch.from_numpy(p).cuda() for p in sets]
    tdev = [None if t is None else torch.from_numpy(t).cuda() for t in tgts]
    fs = [torch.from_numpy(f).cuda() for f in loads]
    forest = ctx.plan_batch(dev, targets=tdev)
    assert forest.info()["n_leaves"] > 8192
    us = forest.execute_instances(fs)
    alone = []
    for k in (0, 1, 2):
        plan = ctx.plan(dev[k], targets=tdev[k])
        alone.append(plan.execute(fs[k]).cpu().numpy())
        if k == 1:
            assert plan.info()["leaf_side"] == side
            perm = plan.export("perm")
            v = plan.execute_sorted(fs[k][torch.from_numpy(perm).cuda().long()].contiguous()).cpu().numpy()
            assert np.array_equal(v, alone[k][perm])
        plan.close()
        assert np.array_equal(us[k].cpu().numpy(), alone[k])
    ctx.close()
    ref = od.direct_sum(tgts[0], sets[0], loads[0])
    assert np.linalg.norm(alone[0] - ref) <= 1e-10 * np.linalg.norm(ref)   # the accuracy target
