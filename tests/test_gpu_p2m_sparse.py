"""P2M of more than 8,192 leaves too wide for an operator in LDS: eight leaves per wave, or a wave per leaf where the
leaves are uneven (12 points on average and more, but less than 0.15 N_leaf).  The same instance gives the
same bits alone (a wave per leaf) and in forests on either side, and is right against the oracle."""
import numpy as np
import pytest

from oracle import direct as od

pytestmark = pytest.mark.gpu


# points per leaf on average, and N_leaf, which a single full leaf brings about
@pytest.mark.parametrize("side", [32, 64])
@pytest.mark.parametrize("mean,max_leaf,uneven", [(5, 20, False), (14, 400, True), (30, 80, False)])
def test_alone_and_in_a_forest(side, mean, max_leaf, uneven):
    import torch

    import paper_1105_3505_amd as lf
    rng = np.random.default_rng(side + mean)
    n_leaf = max_leaf + 2 * mean   # more than the fullest leaf holds, less than its parent

    def leaves(w, mean):   # about mean points in each leaf of a w x w grid, and max_leaf more in one of them
        c = rng.choice((w * side) ** 2, size=w * w * mean, replace=False)
        d = rng.choice(side * side, size=max_leaf, replace=False)
        c = np.unique(np.concatenate([c, (side + d // side) * w * side + side + d % side]))
        return np.ascontiguousarray(np.stack([c // (w * side), c % (w * side)], 1).astype(np.int32))

    first = leaves(16, mean)
    sets = [first] + [leaves(64, mean) for _ in range(3)]
    loads = [rng.standard_normal(len(p)) for p in sets]
    ctx = lf.Context(0, max_leaf=n_leaf)
    dev = [torch.from_numpy(p).cuda() for p in sets]
    fs = [torch.from_numpy(f).cuda() for f in loads]
    plan = ctx.plan(dev[1])
    assert plan.info()["leaf_side"] == side and plan.info()["n_leaves"] > 2731   # so that three make 8,193
    plan.close()
    plan = ctx.plan(dev[0])
    alone = plan.execute(fs[0]).cpu().numpy()
    plan.close()
    forest = ctx.plan_batch(dev)
    info = forest.info()
    per = info["n_points"] / info["n_leaves"]
    assert info["n_leaves"] > 8192 and (12 < per < 0.15 * n_leaf) == uneven
    us = forest.execute_instances(fs)
    assert np.array_equal(us[0].cpu().numpy(), alone)
    u1 = us[1].cpu().numpy()
    ctx.close()
    ref = od.direct_sum(first, first, loads[0])
    assert np.linalg.norm(alone - ref) <= 1e-10 * np.linalg.norm(ref)   # the accuracy target
    some = rng.choice(len(sets[1]), size=400, replace=False)
    ref = od.direct_sum(sets[1][some], sets[1], loads[1])
    assert np.linalg.norm(u1[some] - ref) <= 1e-10 * np.linalg.norm(ref)
