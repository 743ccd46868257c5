"""The work splits of the leaf passes of wide and adaptive leaves (a quarter of a leaf, a leaf or a group
per wave, by how many there are): an instance gives the same bits alone, where its leaves are split over
waves, as in forests large enough for the other splits, and is right against the oracle."""
import numpy as np
import pytest

from oracle import direct as od

pytestmark = pytest.mark.gpu


def _points(kind, n, rng):
    if kind == "curve":   # groups of two leaves
        t = np.sort(rng.uniform(0, 2 * np.pi, n))
        p = np.rint(3 * n * np.stack([1 + np.cos(t), 1 + np.sin(t)], 1))
    else:                 # full groups
        p = rng.integers(0, 16 * int(n ** 0.5), size=(n, 2))
    return np.ascontiguousarray(np.unique(p.astype(np.int32), axis=0))


# copies: enough for a wave per leaf, and (curves, groups of few leaves) a wave per group
@pytest.mark.parametrize("adaptive,kind,copies", [(False, "full", 12), (False, "curve", 12), (False, "curve", 80),
                                                  (True, "full", 40), (True, "curve", 48)])
def test_instance_alone_and_in_forests(adaptive, kind, copies):
    import torch

    import paper_1105_3505_amd as lf
    rng = np.random.default_rng(90)
    sets = [_points(kind, n, rng) for n in [3000] + [14000] * copies]
    loads = [rng.standard_normal(len(p)) for p in sets]
    ctx = lf.Context(0, adaptive=adaptive)
    dev = [torch.from_numpy(p).cuda() for p in sets]
    fs = [torch.from_numpy(f).cuda() for f in loads]
    alone = []
    for k in (0, 1):
        plan = ctx.plan(dev[k])
        assert adaptive or plan.info()["leaf_side"] >= 64
        alone.append(plan.execute(fs[k]).cpu().numpy())
        plan.close()
    plan = ctx.plan_batch(dev)
    assert plan.info()["n_leaves"] > 16384 or not adaptive
    us = plan.execute_instances(fs)
    plan.close()
    for k in (0, 1):
        assert np.array_equal(us[k].cpu().numpy(), alone[k])
    ctx.close()
    ref = od.direct_sum(sets[0], sets[0], loads[0])
    assert np.linalg.norm(alone[0] - ref) <= 1e-10 * np.linalg.norm(ref)   # the accuracy target
