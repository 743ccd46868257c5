"""M2M and L2L of several levels in one launch: plans that use it (one tree, or trees of one height) give the
same bits as the passes level by level, which a forest of trees of different heights takes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _curve(n, rng):
    t = np.sort(rng.uniform(0, 2 * np.pi, n))
    return np.unique(np.rint(3 * n * np.stack([1 + np.cos(t), 1 + np.sin(t)], 1)).astype(np.int32), axis=0)


def _square(n, rng):
    return np.unique(rng.integers(0, int((10 * n) ** 0.5), size=(n, 2)).astype(np.int32), axis=0)


# leaf levels 4 (two levels), 5 (three), 7 and 9 (four, and four and two or three) and 12 (two stages of four)
@pytest.mark.parametrize("make,n,adaptive", [(_square, 4000, False), (_square, 20000, False), (_square, 300000, False),
                                             (_curve, 1500, False), (_curve, 9000, False), (_curve, 40000, False),
                                             (_curve, 250000, False), (_curve, 40000, True)])
def test_same_bits_as_level_by_level(make, n, adaptive):
    import torch

    import paper_1105_3505_amd as lf
    rng = np.random.default_rng(n)
    ctx = lf.Context(0, adaptive=adaptive)
    sets = [make(n, rng), _square(700, rng)]
    fs = [torch.from_numpy(rng.standard_normal(len(p))).cuda() for p in sets]
    dev = [torch.from_numpy(p).cuda() for p in sets]
    one = ctx.plan(dev[0])
    u = one.execute(fs[0]).cpu().numpy()
    again = one.execute(fs[0]).cpu().numpy()
    both = ctx.plan_batch(dev)
    assert one.info()["leaf_level"] >= 4
    v = both.execute_instances(fs)[0].cpu().numpy()
    ctx.close()
    assert np.array_equal(u, again) and np.array_equal(u, v)
