"""M2L kernels chosen by plan size: 16-box column blocks for small plans, half tiles, whole tiles.

All of them run the same products in the same order per box, so an instance's potentials are
the same bits alone (16-box kernel) and in a forest with a companion that moves the launch to
the half-tile or whole-tile kernel.  Point sets at the edges: partly filled column blocks (a
few boxes per class), lists with most slots absent (points on a curve), one full tile and more.
FP64 results also meet the accuracy target against the oracle (relative l2 <= 1e-10).
"""
import numpy as np
import pytest

import workloads as wl
from oracle import direct as od

pytestmark = pytest.mark.gpu


def _curve(m):
    t = np.arange(1, m)
    return np.concatenate([np.stack([0 * t, t], 1), np.stack([t, 0 * t + m], 1)]).astype(np.int32)


def _instances():
    rng = np.random.default_rng(911)
    sets = [wl.uniform_box(rng, 300, 90), wl.uniform_box(rng, 1000, 256), wl.uniform_box(rng, 1100, 4000),
            wl.uniform_box(rng, 9000, 300), _curve(1500)]
    return [(np.ascontiguousarray(xy), wl.zero_sum_loads(rng.standard_normal(len(xy)))) for xy in sets]


@pytest.mark.parametrize("companion", [250_000, 850_000])
@pytest.mark.parametrize("precision", ["fp64", "mixed", "mixed-bf16"])
def test_same_bits_from_every_m2l_kernel(precision, companion):
    import torch

    import paper_1105_3505_amd as lf
    dev = lambda a: torch.from_numpy(a).cuda()
    inst = _instances()
    rng = np.random.default_rng(companion)
    big = wl.uniform_box(rng, companion, int(np.ceil(4 * np.sqrt(companion))))
    ctx = lf.Context(0, precision=precision)
    alone = []
    for xy, f in inst:
        plan = ctx.plan(dev(xy))
        u = plan.execute(dev(f))
        if precision == "fp64":
            ref = od.direct_sum(xy, xy, f)
            assert np.linalg.norm(u.cpu().numpy() - ref) <= 1e-10 * np.linalg.norm(ref)
        alone.append(u)
        plan.close()
    plan = ctx.plan_batch([dev(xy) for xy, _ in inst] + [dev(big)])
    us = plan.execute_instances([dev(f) for _, f in inst] + [dev(wl.zero_sum_loads(rng.standard_normal(companion)))])
    for a, b in zip(alone, us):
        assert torch.equal(a, b)
    plan.close()
    ctx.close()
