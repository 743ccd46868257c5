"""Leaf pass at the edges of its work split, against the FP64 oracle (relative l2 <= 1e-10, the
accuracy target of the whole evaluation).

An 8 x 8 grid of leaves (leaf level 3, so the far field takes part) whose point counts sit around
the multiples the kernels split by: 8 and 16 targets per step of the far field, 32 and 64 targets
per wave, sources in steps of 16, 8, 4 and the rest; empty leaves; parents with one to four leaves.
Leaf sides 8 to 128 cover the window table, the quadrant table and the kernel for wide leaves.
Also plans whose groups number fewer than, about and more than the XCDs' shares of the walk.
"""
import numpy as np
import pytest

import workloads as wl
from oracle import direct as od

pytestmark = pytest.mark.gpu


def _solve(xy, f, max_leaf):
    import torch

    import paper_1105_3505_amd as lf
    ctx = lf.Context(0, max_leaf=max_leaf)
    plan = ctx.plan(torch.from_numpy(xy).cuda())
    info = plan.info()
    u = plan.execute(torch.from_numpy(f).cuda()).cpu().numpy()
    plan.close()
    ctx.close()
    return u, info


@pytest.mark.parametrize("side", [8, 16, 32, 64, 128])
@pytest.mark.parametrize("pick", [(0, 1, 2, 3, 5), (7, 8, 9, 15, 16, 17), (0, 31, 32, 33), (60, 63, 64), (1, 64, 0, 17)])
def test_leaf_counts(side, pick):
    rng = np.random.default_rng(1000 * side + pick[0] + 10 * pick[1])
    counts = rng.choice(pick, size=(8, 8))
    counts[2:4, 2:4] = [[64, 20], [3, 1]]          # a parent over N_leaf: the leaf level is 3
    pts = []
    for i in range(8):
        for j in range(8):
            c = rng.choice(side * side, size=counts[i, j], replace=False)
            pts.append(np.stack([i * side + c % side, j * side + c // side], 1))
    pts.append([[0, 0], [8 * side - 1, 8 * side - 1]])   # the corners fix the root box (may be duplicates)
    xy = np.ascontiguousarray(rng.permutation(np.concatenate(pts)).astype(np.int32))
    f = wl.zero_sum_loads(rng.standard_normal(len(xy)))
    u, info = _solve(xy, f, 65)
    assert (info["leaf_level"], info["leaf_side"]) == (3, side)
    ref = od.direct_sum(xy, xy, f)
    assert np.linalg.norm(u - ref) <= 1e-10 * np.linalg.norm(ref)


@pytest.mark.parametrize("n", [200, 1500, 7000, 30000])
def test_walk_of_few_groups(n):
    rng = np.random.default_rng(n)
    xy = np.ascontiguousarray(wl.uniform_box(rng, n, int(np.ceil(4 * np.sqrt(n)))))
    f = wl.zero_sum_loads(rng.standard_normal(n))
    u, _ = _solve(xy, f, 16)
    ref = od.direct_sum(xy, xy, f)
    assert np.linalg.norm(u - ref) <= 1e-10 * np.linalg.norm(ref)
