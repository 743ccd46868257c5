"""phi as the near field of wide and adaptive leaves computes it, at offsets around the changes of
its evaluation: the radius below which a table is read, powers of two of the squared distance and
the ends of the table's intervals, offsets up to the widest leaves and far beyond the tables.

One unit load at the origin and targets around it in a tree that sums every pair directly gives
u = phi(offset); compared with the host's phi (quadrature table, expansion beyond radius 128)
to 4e-15 absolute: the rounding of a handful of operations on values of order one (and the
expansion's own 4e-15 between the two forms).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = 4e-15


def _targets(offsets):
    o = np.array(sorted(set(offsets)), dtype=np.int64)
    return np.ascontiguousarray(o[(o[:, 0] != 0) | (o[:, 1] != 0)].astype(np.int32))


@pytest.mark.parametrize("stencil", [5, 9])
@pytest.mark.parametrize("adaptive", [False, True])
def test_phi_at_offsets(stencil, adaptive):
    import torch

    import paper_1105_3505_amd as lf
    rng = np.random.default_rng(77)
    ctx = lf.Context(0, stencil=stencil, adaptive=adaptive, max_leaf=4096)
    off = [(x, y) for x in (0, 1, 2, 33, 46, 47, 48, 49, 63, 64, 65, 127) for y in (0, 1, 31, 33, 34, 47, 48, 63, 127)]
    off += [tuple(v) for v in rng.integers(0, 128, size=(300, 2))]
    for r2 in [2304] + [1 << k for k in range(11, 17)]:       # both sides of the changes of interval
        for x in range(0, 128, 3):
            y = int(np.sqrt(max(r2 - x * x, 0)))
            off += [(x, y + d) for d in (-1, 0, 1) if 0 <= y + d < 128]
    src = np.zeros((1, 2), dtype=np.int32)
    for sx, sy in ((1, 1), (-1, 1), (1, -1), (-1, -1)):       # each quadrant, widest near offsets 127 .. 255
        tgt = _targets([(x, y) for x, y in off]) * np.array([sx, sy], dtype=np.int32)
        tgt = np.ascontiguousarray(np.concatenate([tgt, [[127 * sx, 127 * sy], [0, 127 * sy]]]).astype(np.int32))
        plan = ctx.plan(torch.from_numpy(src).cuda(), targets=torch.from_numpy(tgt).cuda())
        u = plan.execute(torch.ones(1, dtype=torch.float64, device="cuda")).cpu().numpy()
        side = plan.info()["leaf_side"]
        plan.close()
        assert side >= 64                                     # the kernels under test
        assert np.max(np.abs(u - lf.host_phi(tgt, stencil=stencil))) <= TOL
    ctx.close()


def test_phi_at_far_offsets_of_adaptive_leaves():
    """Few points far apart: every pair is direct (no box has more points than the skeleton)."""
    import torch

    import paper_1105_3505_amd as lf
    rng = np.random.default_rng(78)
    d = np.concatenate([2 ** np.arange(5, 30), 3 * 2 ** np.arange(5, 28)])
    tgt = np.stack([d, rng.integers(0, d + 1)], 1).astype(np.int32)
    ctx = lf.Context(0, adaptive=True, max_leaf=2)
    plan = ctx.plan(torch.zeros((1, 2), dtype=torch.int32, device="cuda"), targets=torch.from_numpy(tgt).cuda())
    u = plan.execute(torch.ones(1, dtype=torch.float64, device="cuda")).cpu().numpy()
    ref = lf.host_phi(tgt)
    assert np.max(np.abs(u - ref) / np.abs(ref)) <= TOL
    plan.close()
    ctx.close()
