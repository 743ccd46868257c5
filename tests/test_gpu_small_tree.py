"""Trees of at most 2,048 points, whose order and level statistics come from one launch: the same order as a
stable sort by Morton key, and the same tree and bits as in a forest, which is built by the general path."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _morton(xy):
    d = (xy.astype(np.int64) - xy.min(0)).astype(np.uint64)
    m = np.zeros(len(xy), np.uint64)
    for b in range(31):
        m |= ((d[:, 0] >> np.uint64(b)) & np.uint64(1)) << np.uint64(2 * b)
        m |= ((d[:, 1] >> np.uint64(b)) & np.uint64(1)) << np.uint64(2 * b + 1)
    return m


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1000, 1023, 1024, 1025, 2047, 2048, 2049])
@pytest.mark.parametrize("kind", ["square", "repeated", "far", "targets"])
def test_same_as_general_path(n, kind):
    import torch

    import paper_1105_3505_amd as lf
    rng = np.random.default_rng(n)
    if kind == "far":       # root boxes of up to 2^31 cells
        xy = np.concatenate([rng.integers(0, 40, size=(n, 2)) - 20, [[-(1 << 30), 5], [(1 << 30) - 1, 9]]])[-n:]
    else:
        w = int((10 * n) ** 0.5) + 1
        xy = rng.integers(0, w, size=(n, 2)) - 7
    if kind == "repeated":
        xy = xy[rng.integers(0, n, size=n)]
    xy = np.ascontiguousarray(xy.astype(np.int32))
    tgt = np.ascontiguousarray(xy[: n // 2]) if kind == "targets" and n > 1 else None
    src = xy[n // 2:] if tgt is not None else xy
    src = np.ascontiguousarray(src)
    f = torch.from_numpy(rng.standard_normal(len(src))).cuda()
    other = torch.tensor([[3, 4], [5, 5]], dtype=torch.int32, device="cuda")
    ctx = lf.Context(0)
    dev, t = torch.from_numpy(src).cuda(), None if tgt is None else torch.from_numpy(tgt).cuda()
    one = ctx.plan(dev, targets=t)
    both = ctx.plan_batch([dev, other], targets=[t, None])
    pts = src if tgt is None else np.concatenate([src, tgt])
    assert np.array_equal(one.export("perm"), np.argsort(_morton(pts), kind="stable"))
    assert one.info()["leaf_level"] == both.info()["leaf_level"] or kind == "far"
    u = one.execute(f).cpu().numpy()
    v = both.execute_instances([f, torch.ones(2, dtype=torch.float64, device="cuda")])[0].cpu().numpy()
    ctx.close()
    assert np.array_equal(u, v)
