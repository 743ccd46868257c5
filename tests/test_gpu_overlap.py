"""The near field beside the far field's passes (plans of 128 to 16,384 leaves): the same bits as in turn (which the
timing of phases asks for), on the caller's streams, with plans that come and go, and several at once."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _points(n, density, seed):
    rng = np.random.default_rng(seed)
    w = int((n / density) ** 0.5)
    c = rng.choice(w * w, size=n, replace=False)
    return np.stack([c // w, c % w], 1).astype(np.int32)


# leaf sides 8, 16 and 32; leaf counts at both ends of the rule and between
@pytest.mark.parametrize("n,density", [(4000, 0.4), (9000, 0.1), (60000, 0.1), (3300, 0.025), (30000, 0.025),
                                       (150000, 0.025)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_same_bits_as_in_turn(n, density, precision):
    import torch

    import paper_1105_3505_amd as lf
    ctx = lf.Context(0, precision=precision)
    src = torch.from_numpy(_points(n, density, n)).cuda()
    tgt = torch.from_numpy(_points(n // 3, density, n + 1)).cuda()
    f = torch.randn(n, dtype=torch.float64, device="cuda")
    for targets in (None, tgt):
        plan = ctx.plan(src, targets=targets)
        a = plan.execute(f)
        plan.set_timing(True)
        b = plan.execute(f)
        plan.set_timing(False)
        c = plan.execute(f)
        assert torch.equal(a, b) and torch.equal(a, c)
    ctx.close()


def test_streams_and_plans():
    import torch

    import paper_1105_3505_amd as lf
    ctx = lf.Context(0)
    xy = [torch.from_numpy(_points(20000 + 700 * k, 0.03, k)).cuda() for k in range(12)]
    f = [torch.randn(len(p), dtype=torch.float64, device="cuda") for p in xy]
    want = []
    for p, q in zip(xy, f):
        plan = ctx.plan(p)
        plan.set_timing(True)
        want.append(plan.execute(q).clone())
        plan.close()
    streams = [torch.cuda.Stream() for _ in range(3)]
    torch.cuda.synchronize()
    held = []   # more plans alive than there are side streams
    for rep in range(3):
        got = []
        for k in range(12):
            with torch.cuda.stream(streams[k % 3]):
                plan = ctx.plan(xy[k])
                u = plan.execute(f[k])
                u2 = plan.execute(u * 0 + f[k])
                got.append((k, u, u2))
            if k % 2:
                plan.close()   # with its work still in flight: its memory goes to the plans after it
            else:
                held.append(plan)
        torch.cuda.synchronize()
        for k, u, u2 in got:
            assert torch.equal(u, want[k]) and torch.equal(u2, want[k])
    ctx.close()
