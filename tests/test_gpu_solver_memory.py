"""Solver objects hold no vectors between solves: after one solve has made the context's cached blocks,
solves of other objects of the same size take no more memory, and a solve whose vectors are above the
size that is cached leaves none of them.  Solves with other restarts, on other objects' leftovers, give
the bits of the same solves in a context of their own."""
from contextlib import closing

import numpy as np
import pytest

from test_gpu_gmres import snake

pytestmark = pytest.mark.gpu


def _used():
    import torch
    torch.cuda.synchronize()
    free, total = torch.cuda.mem_get_info()
    return total - free


def _delta(n, seed):
    return np.random.default_rng(seed).uniform(-0.5, 0.5, n - 1)


@pytest.mark.parametrize("n,restart", [(20000, 200), (50000, 400)])   # 34 MB; 165 MB: not cached
def test_memory_between_solves(n, restart):
    import torch
    import paper_1105_3505_amd as lf
    with closing(lf.Context(0)) as ctx:
        objs = [lf.Inclusions(ctx, snake(n, 250), _delta(n, k)) for k in range(4)]
        mu = torch.empty(n, dtype=torch.float64, device="cuda")
        for o in objs:                  # each plan's first execute may make a stream, and the runtime its queue
            o.solve(0.8, -0.45, mu, tol=0.5, restart=1)
        start = _used()
        objs[0].solve(0.8, -0.45, mu, tol=1e-10, restart=restart)
        first = _used()
        for o in objs[1:]:
            o.solve(0.8, -0.45, mu, tol=1e-10, restart=restart)
        print("first solve %.1f MB, then %.1f MB" % ((first - start) / 1e6, (_used() - first) / 1e6))
        assert _used() - first < 16 << 20
        if n == 50000:
            assert first - start < 64 << 20
        for o in objs:
            o.close()


def test_shared_blocks_same_bits():
    import paper_1105_3505_amd as lf
    jobs = [(1030, 7), (3000, 40), (1030, 150), (513, 7), (3000, 5)]   # nodes, restart
    alone = []
    for n, restart in jobs:
        with closing(lf.Context(0)) as ctx:
            inc = lf.Inclusions(ctx, snake(n, 40), _delta(n, n))
            mu, st = inc.solve(0.8, -0.45, tol=1e-11, restart=restart)
            alone.append((mu.cpu().numpy(), st))
            inc.close()
    with closing(lf.Context(0)) as ctx:
        objs = {n: lf.Inclusions(ctx, snake(n, 40), _delta(n, n)) for n, _ in jobs}
        for (n, restart), (ref, ref_st) in zip(jobs, alone):
            mu, st = objs[n].solve(0.8, -0.45, tol=1e-11, restart=restart)
            assert st == ref_st and np.array_equal(mu.cpu().numpy(), ref)
        for o in objs.values():
            o.close()
