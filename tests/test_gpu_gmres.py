"""The solvers' Gram-Schmidt steps at the edges of their slices: vectors of a tile (512 elements) less
or more one, of more tiles than blocks, and more than 64 basis vectors.

The inclusions are a snake of bars of random conductances, whose reduced system (eq. 10.4) is far
worse conditioned than scattered bars.  Tolerance: a relative residual r of A mu = b bounds the error of
mu by cond(A) r; r is the solver's tolerance 1e-10 and the FMM's relative error, at most 1e-12, times
|A| |mu| / |b| <= cond(A).  Without a restart the iteration count is that of a dense GMRES, up to one
at either end of the tolerance's step.
"""
from contextlib import closing

import numpy as np
import pytest
from scipy.sparse.linalg import gmres

from oracle import extensions as ox

pytestmark = pytest.mark.gpu

RES = 1e-10


def snake(n, row):
    """n nodes in rows of `row`, alternating in direction, and the n - 1 bars that join them."""
    i = np.arange(n)
    x, y = i % row, i // row
    x = np.where(y % 2 == 1, row - 1 - x, x)
    p = np.stack([x, y], 1).astype(np.int32)
    return np.concatenate([p[:-1], p[1:]], 1)


@pytest.mark.parametrize("n,restart", [(33, 33), (511, 200), (512, 17), (513, 200), (1030, 150)])
def test_inclusions_dense(n, restart):
    import paper_1105_3505_amd as lf
    bars = snake(n, 23)
    delta = 10.0 ** np.random.default_rng(n).uniform(-1.0, 3.0, n - 1)
    nodes, mu_ref = ox.inclusions_solve(bars, delta, 0.8, -0.45)
    _, ends = ox.inclusion_nodes(bars)
    B, S = ox.b_matrix(n, ends, delta), ox._phi_matrix(nodes, nodes)
    A = np.eye(n) + B @ S
    cond = np.linalg.cond(A)
    with closing(lf.Context(0)) as ctx:
        inc = lf.Inclusions(ctx, bars, delta)
        mu, st = inc.solve(0.8, -0.45, tol=RES, restart=restart, max_iter=2000)
        inc.close()
    print(n, st, "cond %.3g" % cond)
    assert st["converged"] == 1
    steps = []
    if restart >= 130:
        gmres(A, -(B @ (S @ (B @ (nodes @ np.array([0.8, -0.45]))))), rtol=RES, restart=restart, maxiter=1,
              callback=steps.append, callback_type="pr_norm")
        assert 64 < len(steps) and abs(st["iterations"] - len(steps)) <= 1
    err = np.linalg.norm(mu.cpu().numpy() - mu_ref) / np.linalg.norm(mu_ref)
    assert err <= cond * (RES + 1e-12 * cond)


def test_inclusions_more_tiles_than_blocks():
    import torch
    import paper_1105_3505_amd as lf
    n = 140003   # 274 tiles: two to a block, the last block's slice is short
    bars = snake(n, 400)
    delta = np.random.default_rng(5).uniform(-0.5, 0.5, n - 1)
    with closing(lf.Context(0)) as ctx:
        inc = lf.Inclusions(ctx, bars, delta)
        mu, st = inc.solve(0.8, -0.45, tol=RES)
        plan = ctx.plan(torch.from_numpy(inc.nodes).cuda())
        node = {(int(a), int(b)): i for i, (a, b) in enumerate(inc.nodes)}
        a = np.array([node[(int(r[0]), int(r[1]))] for r in bars])
        b = np.array([node[(int(r[2]), int(r[3]))] for r in bars])

        def B(s):
            out, d = np.zeros(n), delta * (s[a] - s[b])
            np.add.at(out, a, d)
            np.add.at(out, b, -d)
            return out

        def S(f):
            return plan.execute(torch.from_numpy(f).cuda()).cpu().numpy()

        m = mu.cpu().numpy()
        rhs = -B(S(B(inc.nodes @ np.array([0.8, -0.45]))))
        res = np.linalg.norm(rhs - m - B(S(m))) / np.linalg.norm(rhs)
        inc.close()
    print(st, "residual %.3e" % res)
    # the same sums in another order: equal to rounding
    assert st["converged"] == 1 and res <= RES * (1.0 + 1e-4) + 1e-14
