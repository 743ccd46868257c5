"""Solves that end in an error: a device block refused inside an iteration (LFMM_TEST_FAIL_ALLOC=k fails
the k-th block requested; on a context that checks loads every execute requests one) surfaces as
LFMM_E_NOMEM, leaves none of the solve's memory behind, and the object's next solve, on another stream,
gives the bits of an object that never failed."""
import os
from contextlib import closing

import numpy as np
import pytest

import workloads as wl
from test_gpu_gmres import snake

pytestmark = pytest.mark.gpu

NOMEM = -3
N = 72000                              # with a restart of 512 a basis of 297 MB
OPTS = {"tol": 1e-10, "restart": 512}


def _objects(kind, ctx):
    """A solver object and its solve on a stream."""
    import torch
    import paper_1105_3505_amd as lf
    rng = np.random.default_rng(9)
    if kind == "inclusions":
        obj = lf.Inclusions(ctx, snake(N, 300), rng.uniform(-0.5, 0.5, N - 1))
        return obj, lambda stream: obj.solve(0.8, -0.45, stream=stream, **OPTS)
    gamma, codes, _ = wl.box_boundary(N // 4, N // 4)
    obj = lf.Dirichlet(ctx, gamma, codes)
    g = torch.from_numpy(np.cos(1e-3 * gamma[:, 0]) + 1e-4 * gamma[:, 1]).cuda()
    return obj, lambda stream: obj.solve(g, stream=stream, **OPTS)


@pytest.mark.parametrize("kind", ["inclusions", "dirichlet"])
def test_failure_inside_a_solve(kind):
    import torch
    import paper_1105_3505_amd as lf
    with closing(lf.Context(0)) as ctx:
        obj, solve = _objects(kind, ctx)
        ref, ref_st = solve(None)
        ref = ref.cpu().numpy()
        obj.close()
    with closing(lf.Context(0, check_loads=True)) as ctx:
        obj, solve = _objects(kind, ctx)
        side = torch.cuda.Stream()
        torch.cuda.synchronize()
        for k in (2, 4, 7):
            free = torch.cuda.mem_get_info()[0]
            os.environ["LFMM_TEST_FAIL_ALLOC"] = str(k)
            try:
                with pytest.raises(lf.LfmmError) as e:
                    solve(None)
            finally:
                del os.environ["LFMM_TEST_FAIL_ALLOC"]
            assert e.value.status == NOMEM
            left = free - torch.cuda.mem_get_info()[0]
            print(kind, k, "left behind %.1f MB" % (left / 1e6), flush=True)
            assert left < 64 << 20
            x, st = solve(side)
            side.synchronize()
            assert st == ref_st
            assert np.array_equal(x.cpu().numpy(), ref)
        obj.close()
