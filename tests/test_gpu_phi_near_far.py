"""phi over all offsets of the near field's kernels.

Leaves of side 128 beside each other: offsets up to 255 in both coordinates, so that the squared distance
runs through every octave of the table by octaves, 2^11 to 2^17, with both sides of each power of two, of
ends of the table's intervals within the octaves and of the radius below which a table is read.  Leaves
of the adaptive tree of sides 16 to 256: chunks of sources that are all inside the tables' reach, on its
edge, and beyond.

A unit load in a tree without a far field (leaf level 1, or adaptive boxes of at most as many points as a
skeleton has) gives u = phi(offset); compared with the host's phi (quadrature table, expansion beyond
radius 128) to 4e-15 absolute: the rounding of a handful of operations on values of order one and the
4e-15 that the two expansions may differ by.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = 4e-15


def _on_circles(r2s, top):
    """Lattice points on both sides of the circles of squared radii r2s, coordinates 0 .. top."""
    out = []
    for r2 in r2s:
        for x in range(0, top + 1, 5):
            y = int(np.sqrt(max(r2 - x * x, 0)))
            out += [(x, y + d) for d in (-1, 0, 1, 2) if 0 <= y + d <= top and r2 >= x * x]
    return out


@pytest.mark.parametrize("stencil", [5, 9])
def test_side_128_every_octave(stencil):
    import torch

    import paper_1105_3505_amd as lf
    rng = np.random.default_rng(255)
    edge = (0, 1, 2, 33, 47, 48, 49, 63, 64, 127, 128, 181, 191, 254, 255)
    off = [(x, y) for x in edge for y in edge] + [tuple(v) for v in rng.integers(0, 256, size=(1200, 2))]
    off += _on_circles([48 * 48] + [1 << k for k in range(11, 17)], 255)
    # ends of intervals (256 an octave): each octave's first, middle and last
    off += _on_circles([(1 << k) + ((1 << k) * i) // 256 for k in range(11, 17) for i in (1, 128, 255)], 255)
    off = np.array(sorted(set(off) - {(0, 0)}), dtype=np.int32)
    r2 = (off.astype(np.int64) ** 2).sum(1)
    for k in range(11, 17):
        assert np.any((r2 >= (1 << k)) & (r2 < (1 << k) * 1.01)) and np.any((r2 < (2 << k)) & (r2 > (2 << k) * 0.99)), k
    ctx = lf.Context(0, stencil=stencil, max_leaf=4096)
    one = torch.ones(1, dtype=torch.float64, device="cuda")
    for sx, sy in ((1, 1), (-1, 1), (1, -1), (-1, -1)):
        tgt = np.ascontiguousarray(off * np.array([sx, sy], dtype=np.int32))
        plan = ctx.plan(torch.zeros((1, 2), dtype=torch.int32, device="cuda"), targets=torch.from_numpy(tgt).cuda())
        info = plan.info()
        assert (info["leaf_level"], info["leaf_side"]) == (1, 128)
        u = plan.execute(one).cpu().numpy()
        plan.close()
        assert np.max(np.abs(u - lf.host_phi(tgt, stencil=stencil))) <= TOL
    ctx.close()


# side of the finer leaves; the coarser ones have twice that
@pytest.mark.parametrize("side", [8, 16, 32, 64, 128])
@pytest.mark.parametrize("stencil", [5, 9])
def test_adaptive_chunks_about_the_tables(side, stencil):
    import torch

    import paper_1105_3505_amd as lf
    rng = np.random.default_rng(side)
    ctx = lf.Context(0, adaptive=True, stencil=stencil, max_leaf=20)
    s = 2 * side
    for which in range(4):                       # the quadrant that is refined
        pts = []
        for q in range(4):
            corner = np.array([q & 1, q >> 1]) * s
            if q != which:
                p = np.unique(rng.integers(0, s, size=(16, 2)), axis=0)
                pts.append(corner + np.concatenate([p, [[0, 0], [0, s - 1], [s - 1, 0], [s - 1, s - 1]]]))
                continue
            for c in range(4):
                p = np.unique(rng.integers(0, side, size=(8, 2)), axis=0)
                p = np.concatenate([p, [[0, 0], [0, side - 1], [side - 1, 0], [side - 1, side - 1]]])
                pts.append(corner + np.array([c & 1, c >> 1]) * side + p)
        xy = np.ascontiguousarray(np.unique(np.concatenate(pts), axis=0).astype(np.int32))
        plan = ctx.plan(torch.from_numpy(xy).cuda())
        info = plan.info()
        assert info["adaptive"] == 1 and info["n_leaves"] == 7
        assert info["m2l_pairs"] == 0 and info["m2p_terms"] == 0 and info["p2l_terms"] == 0
        for k in rng.choice(len(xy), size=16, replace=False):
            f = torch.zeros(len(xy), dtype=torch.float64, device="cuda")
            f[int(k)] = 1.0
            u = plan.execute(f).cpu().numpy()
            assert np.max(np.abs(u - lf.host_phi(xy - xy[k], stencil=stencil))) <= TOL
        plan.close()
    ctx.close()


def test_adaptive_instances_of_wide_and_small_leaves():
    """An adaptive instance of wide leaves alone (phi computed) gives the same bits beside one of small leaves, whose
    plan has the tables as well; so does the latter."""
    import torch

    import paper_1105_3505_amd as lf
    rng = np.random.default_rng(5)
    wide = np.unique(np.rint(2000.0 * rng.standard_normal((4000, 2))).astype(np.int32), axis=0)
    small = np.unique(rng.integers(0, 120, size=(3000, 2)).astype(np.int32), axis=0)
    ctx = lf.Context(0, adaptive=True, max_leaf=32)
    sets = [np.ascontiguousarray(p) for p in (wide, small)]
    dev = [torch.from_numpy(p).cuda() for p in sets]
    fs = [torch.from_numpy(rng.standard_normal(len(p))).cuda() for p in sets]
    alone, sides = [], []
    for x, f in zip(dev, fs):
        plan = ctx.plan(x)
        sides.append(plan.info()["leaf_side"])
        alone.append(plan.execute(f))
        plan.close()
    assert sides[0] > 64 >= sides[1]
    plan = ctx.plan_batch(dev)
    us = plan.execute_instances(fs)
    for a, b in zip(alone, us):
        assert torch.equal(a, b)
    plan.close()
    ctx.close()
