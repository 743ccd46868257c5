"""The work a program has this framework do: the cases its speed is measured on.

Every case evaluates the lattice convolution (eq. 1.7) through the package's public entry points:
one-shot solves (plan, execute, release), executes of a resident plan, forests of independent
point sets, the continuous-batching server and the two iterative applications of Section 10.
All inputs are synthetic and made on the GPU from the seed.

    listed()              the cases, plain dicts
    draw(rng)             one more case of the same ranges
    prepare(case, seed)   inputs and the plan or handle a program keeps
    run(state)            one pass and its outputs
    work(case)            bytes and operations one pass cannot do without
    exact(case, seed)     the same outputs from plain 64-bit numpy / torch arithmetic
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_1105_3505_amd as lf

DEV = "cuda"
RANK = 48        # coefficients of a skeleton expansion
LEAF = 16        # points a leaf holds on average in uniform point sets (N_leaf = 64)


# ---- cases ------------------------------------------------------------------------------------

def _points(name, mode, n, side, **more):
    """A point-set case.  mode: "solve" (Context.solve), "plan" (plan, execute, release),
    "execute" (a resident plan's execute) or "sorted" (the same in plan order).  clusters: 0 for
    distinct cells uniform in a side x side box, else the number of Gaussian clusters of deviation
    sigma.  n_tgt: separate targets in the same box (0: the targets are the sources)."""
    case = {"name": name, "kind": "points", "mode": mode, "n": n, "side": side, "clusters": 0, "sigma": 0.0,
            "n_tgt": 0, "precision": "fp64", "stencil": 5, "adaptive": False, "max_leaf": 64, "graph": False}
    case.update(more)
    return case


def listed():
    return [
        # the smallest calls: a thousand points solved once, and a resident plan's execute
        # (one load vector after another on a fixed small lattice patch)
        _points("solve 1e3", "solve", 1000, 256),
        _points("execute 1e3", "execute", 1000, 256),
        # an ordinary ragged problem: potentials at targets of their own, the isotropic 9-point
        # operator, FP32 mixed precision
        _points("targets 6e4 mixed", "plan", 60013, 981, n_tgt=25031, precision="mixed", stencil=9),
        # the headline workload: one million points, each solve with new points (plan built,
        # executed, released), in FP64 and in the fast mixed precision
        _points("solve 1e6", "plan", 1000000, 4096),
        _points("solve 1e6 bf16", "plan", 1000000, 4096, precision="mixed-bf16"),
        # the same points kept: what an iterative method pays per application
        _points("execute 1e6", "execute", 1000000, 4096),
        # strongly non-uniform points, on the uniform-depth tree and on the adaptive one
        _points("clusters 2e6", "plan", 2000000, 1 << 20, clusters=64, sigma=2000.0),
        _points("clusters 2e6 adaptive", "plan", 2000000, 1 << 20, clusters=64, sigma=2000.0, adaptive=True,
                max_leaf=32),
        # 512 independent problems of mixed sizes in one forest
        {"name": "forest 512", "kind": "forest", "count": 512, "lo": 1000, "hi": 100000, "sizes": 4,
         "precision": "fp64"},
        # the server, kept busy: requests of sizes over four decades, uniform or clustered
        {"name": "serving 48", "kind": "serving", "count": 48, "lo": 100, "hi": 1000000, "sizes": 5},
        # Section 10.1: 50,000 modified bars, GMRES and the potential at sample points
        {"name": "inclusions 5e4", "kind": "inclusions", "bars": 50000, "side": 2000, "n_tgt": 20000},
        # Section 10.2: the boundary of a 16384 x 16384 box, GMRES
        {"name": "dirichlet 16384", "kind": "dirichlet", "n1": 16384, "n2": 16384},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["points", "points", "points", "clusters", "clusters", "forest", "serving", "inclusions",
                       "dirichlet"])
    if kind == "points":
        # a box of one occupied cell in 4 to 64, as the uniform workloads have
        n = _log_int(rng, 500, 1000000)
        side = int(math.ceil(math.sqrt(n * math.exp(rng.uniform(math.log(4.0), math.log(64.0))))))
        mode = rng.choice(["solve", "plan", "plan", "execute", "execute", "sorted"])
        case = _points("", mode, n, side, precision=rng.choice(["fp64", "fp64", "mixed-bf16", "mixed"]),
                       stencil=rng.choice([5, 5, 5, 9]))
        if mode in ("plan", "execute") and rng.random() < 0.3:
            case["n_tgt"] = _log_int(rng, max(n // 16, 1), n)
            case["n"] = n - n // 3
        if mode in ("execute", "sorted"):
            case["graph"] = rng.random() < 0.25
    elif kind == "clusters":
        n = _log_int(rng, 20000, 2000000)
        adaptive = rng.random() < 0.5
        case = _points("", rng.choice(["plan", "execute"]), n, 1 << rng.randint(17, 20), clusters=rng.randint(3, 64),
                       sigma=round(math.exp(rng.uniform(math.log(800.0), math.log(2500.0))), 1), adaptive=adaptive,
                       max_leaf=32 if adaptive else 64, precision=rng.choice(["fp64", "fp64", "mixed-bf16"]))
    elif kind == "forest":
        case = {"kind": "forest", "count": _log_int(rng, 8, 512), "lo": 1000, "hi": 100000,
                "sizes": rng.randrange(1 << 20), "precision": rng.choice(["fp64", "fp64", "mixed-bf16"])}
    elif kind == "serving":
        case = {"kind": "serving", "count": rng.randint(4, 48), "lo": 100, "hi": _log_int(rng, 10000, 1000000),
                "sizes": rng.randrange(1 << 20)}
    elif kind == "inclusions":
        bars = _log_int(rng, 500, 50000)
        case = {"kind": "inclusions", "bars": bars, "side": int(math.ceil(math.sqrt(bars * rng.uniform(40.0, 120.0)))),
                "n_tgt": _log_int(rng, 100, 20000)}
    else:
        n1 = _log_int(rng, 200, 16384)
        case = {"kind": "dirichlet", "n1": n1, "n2": max(100, min(16384, int(n1 * rng.uniform(0.4, 1.0))))}
    case.pop("name", None)
    return case


# ---- inputs -----------------------------------------------------------------------------------

def _generator(seed, salt=0):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + int(salt)) % (1 << 62))
    return g


def _uniform(g, n, side):
    """n distinct cells of a side x side box, uniform, as int32 [n, 2]."""
    total = side * side
    if total <= 64 * n and total <= 1 << 26:
        cells = torch.randperm(total, generator=g, device=DEV)[:n]
    else:
        cells = torch.randint(0, total, (n + n // 8 + 64,), generator=g, device=DEV)
        cells = torch.unique(cells)
        cells = cells[torch.randperm(len(cells), generator=g, device=DEV)[:n]]
    return torch.stack([cells % side, cells // side], dim=1).to(torch.int32).contiguous()


def _clusters(g, n, side, count, sigma):
    """n distinct points in `count` Gaussian clusters inside a side x side box."""
    margin = min(3.0 * sigma, side / 4.0)
    centres = margin + (side - 2.0 * margin) * torch.rand(count, 2, generator=g, device=DEV, dtype=torch.float64)
    cells = torch.empty(0, dtype=torch.int64, device=DEV)
    while len(cells) < n:
        m = (n - len(cells)) * 5 // 4 + 64
        which = torch.randint(0, count, (m,), generator=g, device=DEV)
        p = centres[which] + sigma * torch.randn(m, 2, generator=g, device=DEV, dtype=torch.float64)
        p = p.round().to(torch.int64).clamp_(0, side - 1)
        cells = torch.unique(torch.cat([cells, p[:, 0] * side + p[:, 1]]))
    cells = cells[torch.randperm(len(cells), generator=g, device=DEV)[:n]]
    return torch.stack([cells // side, cells % side], dim=1).to(torch.int32).contiguous()


def _loads(g, n):
    """N(0, 1) loads, mean-subtracted and rounded to multiples of 2^-32 so that they sum to
    exactly zero (the well-posedness condition)."""
    x = torch.randn(n, generator=g, device=DEV, dtype=torch.float64)
    k = ((x - x.mean()) * 2.0 ** 32).round().to(torch.int64)
    k[-1] = -k[:-1].sum()
    return k.to(torch.float64) * 2.0 ** -32


def _point_inputs(case, seed):
    g = _generator(seed)
    if case["clusters"]:
        xy = _clusters(g, case["n"], case["side"], case["clusters"], case["sigma"])
    else:
        xy = _uniform(g, case["n"], case["side"])
    tgt = _uniform(g, case["n_tgt"], case["side"]) if case["n_tgt"] else None
    return xy, tgt, _loads(g, case["n"])


def _sizes(case):
    """Sizes of a forest's or a server's point sets, log-uniform, and whether each is clustered."""
    rng = np.random.default_rng(case["sizes"])
    n = np.rint(np.exp(rng.uniform(math.log(case["lo"]), math.log(case["hi"]), case["count"]))).astype(int)
    clustered = rng.uniform(size=case["count"]) < 0.5
    return [max(int(v), 2) for v in n], [bool(c) for c in clustered]


def _many_inputs(case, seed):
    """(xy, f, side of the box) of every point set: uniform in a box of side 4 sqrt n, or for the
    server's clustered requests 8 clusters of deviation sqrt n in a box of side 16 sqrt n."""
    out = []
    for i, (n, clustered) in enumerate(zip(*_sizes(case))):
        g = _generator(seed, i + 1)
        if case["kind"] == "serving" and clustered:
            side = int(math.ceil(16.0 * math.sqrt(n)))
            xy = _clusters(g, n, side, 8, math.sqrt(n))
        else:
            side = int(math.ceil(4.0 * math.sqrt(n)))
            xy = _uniform(g, n, side)
        out.append((xy, _loads(g, n), side))
    return out


def _bars(case, seed):
    """Bar modifications at disjoint places of a side x side box: lattice bars removed, weakened or
    strengthened, diagonal bars added.  Host arrays."""
    rng = np.random.default_rng(seed)
    want, side = case["bars"], case["side"]
    m = 2 * want + 64
    a = rng.integers(0, side, size=(m, 2))
    added = rng.uniform(size=m) < 0.15
    flip = (rng.uniform(size=m) < 0.5)[:, None]
    b = a + np.where(added[:, None], np.where(flip, [1, 1], [1, -1]), np.where(flip, [1, 0], [0, 1]))
    _, inverse, uses = np.unique(np.concatenate([a, b]) @ np.array([4 * side, 1]), return_inverse=True,
                                 return_counts=True)
    keep = np.flatnonzero((uses[inverse] == 1).reshape(2, -1).all(axis=0))[:want]
    a, b, added = a[keep], b[keep], added[keep]
    kind = rng.uniform(size=want)
    delta = np.where(kind < 0.18, -1.0, np.where(kind < 0.6, rng.uniform(-0.9, -0.05, want), rng.uniform(0.05, 3.0, want)))
    delta = np.where(added, rng.uniform(0.1, 2.0, want), delta)
    return np.concatenate([a, b], axis=1).astype(np.int32), delta


FIELD = (1.0, 0.5)   # v = m1 + 0.5 m2 at infinity


def _bar_targets(case, seed):
    return _uniform(_generator(seed, 7), case["n_tgt"], 2 * case["side"])


def _boundary(case):
    """Boundary nodes of the box [0, n1] x [0, n2] without its corners, and outward normal codes."""
    n1, n2 = case["n1"], case["n2"]
    t1, t2 = np.arange(1, n1), np.arange(1, n2)
    g = [np.stack([0 * t2, t2], 1), np.stack([0 * t2 + n1, t2], 1), np.stack([t1, 0 * t1], 1),
         np.stack([t1, 0 * t1 + n2], 1)]
    codes = np.concatenate([np.full(len(t2), 1), np.full(len(t2), 0), np.full(len(t1), 3), np.full(len(t1), 2)])
    return np.concatenate(g).astype(np.int32), codes.astype(np.int8)


def _boundary_values(case, seed):
    """A smooth potential on the boundary plus a little noise."""
    gamma, _ = _boundary(case)
    x = torch.from_numpy(gamma).to(DEV).to(torch.float64) / max(case["n1"], case["n2"])
    g = _generator(seed)
    w = 2.0 * math.pi * torch.rand(4, generator=g, device=DEV, dtype=torch.float64)
    noise = 0.01 * torch.randn(len(x), generator=g, device=DEV, dtype=torch.float64)
    return torch.sin(w[0] + 3.0 * x[:, 0] + w[1] * x[:, 1]) + torch.cos(w[2] + w[3] * x[:, 1]) + noise


# ---- passes -----------------------------------------------------------------------------------

@functools.lru_cache(maxsize=None)
def _context(precision="fp64", stencil=5, adaptive=False, max_leaf=64, graph=False):
    """The contexts a program keeps: one for each set of options."""
    return lf.Context(0, precision=precision, stencil=stencil, adaptive=adaptive, max_leaf=max_leaf, graph=graph)


@functools.lru_cache(maxsize=None)
def _server():
    """The one server of the program, on a context of its own (a server owns its context)."""
    return lf.Server(lf.Context(0))


def prepare(case, seed):
    kind = case["kind"]
    if kind == "points":
        ctx = _context(case["precision"], case["stencil"], case["adaptive"], case["max_leaf"], case["graph"])
        xy, tgt, f = _point_inputs(case, seed)
        s = {"mode": case["mode"], "ctx": ctx, "xy": xy, "tgt": tgt, "f": f}
        if case["mode"] in ("execute", "sorted"):
            s["plan"] = ctx.plan(xy, targets=tgt)
            if case["mode"] == "sorted":
                perm = torch.from_numpy(s["plan"].export("perm")).to(DEV)
                s["f"] = f[perm.long()].contiguous()
        return s
    if kind == "forest":
        sets = _many_inputs(case, seed)
        off = np.cumsum([0] + [len(f) for _, f, _ in sets])
        u = torch.empty(int(off[-1]), dtype=torch.float64, device=DEV)
        return {"mode": "forest", "ctx": _context(case["precision"]), "xys": [xy for xy, _, _ in sets],
                "fs": [f for _, f, _ in sets], "u": u, "us": [u[a:b] for a, b in zip(off.tolist(), off[1:].tolist())]}
    if kind == "serving":
        return {"mode": "serving", "server": _server(), "sets": [(xy, f) for xy, f, _ in _many_inputs(case, seed)]}
    if kind == "inclusions":
        bars, delta = _bars(case, seed)
        return {"mode": "inclusions", "inc": lf.Inclusions(_context(), bars, delta), "tgt": _bar_targets(case, seed)}
    gamma, codes = _boundary(case)
    return {"mode": "dirichlet", "dir": lf.Dirichlet(_context(), gamma, codes), "g": _boundary_values(case, seed)}


def run(state):
    s, mode = state, state["mode"]
    if mode == "solve":
        return s["ctx"].solve(s["xy"], s["f"])
    if mode == "plan":
        plan = s["ctx"].plan(s["xy"], targets=s["tgt"])
        u = plan.execute(s["f"])
        plan.close()
        return u
    if mode == "execute":
        return s["plan"].execute(s["f"])
    if mode == "sorted":
        return s["plan"].execute_sorted(s["f"])
    if mode == "forest":
        plan = s["ctx"].plan_batch(s["xys"])
        plan.execute_instances(s["fs"], s["us"])
        plan.close()
        return s["u"]
    if mode == "serving":
        tickets = [s["server"].submit(xy, f) for xy, f in s["sets"]]
        return [s["server"].wait(t)[0] for t in tickets]
    if mode == "inclusions":
        mu, _ = s["inc"].solve(*FIELD)
        return [mu, s["inc"].potential(*FIELD, mu, s["tgt"])]
    q, _ = s["dir"].solve(s["g"])
    return q


def work(case):
    """Bytes: points and loads in, potentials out, each once.  Operations: the fast method's on
    leaves of LEAF points: near field (9 leaves of sources, one multiply-add each), the outgoing
    and incoming leaf operators, and per box (4/3 boxes per leaf) 27 interactions and two
    translations of RANK x RANK multiply-adds.  Iterative cases: ten applications."""
    kind = case["kind"]
    if kind == "points":
        n, m, times = case["n"] + case["n_tgt"], case["n_tgt"] or case["n"], 1
        moved = 8 * n + 8 * case["n"] + 8 * m if case["mode"] not in ("execute", "sorted") else 8 * case["n"] + 8 * m
    elif kind in ("forest", "serving"):
        n, times = sum(_sizes(case)[0]), 1
        moved = 24 * n
    elif kind == "inclusions":
        n, times = 2 * case["bars"], 10
        moved = 24 * case["bars"] + 8 * n + 16 * case["n_tgt"]
    else:
        n, times = 6 * (case["n1"] + case["n2"]), 10
        moved = 16 * (case["n1"] + case["n2"]) * 2
    per_point = 2 * 9 * LEAF + 4 * RANK
    per_box = (27 + 2) * 2 * RANK * RANK
    return {"bytes": moved, "flops": times * (n * per_point + n * 4 // (3 * LEAF) * per_box)}


# ---- the same in plain 64-bit arithmetic ----------------------------------------------------------

NEAR = 128   # |m| up to which phi comes from its integral; beyond, from its expansion


@functools.lru_cache(maxsize=None)
def _phi_table(stencil):
    """phi at 0 <= n <= m <= NEAR by Gauss-Legendre quadrature of the reduced integral
    phi(m, n) = 1/pi int_0^pi (rho^m cos(n t) - 1) / sqrt(A^2 - B^2) dt for the symbol
    A(t) - B(t) cos t1, rho = (A - sqrt(A^2 - B^2)) / B, and the coefficients of its expansion
    -(1/2pi) log r + sum_k r^-2k sum_j c cos(4 j theta), fitted to the outer part of the table."""
    x, w = np.polynomial.legendre.leggauss(64)             # on [0, pi/256] and its doublings up to pi
    edge = np.concatenate([[0.0], math.pi * 2.0 ** np.arange(-8, 1)])
    width = 0.5 * np.diff(edge)[:, None]
    t, w = (edge[:-1, None] + width * (x + 1.0)).ravel(), (width * w).ravel()
    half = 2.0 * np.sin(0.5 * t) ** 2                      # 1 - cos t
    if stencil == 5:
        a, b, gap = 2.0 + 2.0 * half, np.full_like(t, 2.0), 2.0 * half
    else:
        a, b, gap = 2.0 + 4.0 * half / 3.0, 2.0 - 2.0 * half / 3.0, 2.0 * half
    root = np.sqrt(gap * (a + b))                          # A - B = gap without cancellation
    log_rho = np.log1p(-(root - gap) / b)
    m = np.arange(NEAR + 1)
    decay = np.exp(m[:, None] * log_rho[None, :])
    half_cos = -2.0 * np.sin(0.5 * m[:, None] * t[None, :]) ** 2   # cos(n t) - 1
    weight = w / (math.pi * root)
    table = (decay * weight) @ half_cos.T + (np.expm1(m[:, None] * log_rho[None, :]) @ weight)[:, None]
    mm, nn = np.meshgrid(m, m, indexing="ij")
    pick = (nn <= mm) & (mm >= 40)
    basis = _far_terms(mm[pick].astype(float), nn[pick].astype(float))
    rhs = table[pick] + np.log(np.hypot(mm[pick], nn[pick])) / (2.0 * math.pi)
    scale = np.abs(basis).max(axis=0)
    coef = np.linalg.lstsq(basis / scale, rhs, rcond=None)[0] / scale
    return torch.from_numpy(table).to(DEV), torch.from_numpy(coef).to(DEV)


def _far_terms(x, y):
    """Columns 1, r^-2 {1, c4}, r^-4 {1, c4, c8}, r^-6 {1, c4, c8, c12} (numpy or torch)."""
    stack = np.stack if isinstance(x, np.ndarray) else torch.stack
    r2 = x * x + y * y
    c2 = (x * x - y * y) / r2
    c4 = 2.0 * c2 * c2 - 1.0
    c8, i = 2.0 * c4 * c4 - 1.0, 1.0 / r2
    c12, one = 2.0 * c4 * c8 - c4, 0.0 * r2 + 1.0
    return stack([one, i, i * c4, i ** 2, i ** 2 * c4, i ** 2 * c8, i ** 3, i ** 3 * c4, i ** 3 * c8, i ** 3 * c12], -1)


def _phi(dx, dy, stencil):
    """phi at integer offsets (torch int64 tensors of one shape)."""
    table, coef = _phi_table(stencil)
    hi, lo = torch.maximum(dx.abs(), dy.abs()), torch.minimum(dx.abs(), dy.abs())
    x, y = hi.clamp(min=1).to(torch.float64), lo.to(torch.float64)
    far = _far_terms(x, y) @ coef - torch.log(x * x + y * y) / (4.0 * math.pi)
    near = table[hi.clamp(max=NEAR), lo.clamp(max=NEAR)]
    return torch.where(hi <= NEAR, near, far)


@functools.lru_cache(maxsize=8)
def _spectrum(size, stencil):
    """Transform of phi on a periodic size x size grid."""
    k = torch.arange(size, device=DEV)
    k = torch.minimum(k, size - k)
    grid = torch.empty(size, size, dtype=torch.float64, device=DEV)
    step = max(1, (1 << 22) // size)
    for i in range(0, size, step):
        a = k[i:i + step, None].expand(-1, size)
        grid[i:i + step] = _phi(a, k[None, :].expand(a.shape[0], -1), stencil)
    return torch.fft.rfft2(grid)


def _convolve(src, f, tgt, side, stencil):
    """u = phi * f for points of a side x side box, by FFT on the doubled box."""
    size = 1 << (2 * side - 1).bit_length()
    grid = torch.zeros(size, size, dtype=torch.float64, device=DEV)
    grid.index_put_((src[:, 0].long(), src[:, 1].long()), f, accumulate=True)
    grid = torch.fft.irfft2(torch.fft.rfft2(grid) * _spectrum(size, stencil), s=(size, size))
    return grid[tgt[:, 0].long(), tgt[:, 1].long()]


def _direct(src, f, tgt, stencil):
    out = torch.empty(len(tgt), dtype=torch.float64, device=DEV)
    step = max(1, (1 << 24) // len(src))
    s = src.long()
    for i in range(0, len(tgt), step):
        d = tgt[i:i + step].long()[:, None, :] - s[None, :, :]
        out[i:i + step] = _phi(d[..., 0], d[..., 1], stencil) @ f
    return out


def _exact_field(src, f, tgt, side, stencil):
    """The field of one point set, or None where it would take too long."""
    if len(src) * len(tgt) <= 1 << 30:
        return _direct(src, f, tgt, stencil)
    if side <= 8192:
        return _convolve(src, f, tgt, side, stencil)
    return None


def _gmres(apply, b, tol=1e-14, most=120):
    """Full GMRES (modified Gram-Schmidt twice) from zero."""
    beta = b.norm()
    basis, hess = [b / beta], torch.zeros(most + 1, most, dtype=torch.float64)
    for j in range(most):
        w = apply(basis[j])
        for _ in range(2):
            for i, v in enumerate(basis):
                h = torch.dot(v, w)
                hess[i, j] += h.item()
                w = w - h * v
        hess[j + 1, j] = w.norm().item()
        rhs = torch.zeros(j + 2, 1, dtype=torch.float64)
        rhs[0] = beta.item()
        y = torch.linalg.lstsq(hess[:j + 2, :j + 1], rhs).solution
        left = (hess[:j + 2, :j + 1] @ y - rhs).norm().item()
        if left <= tol * beta.item() or hess[j + 1, j] == 0.0:
            break
        basis.append(w / hess[j + 1, j].item())
    return torch.stack(basis[:len(y)], 1) @ y[:, 0].to(DEV)


def _exact_inclusions(case, seed):
    """mu + B S mu = -B S B v on the bars' nodes (in order of first appearance) and the potential
    u = v - S (B v + mu) at the targets."""
    bars, delta = _bars(case, seed)
    ends = torch.from_numpy(bars.reshape(-1, 2).astype(np.int64))
    keys = ((ends[:, 0] << 32) + ends[:, 1]).numpy()
    _, first, inverse = np.unique(keys, return_index=True, return_inverse=True)
    order = np.argsort(first)
    rank = np.empty_like(order)
    rank[order] = np.arange(len(order))
    idx = torch.from_numpy(rank[inverse].reshape(-1, 2)).to(DEV)
    low = 2   # a diagonal bar may step one node below the box
    nodes = (ends[torch.from_numpy(first[order])]).to(DEV)
    tgt = _bar_targets(case, seed).long()
    d = torch.from_numpy(delta).to(DEV)

    def field(x, at):
        return _convolve(nodes + low, x, at + low, 2 * case["side"] + 2 * low, 5)

    def apply_b(w):
        t = d * (w[idx[:, 0]] - w[idx[:, 1]])
        out = torch.zeros_like(w)
        return out.index_add_(0, idx[:, 0], t).index_add_(0, idx[:, 1], -t)

    v = FIELD[0] * nodes[:, 0].to(torch.float64) + FIELD[1] * nodes[:, 1].to(torch.float64)
    bv = apply_b(v)
    mu = _gmres(lambda x: x + apply_b(field(x, nodes)), -apply_b(field(bv, nodes)))
    vt = FIELD[0] * tgt[:, 0].to(torch.float64) + FIELD[1] * tgt[:, 1].to(torch.float64)
    return [mu, vt - field(bv + mu, tgt)]


def exact(case, seed):
    kind = case["kind"]
    if kind == "points":
        xy, tgt, f = _point_inputs(case, seed)
        if case["mode"] == "sorted":
            return None          # the plan's own point order
        return _exact_field(xy, f, xy if tgt is None else tgt, case["side"], case["stencil"])
    if kind == "forest":
        return torch.cat([_exact_field(xy, f, xy, side, 5) for xy, f, side in _many_inputs(case, seed)])
    if kind == "serving":
        return [_exact_field(xy, f, xy, side, 5) for xy, f, side in _many_inputs(case, seed)]
    if kind == "inclusions":
        return _exact_inclusions(case, seed)
    return None                  # the box's own lattice is too large for a plain transform
