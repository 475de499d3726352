"""What the performance of this library is measured on: the calls its users
make, over the range of grids, energies, precisions and options they make them
with.  Every input is made from a seed alone; `exact` holds the same methods in
plain 64-bit torch.

Paths (the "path" of a case)
  gibbs       one product y = xi x (`gibbs_apply`) on a 1D, 2D or 3D grid
  flow        JKO steps under one of the energies (`flow`) on a 1D, 2D or 3D grid,
              at a fixed iteration count or to a tolerance, the absorption switch
              watched or not
  log         JKO steps of a crowd whose peaks exceed the capacity: the scalings
              leave float32's comfortable range and the step goes on (or starts)
              in the log domain
  attraction  the Wasserstein attraction towards a shifted target (two couplings)
  gradient    forward and backward through `JKOFlowFn`
  room        the heat-kernel operator of a room with obstacles, stored
  solve       the same by solves per product, where a room is too large to store
"""
import math
import random

import torch

import paper_1502_06216_amd as jk

F32, F64 = torch.float32, torch.float64


# ------------------------------------------------------------------- the cases

def _case(path, shape, **kw):
    c = dict(path=path, n0=shape[0], n1=shape[1] if len(shape) > 1 else 0, n2=shape[2] if len(shape) > 2 else 0,
             kind="congestion", precision="fp32", gamma=1e-3, tau=1e-2, steps=1, iters=300, tol=0.0,
             absorb=math.inf, on_a=False)
    c.update(kw)
    return c


def listed():
    named = [
        # The smallest call: one product on a 32 x 32 grid.  Its launches and the host's share are what counts.
        ("gibbs-32", _case("gibbs", (32, 32), gamma=2e-3)),
        # The smallest flow (crowd32): a scalar capacity, no obstacles, fixed 300 iterations per step.
        ("crowd-32", _case("flow", (32, 32), gamma=2e-3, tau=5e-3, steps=2)),
        # The headline workload (crowd256): one step in tolerance mode with six obstacles; it runs to its cap.
        ("crowd-256", _case("flow", (256, 256), gamma=2e-4, tau=2e-3, iters=1000, tol=1e-8)),
        # A grid whose axes are no multiple of anything, split-BF16, with the absorption switch watched.
        ("crowd-ragged", _case("flow", (201, 161), gamma=4e-4, tau=2e-3, precision="split_bf16", absorb=60.0,
                               on_a=True)),
        # Nonlinear diffusion on 512 x 512 (gen512): generalised entropies with exponents 1 to 2, split-BF16.
        ("diffusion-512", _case("flow", (512, 512), kind="gen_entropy", gamma=1e-4, tau=1e-3,
                                precision="split_bf16")),
        # 3D crowd motion (crowd128c) at its configuration: 300 iterations, the switch on max|log a| > 50.
        ("volume-128", _case("flow", (128, 128, 128), gamma=5e-4, tau=2e-3, absorb=50.0, on_a=True)),
        # A ragged volume under the entropy, split-BF16, short steps.
        ("volume-ragged", _case("flow", (45, 38, 51), kind="entropy", gamma=6e-3, tau=1.5e-2, steps=2, iters=50,
                                precision="split_bf16")),
        # The crowd drawn to a density a little away (as crowd256_attraction): two stacked couplings, a wide band.
        ("attraction-256", _case("attraction", (256, 256), kind="attraction")),
        # A training step (crowd256_fixed, two of its steps): forward and the hand-written adjoint.
        ("gradient-256", _case("gradient", (256, 256), gamma=2e-4, tau=2e-3, steps=2)),
        # The literal crowd (peaks above the capacity): the step switches to the log domain and ends there.
        ("log-256", _case("log", (256, 256), gamma=2e-4, tau=2e-3, iters=100, absorb=50.0)),
        # Crowd motion in a room with obstacles on the stored heat-kernel operator (heat100).
        ("room-100", _case("room", (100, 100), gamma=1e-3, tau=2e-2)),
        # A room beyond the stored operator: every product is its implicit solves.
        ("solve-300", _case("solve", (300, 300), gamma=10.0 / 90000.0, tau=200.0 / 90000.0, iters=20)),
    ]
    return [dict(c, name=n) for n, c in named]


def _size(rng, lo, hi):
    """A size in [lo, hi], spread over its logarithm; one in four is a multiple of 32."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.25:
        n = max(32, 32 * int(round(n / 32)))
    return min(hi, max(lo, n))


def draw(rng):
    path = rng.choice(["gibbs", "flow", "flow", "volume", "attraction", "gradient", "log", "room", "solve"])
    prec = rng.choice(["fp32", "split_bf16"])
    ratio = rng.choice([2.5, 4.0, 10.0])          # tau / gamma of the configurations
    cells = rng.uniform(1.5, 5.0)                 # the kernel's width in cells

    def width(shape, least=0.0, **kw):
        g = (max(cells, least) / max(shape)) ** 2
        return dict(dict(gamma=g, tau=ratio * g, precision=prec), **kw)

    if path == "gibbs":
        d = rng.choice([1, 2, 2, 3])
        shape = tuple(_size(rng, *r) for r in {1: [(32, 1024)], 2: [(32, 1024)] * 2, 3: [(24, 128)] * 3}[d])
        return _case("gibbs", shape, **width(shape))
    if path == "flow":
        d = rng.choice([1, 2, 2, 2, 2])
        kind = rng.choice(["congestion", "congestion", "entropy", "porous", "gen_entropy", "zero"])
        shape = tuple(_size(rng, 32, 1024 if d == 1 else 512) for _ in range(d))
        opt = rng.choice([dict(), dict(), dict(tol=1e-6), dict(absorb=60.0, on_a=True)])
        if kind == "entropy":                     # one gentle step: its minimum is at p = 1, far above a density
            return _case("flow", shape, kind=kind, iters=rng.choice([50, 100, 300]),
                         **dict(width(shape), tau=2.5 * width(shape)["gamma"]))
        return _case("flow", shape, kind=kind, iters=rng.choice([50, 100, 300]), steps=rng.choice([1, 2]),
                     **width(shape), **opt)
    if path == "volume":
        kind = rng.choice(["congestion", "entropy", "zero"])
        shape = tuple(_size(rng, 24, 128) for _ in range(3))
        kw = width(shape)
        if kind == "entropy":
            kw["tau"] = 2.5 * kw["gamma"]
        return _case("flow", shape, kind=kind, iters=rng.choice([20, 50, 100]), **kw)
    if path == "attraction":
        shape = (_size(rng, 40, 256), _size(rng, 40, 256))
        return _case("attraction", shape, kind="attraction", precision=prec, iters=rng.choice([50, 100, 300]))
    if path == "gradient":
        # in FP32, as training runs: the capacity makes the loss piecewise smooth, and split-BF16's rounding
        # moves cells across its kinks
        shape = (_size(rng, 32, 256), _size(rng, 32, 256))
        return _case("gradient", shape, iters=rng.choice([50, 100, 300]), steps=rng.choice([1, 2]),
                     **width(shape, 3.0, precision="fp32"))
    if path == "log":
        shape = (_size(rng, 48, 256), _size(rng, 48, 256))
        return _case("log", shape, iters=rng.choice([30, 45, 60]), absorb=rng.choice([0.0, 50.0]), **width(shape))
    lo, hi, iters = (40, 100, rng.choice([50, 100, 300])) if path == "room" else (120, 300, rng.choice([5, 10, 20]))
    shape = (_size(rng, lo, hi), _size(rng, lo, hi))
    g = 10.0 / max(shape) ** 2
    return _case(path, shape, gamma=g, tau=20.0 * g, iters=iters)


# ---------------------------------------------------------------------- inputs

def _shape(c):
    return tuple(n for n in (c["n0"], c["n1"], c["n2"]) if n)


def _mesh(shape):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    axes = [(torch.arange(n, dtype=F64, device=dev) + 0.5) / n for n in shape]
    return torch.meshgrid(*axes, indexing="ij")


def _bumps(rng, X, count, boxes, lo=None, hi=None, sigma=0.05):
    """Gaussian bumps outside the boxes, mass 1 (on the cells outside them)."""
    d = len(X)
    lo, hi = lo or [0.1] * d, hi or [0.9] * d
    p, m, tries = torch.zeros_like(X[0]), 0, 0
    while m < count:
        c = [rng.uniform(lo[k], hi[k]) for k in range(d)]
        tries += 1
        if tries < 200 and any(all(a <= x < a + s for x, a, s in zip(c, *box)) for box in boxes):
            continue
        r2 = sum((X[k] - c[k]) ** 2 for k in range(d))
        p += rng.uniform(0.2, 1.0) * torch.exp(-r2 / (2 * sigma * sigma))
        m += 1
    inside = _inside(X, boxes)
    p = torch.where(inside, torch.zeros_like(p), p)
    return p / p.sum(), inside


def _boxes(rng, d, count):
    out = []
    for _ in range(count):
        s = [rng.uniform(0.05, 0.15) for _ in range(d)]
        out.append(([rng.uniform(0.0, 1.0 - x) for x in s], s))
    return out


def _inside(X, boxes):
    m = torch.zeros_like(X[0], dtype=torch.bool)
    for corner, side in boxes:
        b = torch.ones_like(m)
        for x, a, s in zip(X, corner, side):
            b &= (x >= a) & (x < a + s)
        m |= b
    return m


def _projected(p, kappa):
    """min(c p, kappa) with the mass 1 (the capacity dominates the density, as the method asks)."""
    lo, hi = torch.zeros_like(p.sum()), torch.full_like(p.sum(), 64.0)
    for _ in range(60):
        mid = 0.5 * (lo + hi)
        low = torch.minimum(mid * p, kappa).sum() < 1.0
        lo, hi = torch.where(low, mid, lo), torch.where(low, hi, mid)
    q = torch.minimum(hi * p, kappa)
    return torch.minimum(q / q.sum(), kappa)


def _inputs(c, seed):
    """The fields of a case as float32 tensors, by name."""
    shape = _shape(c)
    d, N = len(shape), math.prod(shape)
    rng = random.Random(f"{seed} {shape}")
    X = _mesh(shape)
    out = {}
    if c["path"] == "gibbs":
        g = torch.Generator().manual_seed(int(seed))
        out["x"] = torch.rand(shape, generator=g).to(X[0].device)
    elif c["path"] in ("room", "solve"):
        n0 = shape[0]
        free = ~((X[0] >= 0.55) & (X[0] < 0.55 + max(0.03, 1.5 / n0)) & ((X[1] - 0.5).abs() >= 0.08))
        pillars = [([rng.uniform(0.1, 0.35), rng.uniform(0.1, 0.8)], [0.08, 0.08]) for _ in range(3)]
        free &= ~_inside(X, pillars)
        p, _ = _bumps(rng, X, 4, pillars, [0.08, 0.1], [0.42, 0.9])
        p = torch.where(free, p, torch.zeros_like(p))
        p = _projected(p / p.sum(), 0.2 * p.max())
        out["p"], out["free"] = p, free
        out["w"] = torch.sqrt((X[0] - 0.95) ** 2 + (X[1] - 0.5) ** 2)
        out["cap"] = p.max()
    elif c["kind"] in ("porous", "entropy", "gen_entropy", "zero"):
        g = torch.Generator().manual_seed(int(seed))
        p = (0.5 + torch.rand(shape, generator=g, dtype=F64)).to(X[0].device)
        for ax, n in enumerate(shape):          # smoothed noise, std 0.02
            x = (torch.arange(n, dtype=F64, device=p.device) + 0.5) / n
            G = torch.exp(-((x[:, None] - x[None, :]) ** 2) / (2 * 0.02 ** 2))
            p = _along(G / G.sum(1, keepdim=True), p, ax)
        out["p"] = p / p.sum()
        if c["kind"] == "gen_entropy":
            out["m_field"] = 1.0 + math.prod(torch.sin(math.pi * x) for x in X)
        elif c["kind"] != "zero":
            out["coef"] = 1.0 + 0.9 * math.prod(torch.sin(6 * math.pi * x) for x in X)
    else:
        small = N < 48 ** d
        boxes = [] if small or d == 1 else _boxes(rng, d, 6 if d == 2 else 10)
        cap = (1.5 if small or d == 1 else 1.2) / N
        exit_ = [0.9] + [0.5] * (d - 1)
        # (a crowd that is drawn along the first axis starts far enough from its lower edge to stay whole)
        lo = [0.2 if c["path"] == "attraction" else 0.1] + [0.1] * (d - 1)
        p, inside = _bumps(rng, X, 3 if small else 8 if d < 3 else 16, boxes, lo)
        kappa = torch.where(inside, torch.zeros_like(p), torch.full_like(p, cap))
        out["w"] = sum((X[k] - exit_[k]) ** 2 for k in range(d))
        if not boxes and c["path"] == "flow":
            out["cap"] = kappa.max()            # a scalar capacity
        else:
            out["kappa"] = kappa
        shift = max(1, round(0.04 * shape[0]))
        if c["path"] == "attraction":
            # all of the target stays on the grid, so no mass has to travel far, and the thin tails (below 1e-9 of
            # the peak) are no crowd: the scalings, whose logs span 2 * shift / gamma, stay in float32's range
            p[:shift] = 0.0
            p = torch.where(p < 1e-9 * p.max(), torch.zeros_like(p), p)
        out["p"] = p if c["path"] == "log" else _projected(p, kappa)
        if c["path"] == "attraction":
            out.pop("w")
            out["target"] = torch.roll(out["p"], -shift, 0)
        elif c["path"] == "gradient":
            g = torch.Generator().manual_seed(int(seed) + 1)
            out["dp"] = (torch.rand(shape, generator=g) - 0.5).to(p.device)
    return {k: (v.to(torch.uint8) if v.dtype == torch.bool else v.to(F32)).contiguous() for k, v in out.items()}


def _density_scale(c):
    return float(math.prod(_shape(c))) if c["kind"] in ("porous", "gen_entropy") else 1.0


def prepare(case, seed):
    c = case
    f = _inputs(c, seed)
    st = dict(case=c, **f)
    if c["path"] == "gradient":
        st["p"].requires_grad_()
        st["w"].requires_grad_()
    elif c["path"] in ("room", "solve"):
        st["op"] = jk.HeatOperator(_shape(c), c["gamma"], 10, mask=f["free"], per_product=c["path"] == "solve")
    if c["path"] not in ("gibbs", "gradient"):
        st["energy"] = jk.EnergySpec(kind=c["kind"], w=f.get("w"), kappa=f.get("kappa"),
                                     kappa_scalar=float(f["cap"]) if "cap" in f else math.inf, coef=f.get("coef"),
                                     m=2.0, density_scale=_density_scale(c), m_field=f.get("m_field"),
                                     target=f.get("target"))
    return st


def run(state):
    s, c = state, state["case"]
    if c["path"] == "gibbs":
        return jk.gibbs_apply(s["x"], c["gamma"], c["precision"])
    if c["path"] == "gradient":
        pT = jk.JKOFlowFn.apply(s["p"], s["w"], s["kappa"], c["gamma"], c["tau"], c["steps"], c["iters"],
                                c["precision"])
        gp, gw = torch.autograd.grad(pT, (s["p"], s["w"]), s["dp"])
        return dict(p=pT, gp=gp, gw=gw)
    if c["path"] in ("room", "solve"):
        p, st = s["op"].flow(s["p"], s["energy"], c["tau"], c["steps"], max_iters=c["iters"])
    else:
        p, st, _ = jk.flow(s["p"], s["energy"], c["gamma"], c["tau"], c["steps"], max_iters=c["iters"], tol=c["tol"],
                           precision=c["precision"], absorb_threshold=c["absorb"], absorb_on_a=c["on_a"])
    return dict(p=p, iters=[x["iters"] for x in st]) if c["tol"] == 0.0 else dict(p=p)


def work(case):
    c = case
    shape = _shape(c)
    N = math.prod(shape)
    applications = 1 if c["path"] == "gibbs" else 2 * c["iters"] * c["steps"]
    if c["path"] in ("room", "solve"):
        free = 0.94 * N
        if c["path"] == "room":      # the operator's upper triangle once; a product is one flop pair per entry
            return dict(bytes=2.0 * free * free + 13.0 * N, flops=applications * 2.0 * free * free)
        return dict(bytes=13.0 * N, flops=applications * 10 * 10.0 * free)   # ten solves, a few flops a cell each
    # a product: per axis the factor's entries that float32 can hold (the band where exp does not underflow)
    reach = math.sqrt(152 * math.log(2) * c["gamma"])
    taps = sum(min(n, 2 * int(reach * n) + 1) for n in shape)
    flops = 2.0 * N * taps * applications
    fields = 2
    if c["path"] != "gibbs":
        fields += dict(congestion=2, attraction=2, gen_entropy=1, entropy=1, porous=1, zero=0)[c["kind"]]
    if c["path"] == "attraction":
        flops *= 2
    if c["path"] == "gradient":     # the reverse sweep, from stored or recomputed products
        flops *= 2
        fields += 3
    return dict(bytes=4.0 * N * fields, flops=flops)


# ------------------------------------------------------- the methods in 64 bits

def _along(K, x, ax):
    """K applied along axis ax of x."""
    y = x.movedim(ax, 0)
    return (K @ y.reshape(y.shape[0], -1)).reshape(K.shape[0], *y.shape[1:]).movedim(0, ax).contiguous()


def _dist2(n, dev):
    i = torch.arange(n, dtype=F64, device=dev) / n
    return (i[:, None] - i[None, :]) ** 2


def _gibbs(shape, gamma, dev):
    Ks = [torch.exp(-_dist2(n, dev) / gamma) for n in shape]

    def xi(x):
        for ax in reversed(range(len(shape))):
            x = _along(Ks[ax], x, ax)
        return x
    return xi


def _gibbs_log(shape, gamma, dev):
    Cs = [_dist2(n, dev) / gamma for n in shape]

    def one(C, x, ax):
        y = x.movedim(ax, -1)
        out = torch.empty_like(y)
        flat, res = y.reshape(-1, y.shape[-1]), out.view(-1, y.shape[-1])
        for r in range(0, flat.shape[0], 128):
            res[r:r + 128] = torch.logsumexp(flat[r:r + 128, None, :] - C[None], -1)
        return out.movedim(-1, ax).contiguous()

    def lxi(x):
        for ax in reversed(range(len(shape))):
            x = one(Cs[ax], x, ax)
        return x
    return lxi


def _heat(c, free):
    """The heat kernel's product: dense where the room is small, else by solves."""
    n = _shape(c)
    L = 10
    nu = [c["gamma"] * k * k / L for k in n]
    fr = free.to(F64)
    W = []                                  # weights of the four neighbours
    for ax in (0, 1):
        both = fr.narrow(ax, 1, n[ax] - 1) * fr.narrow(ax, 0, n[ax] - 1) * nu[ax]
        W.append(both)

    def M(x):                               # (..., n0, n1)
        y = x.clone()
        for ax, w in zip((-2, -1), W):
            m = x.shape[ax]
            f = w * (x.narrow(ax, 1, m - 1) - x.narrow(ax, 0, m - 1))
            y.narrow(ax, 1, m - 1).add_(f)
            y.narrow(ax, 0, m - 1).sub_(f)
        return y

    beta = 1 + 4 * sum(nu)
    if c["path"] == "room":
        at = free.reshape(-1).nonzero().reshape(-1)
        eye = torch.zeros(at.numel(), *n, dtype=F64, device=free.device)
        eye.view(at.numel(), -1)[torch.arange(at.numel(), device=at.device), at] = 1.0
        A = torch.cat([M(e).view(e.shape[0], -1)[:, at] for e in eye.split(1024)])
        del eye
        I = torch.eye(at.numel(), dtype=F64, device=A.device)
        Z = I * (2 / (1 + beta))            # Newton-Schulz: the residual squares each time
        for _ in range(9):
            Z = Z @ (2 * I - A @ Z)
        Z2 = Z @ Z
        Z4 = Z2 @ Z2
        op = Z4 @ Z4 @ Z2

        def product(x):
            y = torch.zeros_like(x)
            y.view(-1)[at] = op @ x.reshape(-1)[at]
            return y
        return product
    theta, delta = 0.5 * (beta + 1), 0.5 * (beta - 1)
    steps = int(math.ceil(math.log(1e-18) / math.log((math.sqrt(beta) - 1) / (math.sqrt(beta) + 1))))

    def product(x):
        x = x * fr
        for _ in range(L):                  # Chebyshev iterations of M y = x from the guess x
            y, r = x.clone(), x - M(x)
            dvec, rho = r / theta, delta / theta
            for _ in range(steps):
                y += dvec
                r = r - M(dvec)
                nxt = 1 / (2 * theta / delta - rho)
                dvec, rho = nxt * rho * dvec + (2 * nxt / delta) * r, nxt
            x = y
        return x
    return product


def _prox(c, f, sigma):
    """Prox of a case's energy at s (logs to logs where the case is a log one)."""
    kind = c["kind"]
    if kind == "congestion":
        kap = f["kappa"].to(F64) if "kappa" in f else f["cap"].to(F64)
        w = f["w"].to(F64)
        if c["path"] == "log":
            return lambda ls: torch.minimum(ls - sigma * w, torch.log(kap))
        return lambda s: torch.minimum(s * torch.exp(-sigma * w), kap)
    if kind == "entropy":
        e = 1 / (1 + sigma * f["coef"].to(F64))
        return lambda s: s ** e
    D = _density_scale(c)
    if kind == "porous":                    # m = 2: log p + k p = log s
        lk = torch.log(sigma * f["coef"].to(F64) * 2 * D)

        def porous(s):
            lz = lk + torch.log(s)
            v = torch.where(lz < 1, torch.log1p(torch.exp(lz.clamp(max=1))), lz - torch.log(lz.clamp(min=1)))
            for _ in range(12):
                v = v - (torch.log(v) + v - lz) * v / (1 + v)
            return s * torch.exp(-v)
        return porous
    if kind == "gen_entropy":
        m = f["m_field"].to(F64)
        cc, eps = sigma * m, m - 1

        def gen(s):
            Lg = torch.log(s * D)
            y = Lg / (1 + cc)
            small = eps <= 0
            es = torch.where(small, torch.ones_like(eps), eps)
            y = torch.where((Lg > 0) & ~small, torch.minimum(y, torch.log1p(es * Lg.clamp(min=0) / cc) / es), y)
            for _ in range(30):
                g = torch.where(small, y, torch.expm1(es * y) / es)
                y = y - (y + cc * g - Lg) / (1 + cc * torch.exp(es * y * (~small)))
            return torch.exp(y) / D
        return gen
    return lambda s: s


def _over(a, b):
    return torch.where(a == 0, torch.zeros_like(a), a / b)


def _step(c, q, xi, prox):
    """One step; in tolerance mode it stops as the library does."""
    a = torch.ones_like(q)
    p = b = None
    for k in range(1, c["iters"] + 1):
        t = xi(a)
        if c["tol"] > 0 and k > 1 and (k - 1) % 10 == 0 and float((b * t - q).abs().sum()) <= c["tol"]:
            return p
        b = _over(q, t)
        s = xi(b)
        p = prox(s)
        a = _over(p, s)
    return p


def exact(case, seed):
    c = case
    f = _inputs(c, seed)
    shape = _shape(c)
    dev = next(iter(f.values())).device
    if c["path"] == "gibbs":
        return _gibbs(shape, c["gamma"], dev)(f["x"].to(F64))
    sigma = c["tau"] / c["gamma"]
    q = f["p"].to(F64)
    if c["path"] == "gradient":
        p0, w, kap = q.clone().requires_grad_(), f["w"].to(F64).requires_grad_(), f["kappa"].to(F64)
        xi = _gibbs(shape, c["gamma"], dev)
        p = p0
        for _ in range(c["steps"]):
            q, a = p, torch.ones_like(p)
            for _ in range(c["iters"]):
                t = xi(a)
                b = q / t.clamp(min=1e-300)
                s = xi(b)
                z = s * torch.exp(-sigma * w)
                p = torch.where(z < kap, z, kap)
                a = p / s.clamp(min=1e-300)
        gp, gw = torch.autograd.grad(p, (p0, w), f["dp"].to(F64))
        return dict(p=p.detach(), gp=gp, gw=gw)
    none = {} if c["tol"] else dict(iters=[None] * c["steps"])
    if c["path"] == "log":
        lxi, prox = _gibbs_log(shape, c["gamma"], dev), _prox(c, f, sigma)
        p = q
        for _ in range(c["steps"]):
            lq, la = torch.log(p), torch.zeros_like(p)
            for _ in range(c["iters"]):
                lb = lq - lxi(la)
                ls = lxi(lb)
                lp = prox(ls)
                la = torch.where(lp == -math.inf, lp, lp - ls)
            p = torch.exp(lp)
        return dict(p=p, **none)
    if c["path"] == "attraction":
        xi, kap, al = _gibbs(shape, c["gamma"], dev), f["kappa"].to(F64), 1 / (1 + c["tau"])
        p = q
        for _ in range(c["steps"]):
            q = p
            r = f["target"].to(F64)
            r = r * (q.sum() / r.sum())
            a1, a2 = torch.ones_like(q), torch.ones_like(q)
            for _ in range(c["iters"]):
                b1, b2 = _over(q, xi(a1)), _over(r, xi(a2))
                s1, s2 = xi(b1), xi(b2)
                p = torch.minimum(s1 ** al * s2 ** (1 - al), kap)
                a1, a2 = _over(p, s1), _over(p, s2)
        return dict(p=p, **none)
    if c["path"] in ("room", "solve"):
        xi = _heat(c, f["free"])
    else:
        xi = _gibbs(shape, c["gamma"], dev)
    prox = _prox(c, f, sigma)
    p = q
    for _ in range(c["steps"]):
        p = _step(c, p, xi, prox)
    return dict(p=p, **none)
