"""Performance cases of the solver: its public entry points over the sizes, precisions and problem
kinds that it is used with.

A case is a dict of plain values: "kind" (the entry point and problem, below), "precision" ("fp64"
or "mixed"; for dst1 "fp32" or "fp64"), the intervals "nx", "ny", "nz" (nz = 0: 2-D) and what the
kind needs beside them.  Kinds:

  poisson_call   poisson_noalloc: a Dirichlet solve without a handle
  dst1           dst1: one batched sine transform along one axis
  poisson        Solver.poisson: a Dirichlet solve with a kept handle
  schur          Solver.schur_apply: the operator of a caller's own Krylov method
  solve_new      Solver(...) and solve: one problem from its data to u
  solve          Solver.solve with a kept handle
  batch          solve_batched: uneven 2-D instances in one call
  varbeta        solve with nodal alpha and beta, one clamped face, Navier faces elsewhere
  triharmonic    solve of the sixth-order equation, one clamped face, Navier faces elsewhere
"""
import math
import random
from types import SimpleNamespace

import torch

import paper_2609_16478_amd as ah

TWO_PI = 2.0 * math.pi
BATCH_SIZES = (64, 96, 128, 192, 256, 384, 512)


def _case(kind, precision, n, **more):
    return dict(kind=kind, precision=precision, nx=n[0], ny=n[1], nz=n[2] if len(n) > 2 else 0, **more)


def listed():
    def named(name, *a, **k):
        return dict(_case(*a, **k), name=name)

    return [
        # the smallest call: one Dirichlet solve inside a caller's loop; latency and launches
        named("poisson_call_2d_64", "poisson_call", "fp64", (64, 64)),
        # a stand-alone single-precision transform on a grid of no special lengths
        named("dst1_fp32_3d_200x150x120", "dst1", "fp32", (200, 150, 120), axis=1),
        # fast Poisson solver on a ragged box: lengths chosen by the user's geometry
        named("poisson_3d_100x90x75", "poisson", "fp64", (100, 90, 75)),
        # the Schur operator on its own in a caller's Krylov method, medium 3-D grid
        named("schur_3d_256", "schur", "fp64", (256, 256, 256)),
        # one small problem from its data to u: the tests' and the smoke run's size
        named("solve_new_2d_32", "solve_new", "fp64", (32, 32)),
        # a 2-D plate on a grid of decimal lengths
        named("solve_2d_500x300", "solve", "fp64", (500, 300)),
        # the 2-D variable-coefficient configuration in mixed precision
        named("solve_2d_1024_mixed", "solve", "mixed", (1024, 1024)),
        # the 3-D variable-coefficient configuration, medium, mixed precision
        named("solve_3d_128_mixed", "solve", "mixed", (128, 128, 128)),
        # the same, large: arrays far beyond the caches, mixed precision
        named("solve_3d_768_mixed", "solve", "mixed", (768, 768, 768)),
        # the batched workload: uneven small 2-D instances in one call
        named("batch_64_mixed", "batch", "mixed", (512, 512), count=64, mix=0),
        # variable alpha and beta (Table 2's setting)
        named("varbeta_3d_128", "varbeta", "fp64", (128, 128, 128)),
        # the sixth-order equation (Table 5's setting)
        named("triharmonic_3d_128", "triharmonic", "fp64", (128, 128, 128)),
    ]


def _size(rng, lo, hi, friendly=False):
    """An interval count in [lo, hi], log-uniform: a length 2^k or 3 2^k, a multiple of ten, or any."""
    v = min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))
    style = 0.0 if friendly else rng.random()
    if style < 0.4:
        usual = [b << k for b in (1, 3) for k in range(2, 13) if lo <= (b << k) <= hi]
        return min(usual, key=lambda u: abs(math.log(u / v)))
    if style < 0.7:
        return min(hi, max(lo, 10 * int(round(v / 10.0))))
    return v


def _grid(rng, dim, lo, hi, friendly=False):
    first = _size(rng, lo, hi, friendly)
    if rng.random() < 0.4:
        return (first,) * dim
    return (first,) + tuple(_size(rng, max(lo, first // 3), min(hi, 3 * first), friendly) for _ in range(dim - 1))


def draw(rng):
    kind = rng.choice(["poisson_call", "dst1", "poisson", "schur", "solve_new", "solve", "solve", "solve_mixed",
                       "solve_mixed", "batch", "varbeta", "triharmonic"])
    dim = rng.choice([2, 3])
    if kind == "poisson_call":
        return _case(kind, "fp64", _grid(rng, dim, 16, 1024 if dim == 2 else 128))
    if kind == "dst1":
        return _case(kind, rng.choice(["fp32", "fp64"]), _grid(rng, dim, 32, 2048 if dim == 2 else 256),
                     axis=rng.randrange(dim))
    if kind in ("poisson", "schur"):
        return _case(kind, "fp64", _grid(rng, dim, 32, 2048 if dim == 2 else 256))
    if kind == "solve_new":
        return _case(kind, "fp64", _grid(rng, dim, 16, 512 if dim == 2 else 96))
    if kind == "solve":
        return _case(kind, "fp64", _grid(rng, dim, 48, 2048 if dim == 2 else 160))
    if kind == "solve_mixed":  # mixed precision: large grids, on lengths chosen for the transform
        return _case("solve", "mixed", _grid(rng, dim, 64, 2048 if dim == 2 else 512, friendly=True))
    if kind == "batch":
        top = rng.choice([128, 256, 384, 512])
        return _case(kind, rng.choice(["fp64", "mixed"]), (top, top), count=rng.randint(8, 64),
                     mix=rng.randrange(1 << 16))
    return _case(kind, "fp64", _grid(rng, 3, 24, 128))  # varbeta, triharmonic


# --------------------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------------------

def _intervals(case):
    return (case["nx"], case["ny"]) + ((case["nz"],) if case["nz"] else ())


def _box(n):
    """A box of equal spacings, its longest side 1."""
    return tuple(v / max(n) for v in n)


def _axes(n, hi):
    """Node coordinates per axis, shaped for broadcasting in memory order (z, y, x)."""
    out = []
    for a in range(len(n)):
        c = torch.linspace(0.0, hi[a], n[a] + 1, dtype=torch.float64, device="cuda")
        out.append(c.reshape([-1 if b == a else 1 for b in reversed(range(len(n)))]))
    return out


def _waves(rng, x, count=3, top=6.0):
    """A smooth field: a few products of cosines of random wave numbers and phases."""
    total = None
    for _ in range(count):
        term = rng.uniform(0.5, 1.5)
        for c in x:
            term = term * torch.cos(rng.uniform(1.0, top) * math.pi * c + rng.uniform(0.0, TWO_PI))
        total = term if total is None else total + term
    return total


def _face_data(rng, n, hi, faces, amp):
    """A nodal field that is a smooth bump (zero on the edges) on each of `faces`, zero elsewhere."""
    x = _axes(n, hi)
    out = torch.zeros([m + 1 for m in reversed(n)], dtype=torch.float64, device="cuda")
    dim = len(n)
    for f in faces:
        a, side = f // 2, f % 2
        bump = rng.uniform(-amp, amp)
        for b in range(dim):
            if b != a:
                bump = bump * torch.sin(rng.randint(1, 3) * math.pi * x[b] / hi[b])
        dst = out.select(dim - 1 - a, n[a] if side else 0)
        dst.copy_(bump.squeeze(dim - 1 - a))
    return out


def _problem(kind, n, rng, strength=0.6):
    """The data of one problem: what a caller hands to Solver or solve_batched."""
    dim, hi = len(n), _box(n)
    x = _axes(n, hi)
    p = SimpleNamespace(n=n, lo=(0.0,) * dim, hi=hi, gD=None, lapgD=None, gL=None, beta=0.0, navier=())
    p.f = 100.0 * _waves(rng, x)
    if kind == "triharmonic":  # clamped at x = 0, Navier elsewhere
        p.alpha = None
        p.navier = (False,) + (True,) * (2 * dim - 1)
        p.gN = _face_data(rng, n, hi, [0], 1.0)
        p.gNN = p.lapu = p.tang4 = None
        p.bilap = _face_data(rng, n, hi, range(1, 2 * dim), 10.0)
    elif kind == "varbeta":  # alpha = |x|^2 + 1, beta = x + y + z + 10
        p.alpha = sum(c * c for c in x) + 1.0
        p.beta = sum(x) + 10.0
        p.navier = (False,) + (True,) * (2 * dim - 1)
        p.gN = _face_data(rng, n, hi, [0], 1.0)
        p.gL = _face_data(rng, n, hi, range(1, 2 * dim), 10.0)
    else:  # clamped on every face, alpha > 0 oscillating
        bump = rng.uniform(0.2, strength) * torch.sin(TWO_PI * rng.randint(1, 3) * x[0])
        for c in x[1:]:
            bump = bump * torch.cos(TWO_PI * rng.randint(1, 3) * c)
        p.alpha = bump + 1.0
        p.gN = _face_data(rng, n, hi, [0, 2 * dim - 1], 1.0)
    return p


def _batch_grids(case):
    pick = random.Random(case["mix"])
    return [(m, m) for m in (pick.choice([s for s in BATCH_SIZES if s <= case["nx"]]) for _ in range(case["count"]))]


def _normal(shape, seed, dtype=torch.float64):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(shape, generator=g, dtype=dtype, device="cuda")


def prepare(case, seed):
    n, kind = _intervals(case), case["kind"]
    rng = random.Random(seed)
    hi = _box(n)
    mode = ah.MIXED if case["precision"] == "mixed" else ah.FP64
    inner = [m - 1 for m in reversed(n)]
    s = SimpleNamespace(kind=kind, n=n, hi=hi, lo=(0.0,) * len(n), mode=mode)
    if kind == "poisson_call":
        s.g = _normal(inner, seed)
    elif kind == "dst1":
        s.axis, s.mode = case["axis"], ah.MIXED if case["precision"] == "fp32" else ah.FP64
        s.g = _normal(inner, seed, torch.float32 if case["precision"] == "fp32" else torch.float64)
    elif kind == "solve_new":
        s.problem = _problem(kind, n, rng)
    elif kind == "batch":
        s.problems = [_problem(kind, m, rng, strength=0.8) for m in _batch_grids(case)]
    else:
        # bench.py's Schur tolerance for the mixed solves, the default elsewhere
        opts = {"tol": 1e-10} if mode == ah.MIXED else {}
        s.solver = ah.Solver(_problem(kind, n, rng), precision=mode, **opts)
        if kind == "poisson":
            s.g = _normal(inner, seed)
        elif kind == "schur":
            s.q = _normal([s.solver.nq], seed)
    return s


def run(s):
    if s.kind == "poisson_call":
        return ah.poisson_noalloc(s.n, s.lo, s.hi, s.g)
    if s.kind == "dst1":
        return ah.dst1(s.g, s.axis, s.mode)
    if s.kind == "poisson":
        return s.solver.poisson(s.g)
    if s.kind == "schur":
        return s.solver.schur_apply(s.q)
    if s.kind == "solve_new":
        with ah.Solver(s.problem, precision=s.mode) as solver:
            return solver.solve()[0]
    if s.kind == "batch":
        return ah.solve_batched(s.problems, precision=s.mode, tol=1e-10)[0]
    return s.solver.solve()[0]


def _transform_flops(n, axes):
    """Of one sine transform of every pencil along each of `axes`: about 2.5 N log2 N a pencil."""
    pts = 1.0
    for m in n:
        pts *= m - 1
    return sum(2.5 * pts * math.log2(n[a]) for a in axes)


def work(case):
    """Each input read once, each output written once; the transforms that lead from the one to the other once."""
    n, kind = _intervals(case), case["kind"]
    dim = len(n)

    def prod(v):
        return float(math.prod(v))

    nodal, inner = prod(m + 1 for m in n), prod(m - 1 for m in n)
    if kind == "dst1":
        return {"bytes": 2 * inner * (4 if case["precision"] == "fp32" else 8), "flops": _transform_flops(n, [case["axis"]])}
    if kind in ("poisson", "poisson_call"):
        return {"bytes": 16 * inner, "flops": 2 * _transform_flops(n, range(dim))}
    if kind == "schur":  # q in and out and the nodal coefficient; two transform solves
        nq = 2 * sum(inner / (m - 1) for m in n)
        return {"bytes": 16 * nq + 8 * nodal, "flops": 4 * _transform_flops(n, range(dim))}
    grids = _batch_grids(case) if kind == "batch" else [n]
    fields = {"varbeta": 4, "triharmonic": 2}.get(kind, 3)  # alpha, f, beta and u, where the problem has them
    solves = 3 if kind == "triharmonic" else 2
    return {"bytes": sum(8 * fields * prod(v + 1 for v in m) for m in grids),
            "flops": sum(2 * solves * _transform_flops(m, range(len(m))) for m in grids)}


# --------------------------------------------------------------------------------------
# the same in plain torch, 64 bits
# --------------------------------------------------------------------------------------

def _sine(x, dim):
    """DST-I along `dim`, sum_m x_m sin(pi k m / N), by an odd extension."""
    z = torch.zeros_like(x.narrow(dim, 0, 1))
    e = torch.cat([z, x, z, -x.flip(dim)], dim)
    return -0.5 * torch.fft.rfft(e, dim=dim).imag.narrow(dim, 1, x.shape[dim])


class _Grid:
    """The compact operators on a box: L and M of nodal fields, and Dirichlet solves with L - c M."""

    def __init__(self, n, hi):
        self.n, self.dim = n, len(n)
        self.h = [hi[a] / n[a] for a in range(self.dim)]
        i2 = [1.0 / (v * v) for v in self.h]
        d = self.dim
        self.edge = {(a, b): (i2[a] + i2[b]) / 12.0 for a in range(d) for b in range(a + 1, d)}
        self.face = [i2[a] - 2.0 * sum(w for ab, w in self.edge.items() if a in ab) for a in range(d)]
        self.mid = -2.0 * sum(self.face) - 4.0 * sum(self.edge.values())
        self.m0 = 1.0 - 2.0 * d / 12.0
        s, lam, mu = [], 0.0, self.m0
        for a in range(d):
            k = torch.arange(1, n[a], dtype=torch.float64, device="cuda")
            s.append((2.0 * torch.cos(math.pi * k / n[a])).reshape([-1 if b == a else 1 for b in reversed(range(d))]))
            lam = lam + self.face[a] * s[a]
            mu = mu + s[a] / 12.0
        for (a, b), w in self.edge.items():
            lam = lam + w * s[a] * s[b]
        self.lam, self.mu = lam + self.mid, mu

    def at(self, x, off):
        """The interior-sized view of nodal `x` moved by `off` (per axis)."""
        for a in range(self.dim):
            x = x.narrow(self.dim - 1 - a, 1 + off[a], self.n[a] - 1)
        return x

    def unit(self, a, s):
        return [s if b == a else 0 for b in range(self.dim)]

    def L(self, x):
        out = self.mid * self.at(x, [0] * self.dim)
        for a in range(self.dim):
            out = out + self.face[a] * (self.at(x, self.unit(a, 1)) + self.at(x, self.unit(a, -1)))
        for (a, b), w in self.edge.items():
            for s in (1, -1):
                for t in (1, -1):
                    out = out + w * self.at(x, [s if c == a else t if c == b else 0 for c in range(self.dim)])
        return out

    def M(self, x):
        out = self.m0 * self.at(x, [0] * self.dim)
        for a in range(self.dim):
            out = out + (self.at(x, self.unit(a, 1)) + self.at(x, self.unit(a, -1))) / 12.0
        return out

    def solve(self, g, c=0.0):
        for a in range(self.dim):
            g = _sine(g, self.dim - 1 - a)
        g = g / (self.lam - c * self.mu)
        for a in range(self.dim):
            g = _sine(g, self.dim - 1 - a) * (2.0 / self.n[a])
        return g

    def nodal(self, inner=None, q=None):
        """A nodal field of interior values and face values (Q's order), zero on the edges."""
        x = torch.zeros([m + 1 for m in reversed(self.n)], dtype=torch.float64, device="cuda")
        if inner is not None:
            self.at(x, [0] * self.dim).copy_(inner)
        if q is not None:
            at = 0
            for f in range(2 * self.dim):
                v = self.on_face(x, f)
                v.copy_(q[at:at + v.numel()].reshape(v.shape))
                at += v.numel()
        return x

    def on_face(self, x, f, depth=0):
        """Nodal values on the interior of face f, or `depth` layers inside it."""
        a, side = f // 2, f % 2
        for b in range(self.dim):
            if b != a:
                x = x.narrow(self.dim - 1 - b, 1, self.n[b] - 1)
        return x.select(self.dim - 1 - a, self.n[a] - depth if side else depth)


def _residual(G, p, q, data):
    """(R(Q), U): the boundary residual of the fields that face values Q (and, with `data`, the problem's) give."""
    tri = hasattr(p, "bilap")
    V = G.nodal(q=q)
    zero = torch.zeros([m - 1 for m in reversed(G.n)], dtype=torch.float64, device="cuda")
    rhs = G.M(p.f.expand(V.shape)) if data else zero
    if tri:
        W = G.nodal(G.solve(rhs - G.L(V)), q)
        U = G.nodal(G.solve(G.M(G.nodal(G.solve(G.M(W))))))
    else:
        alpha = p.alpha.expand(V.shape)
        c = p.beta / alpha if torch.is_tensor(p.beta) else torch.full_like(alpha, p.beta) / alpha
        cm = 0.5 * float(c.max() + c.min())
        rhs = -rhs - G.L(V) + G.M(c * V)
        vi = G.solve(rhs, cm)
        for _ in range(60 if float(c.max() - c.min()) > 1e-14 else 0):
            new = G.solve(rhs + G.M((c - cm) * G.nodal(vi)), cm)
            done = float((new - vi).norm()) <= 1e-15 * float(new.norm())
            vi = new
            if done:
                break
        U = G.nodal(G.solve(G.M(G.nodal(vi, q) / alpha)))
    w = (-104.0, 57.0 / 2.0, -56.0 / 9.0, 11.0 / 16.0) if tri else (6.0, -1.5, 2.0 / 9.0)
    out, at = [], 0
    for f in range(2 * G.dim):
        h = G.h[f // 2]
        Q = G.on_face(V, f)
        known = 0.0
        if p.navier and p.navier[f]:
            if data:
                known = G.on_face(p.bilap, f) if tri else G.on_face(alpha, f) * G.on_face(p.gL, f)
        else:
            known = sum(v * G.on_face(U, f, k + 1) for k, v in enumerate(w))
            if data:
                known = known + (-755.0 / 12.0 if tri else 11.0 / 3.0) * h * G.on_face(p.gN, f)
            known = known / h ** 4 if tri else G.on_face(alpha, f) * known / h ** 2
        out.append((known - Q).reshape(-1))
        at += Q.numel()
    return torch.cat(out), U


def _gmres(apply, b, tol=1e-14, most=250):
    """Full GMRES, twice orthogonalised, until the residual is tol of b or stops falling near it."""
    beta = float(b.norm())
    V = torch.zeros(most + 1, b.numel(), dtype=torch.float64, device="cuda")
    H = torch.zeros(most + 1, most, dtype=torch.float64)
    V[0] = b / beta
    rhs = torch.zeros(most + 1, 1, dtype=torch.float64)
    rhs[0] = beta
    best = math.inf
    for j in range(most):
        w = apply(V[j])
        for _ in range(2):
            d = V[:j + 1] @ w
            w = w - d @ V[:j + 1]
            H[:j + 1, j] += d.cpu()
        H[j + 1, j] = float(w.norm())
        V[j + 1] = w / float(H[j + 1, j])
        if j % 4 == 3 or j == most - 1:
            y = torch.linalg.lstsq(H[:j + 2, :j + 1], rhs[:j + 2]).solution
            r = float((rhs[:j + 2] - H[:j + 2, :j + 1] @ y).norm()) / beta
            if r <= tol or (r < 1e-11 and r > 0.9 * best):
                break
            best = r
    return y[:, 0].to(V.device) @ V[:y.shape[0]]


def _exact_solution(p):
    G = _Grid(p.n, p.hi)
    nq = sum(G.on_face(G.nodal(), f).numel() for f in range(2 * G.dim))
    b = -_residual(G, p, torch.zeros(nq, dtype=torch.float64, device="cuda"), True)[0]
    q = _gmres(lambda v: _residual(G, p, v, False)[0], b)
    return _residual(G, p, q, True)[1]


def exact(case, seed):
    n, kind = _intervals(case), case["kind"]
    if math.prod(m + 1 for m in n) > 20e6 and kind not in ("dst1", "poisson", "poisson_call", "schur"):
        return None  # a 64-bit solve of this size takes too long
    rng = random.Random(seed)
    inner = [m - 1 for m in reversed(n)]
    if kind == "dst1":
        x = _normal(inner, seed, torch.float32 if case["precision"] == "fp32" else torch.float64)
        return _sine(x.double(), len(n) - 1 - case["axis"])
    if kind in ("poisson", "poisson_call"):
        return _Grid(n, _box(n)).solve(_normal(inner, seed))
    if kind == "batch":
        return [_exact_solution(_problem(kind, m, rng, strength=0.8)) for m in _batch_grids(case)]
    p = _problem(kind, n, rng)
    if kind == "schur":
        G = _Grid(n, p.hi)
        nq = 2 * sum(math.prod(inner) // (m - 1) for m in n)
        return _residual(G, p, _normal([nq], seed), False)[0]
    return _exact_solution(p)
