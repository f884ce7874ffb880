"""Performance cases: what a program built on this framework has it do.

A ground-state run (and a caller's own optimiser) spends its time in a few
public calls: Hessian-vector products at a fixed point (the truncated CG), the
energy and the Riemannian gradient (line searches, the first-order warm start),
the retraction, the mesh-to-mesh prolongation of the cascadic hierarchy, the
batched products of many small problems, the differentiable energy, and the
Newton solve that strings them together.  ``listed()`` holds one case of each
at the sizes of the repository's own workloads (spin-1 1D 128, spin-2 2D
256^2, spin-3 3D 128^3, spin-2 3D 96^3, 64 spin-1 2D problems of uneven grids)
plus a ragged 3D grid; ``draw`` spreads the same calls over spins, dimensions,
supported line lengths (2^k and 3 2^k, 4..512), precisions and options.

Inputs are seeded noise under a Gaussian envelope, as the repository's
workloads use, mapped onto the two-constraint manifold (mass 1, magnetization
M) by giving component l the population of a spin-coherent state; directions
are white noise projected onto the tangent space.
"""

import math

import numpy as np
import torch

from paper_1907_01194_amd import workloads as W
from paper_1907_01194_amd.binding import Batch, Problem

DEV = "cuda" if torch.cuda.is_available() else "cpu"
SIZES = (4, 6, 8, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256, 384, 512)
BATCH_SIZES = (16, 32, 64, 128, 256)
MAX_POINTS = 7 * 128 ** 3          # complex values of the largest field
BETA = {1: (100.0, -0.5), 2: (100.0, 1.0, -1.0), 3: (500.0, 5.0, -5.0, 2.0)}


# ------------------------------------------------------------------ the cases

def listed():
    return [
        # one CG product of the smallest workload: launches and latency
        dict(name="hvp-f1-1d-128", op="hvp", F=1, nx=128, ny=0, nz=0, L=16.0, M=0.5, prec="fp64",
             riem=True, sigma=0.01, dot=False),
        # one step of a caller's own CG (the product and its curvature on the host)
        dict(name="hvpdot-f2-2d-256", op="hvp", F=2, nx=256, ny=256, nz=0, L=12.0, M=0.3, prec="fp64",
             riem=True, sigma=0.01, dot=True),
        # the flagship product, in both precisions
        dict(name="hvp-f3-3d-128-fp64", op="hvp", F=3, nx=128, ny=128, nz=128, L=8.0, M=0.2, prec="fp64",
             riem=True, sigma=0.01, dot=False),
        dict(name="hvp-f3-3d-128-mixed", op="hvp", F=3, nx=128, ny=128, nz=128, L=8.0, M=0.2, prec="mixed",
             riem=True, sigma=0.01, dot=False),
        # an elongated trap: other lengths on every axis, radix-3 lines, the Euclidean product
        dict(name="hvp-f1-3d-192x48x96", op="hvp", F=1, nx=192, ny=48, nz=96, L=12.0, M=0.5, prec="mixed",
             riem=False, sigma=0.0, dot=False),
        # one energy evaluation of a line search
        dict(name="energy-f1-2d-512", op="energy", F=1, nx=512, ny=512, nz=0, L=16.0, M=0.5, prec="fp64"),
        # one Riemannian gradient of the first-order warm start
        dict(name="rgrad-f2-2d-256", op="grad", F=2, nx=256, ny=256, nz=0, L=12.0, M=0.3, prec="fp64", riem=True),
        # the differentiable energy: value, backward and double backward
        dict(name="autograd-f2-3d-96", op="autograd", F=2, nx=96, ny=96, nz=96, L=12.0, M=0.3, prec="fp64"),
        # one retraction of a large field
        dict(name="retract-f3-3d-128", op="retract", F=3, nx=128, ny=128, nz=128, L=8.0, M=0.2, prec="fp64",
             kind=1, t=0.5),
        # mesh transfer of the cascadic hierarchy (the sizes are the coarse mesh's)
        dict(name="prolong-f3-3d-64", op="prolong", F=3, nx=64, ny=64, nz=64, L=8.0, M=0.2, prec="fp64"),
        # the batched product of many uneven problems
        dict(name="batch-hvp-64", op="batch", F=1, count=64, lo=64, hi=256, L=12.0, prec="mixed", riem=True,
             kappa=True, pick=5),
        # a whole call: the Newton solve within an iteration budget
        dict(name="solve-f2-2d-256", op="solve", F=2, nx=256, ny=256, nz=0, L=12.0, M=0.3, prec="fp64",
             rgbb=10, outer=2, cg=12),
    ]


def _axes(rng, dim, F, small, most):
    """dim line lengths, each spread over the logarithm of its range, the field within `most` values."""
    while True:
        n = []
        for _ in range(dim):
            v = math.exp(rng.uniform(math.log(small), math.log(512.0)))
            n.append(min(SIZES, key=lambda s: abs(math.log(s / v))))
        if (2 * F + 1) * np.prod(n) <= most:
            return n + [0] * (3 - dim)


def draw(rng):
    op = rng.choice(["hvp"] * 5 + ["energy", "grad", "grad", "autograd", "retract", "prolong", "batch", "batch"])
    F = rng.choice([1, 2, 3])
    M = round(rng.uniform(0.05, 0.9 * F), 3)
    L = rng.choice([8.0, 12.0, 16.0])
    prec = rng.choice(["fp64", "mixed"])
    if op == "batch":
        lo = rng.choice(BATCH_SIZES[:4])
        hi = rng.choice([s for s in BATCH_SIZES if s >= lo])
        return dict(op="batch", F=rng.choice([1, 1, 2]), count=rng.randint(2, 48), lo=lo, hi=hi, L=L, prec=prec,
                    riem=rng.random() < 0.7, kappa=rng.random() < 0.5, pick=rng.randint(0, 10 ** 6))
    dim = rng.choice([1, 2, 2, 3, 3, 3])
    most = MAX_POINTS // 4 if op == "autograd" else MAX_POINTS
    if op == "prolong":
        while True:
            nx, ny, nz = _axes(rng, dim, F, 8.0, MAX_POINTS >> dim)
            if max(nx, ny, nz) <= 128:
                break
    else:
        nx, ny, nz = _axes(rng, dim, F, 64.0 if dim == 1 else 12.0, most)
    if op != "hvp":
        prec = "fp64"      # these calls run in FP64 whatever the handle's work precision
    c = dict(op=op, F=F, nx=nx, ny=ny, nz=nz, L=L, M=M, prec=prec)
    if op == "hvp":
        riem = rng.random() < 0.8
        c.update(riem=riem, sigma=round(rng.uniform(0.0, 0.1), 4) if riem else 0.0, dot=riem and rng.random() < 0.4)
    elif op == "grad":
        c.update(riem=rng.random() < 0.7)
    elif op == "retract":
        c.update(kind=rng.choice([1, 2, 3]), t=round(rng.uniform(0.1, 1.0), 3))
    return c


# ------------------------------------------------------------------ inputs

def _n(case):
    return tuple(int(case[k]) for k in ("nx", "ny", "nz") if case[k])


def _potential(*xs):
    return sum(0.5 * x * x + 10.0 * np.sin(0.25 * np.pi * x) ** 2 for x in xs)


def _spec(F, n, L, M, beta=None):
    d = len(n)
    return W.make_spec("case", F, n, (-L,) * d, (L,) * d, _potential, beta or BETA[F], M)


def _cn(gen, shape):
    return torch.complex(torch.randn(shape, generator=gen, device=DEV, dtype=torch.float64),
                         torch.randn(shape, generator=gen, device=DEV, dtype=torch.float64)) * math.sqrt(0.5)


def _axis(n, L, a, d):
    """Nodes of axis a (x first) broadcast over the grid [z][y][x]."""
    x = -L + (2.0 * L / n[a]) * torch.arange(n[a], device=DEV, dtype=torch.float64)
    return x.reshape([n[a] if b == d - 1 - a else 1 for b in range(d)])


def _lv(F, d):
    return torch.arange(F, -F - 1, -1, device=DEV, dtype=torch.float64).reshape((-1,) + (1,) * d)


def _dot(a, b):
    return float((torch.view_as_real(a) * torch.view_as_real(b)).sum())


def _point(gen, F, n, L, M):
    """A point of the manifold: enveloped noise, component l populated as in a spin-coherent state."""
    d, K = len(n), 2 * F + 1
    env = torch.exp(-0.25 * sum(_axis(n, L, a, d) ** 2 for a in range(d)))
    u = _cn(gen, (K,) + tuple(reversed(n))) * env
    p = 0.5 * (1.0 + M / F)
    pop = torch.tensor([math.comb(2 * F, i) * p ** (2 * F - i) * (1 - p) ** i for i in range(K)],
                       device=DEV, dtype=torch.float64)
    nrm = torch.view_as_real(u).reshape(K, -1).square().sum(1)
    return u * (pop / nrm).sqrt().reshape((-1,) + (1,) * d)


def _project(F, u, w):
    """Orthogonal projection of w onto the tangent space of the two constraints at u."""
    l = _lv(F, u.dim() - 1)
    lu = l * u
    a11, a12, a22 = _dot(u, u), _dot(u, lu), _dot(lu, lu)
    r1, r2 = _dot(u, w), _dot(lu, w)
    det = a11 * a22 - a12 * a12
    return w - ((a22 * r1 - a12 * r2) / det) * u - ((a11 * r2 - a12 * r1) / det) * lu


def _inputs(case, seed):
    """(point u, unit tangent direction z) of a case, made from the seed alone."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    F, n, L, M = case["F"], _n(case), case["L"], case["M"]
    u = _point(gen, F, n, L, M)
    z = _project(F, u, _cn(gen, u.shape))
    return u, z / math.sqrt(_dot(z, z))


def _batch_problems(case):
    """(line length, beta1, M) of every problem of a batch: part of the case, not of the inputs."""
    rng = np.random.default_rng(case["pick"])
    sizes = [s for s in BATCH_SIZES if case["lo"] <= s <= case["hi"]]
    return [(int(rng.choice(sizes)), float(rng.uniform(-1, 1)), float(rng.uniform(0, 0.9)))
            for _ in range(case["count"])]


def _batch_beta(F, b1):
    return {1: (100.0, b1), 2: (100.0, b1, -1.0), 3: (100.0, b1, 10.0, 1.0)}[F]


def _batch_inputs(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    us, zs = [], []
    for n, _, M in _batch_problems(case):
        u = _point(gen, case["F"], (n, n), case["L"], M)
        z = _project(case["F"], u, _cn(gen, u.shape))
        us.append(u)
        zs.append(z / math.sqrt(_dot(z, z)))
    return us, zs


# ------------------------------------------------------------------ one pass

def prepare(case, seed):
    op = case["op"]
    if op == "batch":
        us, zs = _batch_inputs(case, seed)
        b = Batch([_spec(case["F"], (n, n), case["L"], M, _batch_beta(case["F"], b1))
                   for n, b1, M in _batch_problems(case)], case["prec"])
        for p, u in zip(b.problems, us):
            p.set_point(u)
        wd = b.problems[0].work_dtype
        return dict(case=case, b=b, Z=[z.to(wd) for z in zs], sigma=[0.01] * len(zs))
    u, z = _inputs(case, seed)
    n = _n(case)
    p = Problem(_spec(case["F"], n, case["L"], case["M"]), case["prec"])
    s = dict(case=case, p=p, X=u)
    if op == "hvp":
        p.set_point(u)
        s["Z"] = z.to(p.work_dtype)
    elif op == "retract":
        s["Z"] = z
    elif op == "autograd":
        s["X"] = u.requires_grad_(True)
        s["Z"] = z
    elif op == "prolong":
        s["fine"] = Problem(_spec(case["F"], tuple(2 * m for m in n), case["L"], case["M"]), case["prec"])
    return s


def run(s):
    from paper_1907_01194_amd import autograd
    case = s["case"]
    op = case["op"]
    if op == "hvp":
        if case["dot"]:
            return s["p"].hvp_dot(s["Z"], sigma=case["sigma"])
        return s["p"].hvp(s["Z"], riemannian=case["riem"], sigma=case["sigma"])
    if op == "energy":
        return np.float64(s["p"].energy(s["X"]))
    if op == "grad":
        G, E, gn = s["p"].grad(s["X"], riemannian=case["riem"])
        return G, np.float64(E), np.float64(gn)
    if op == "autograd":
        E = autograd.energy(s["X"], s["p"])
        (G,) = torch.autograd.grad(E, s["X"], create_graph=True)
        (HZ,) = torch.autograd.grad(G, s["X"], grad_outputs=s["Z"].to(G.dtype))
        return E.detach(), G.detach(), HZ
    if op == "retract":
        return s["p"].retract(s["X"], s["Z"], case["t"], case["kind"])
    if op == "prolong":
        return s["p"].prolong(s["X"], s["fine"])
    if op == "batch":
        H, k = s["b"].hvp(s["Z"], riemannian=case["riem"], sigma=s["sigma"], kappa=case["kappa"])
        # neighbouring problems' products side by side, in a few outputs
        flat = torch.cat([h.reshape(-1) for h in H])
        # (kappa carries the products' precision: compare it as a value of that precision)
        return (flat, np.array(k, np.float64 if case["prec"] == "fp64" else np.float32)) if k is not None else flat
    if op == "solve":
        X = s["X"].clone()
        _, st = s["p"].newton_solve(X, check=False, tol=1e-9, rgbb_maxit=case["rgbb"], rgbb_tol=1e-9,
                                    maxit=case["outer"], cg_maxit=case["cg"], cg_per_digit=0.0)
        return X, np.float64(st["E"]), np.float64(st["gnorm"])
    raise ValueError(op)


# ------------------------------------------------------------------ what a pass cannot do without

def _flops(F, n, grad=False):
    """Transforms along every axis and the pointwise spin terms of one product or gradient."""
    K = 2 * F + 1
    pts = float(np.prod(n))
    point = {1: 150.0, 2: 450.0, 3: 1100.0}[F] * (0.5 if grad else 1.0)
    return K * pts * sum(10.0 * math.log2(m) for m in n) + pts * point


def work(case):
    op, F = case["op"], case["F"]
    K = 2 * F + 1
    c = 16 if case["prec"] == "fp64" else 8
    r = c // 2
    if op == "batch":
        w = [(n, float(n * n)) for n, _, _ in _batch_problems(case)]
        return dict(bytes=sum(p * (3 * K * c + r) for _, p in w), flops=sum(_flops(F, (n, n)) for n, _ in w))
    n = _n(case)
    pts = float(np.prod(n))
    f, g = _flops(F, n), _flops(F, n, True)
    if op == "hvp":       # X, Z, V in; HZ out
        return dict(bytes=pts * (3 * K * c + r), flops=f)
    if op == "energy":    # X, V in
        return dict(bytes=pts * (16 * K + 8), flops=0.6 * g)
    if op == "grad":      # X, V in; G out
        return dict(bytes=pts * (32 * K + 8), flops=g)
    if op == "autograd":  # the energy, the gradient, the product (whose direction and result are c128)
        return dict(bytes=pts * (16 * K + 8 + 32 * K + 8 + 32 * K + c * K + r), flops=1.6 * g + f)
    if op == "retract":   # X, Xi in; Xout out
        return dict(bytes=pts * 48 * K, flops=pts * K * 20.0)
    if op == "prolong":   # the coarse field in, the fine field out
        d = len(n)
        return dict(bytes=pts * 16 * K * (1 + 2 ** d),
                    flops=K * pts * sum(2 ** a * 10.0 * math.log2(m) for a, m in enumerate(n)))
    # solve: per warm-start iteration a gradient and a retraction, per CG iteration a product
    return dict(bytes=pts * (case["rgbb"] * (32 * K + 8 + 48 * K) + case["outer"] * case["cg"] * (3 * K * c + r)),
                flops=case["rgbb"] * g + case["outer"] * case["cg"] * f)


# ------------------------------------------------------------------ the same values in plain 64-bit torch

def _spin(F):
    """Dense spin matrices f_x, f_y, f_z, the singlet matrix and the quintet matrices as (K, K) tensors."""
    K = 2 * F + 1
    up = np.zeros((K, K))
    for i in range(1, K):
        m = F - i
        up[i - 1, i] = math.sqrt(F * (F + 1) - m * (m + 1))
    f = [0.5 * (up + up.T) + 0j, -0.5j * (up - up.T), np.diag(np.arange(F, -F - 1, -1)) + 0j]
    A = None
    if F >= 2:
        A = np.zeros((K, K), complex)
        for i in range(K):
            A[i, K - 1 - i] = (-1) ** i / math.sqrt(K)
    quint = []
    if F == 3:
        s = math.sqrt
        v1 = [5 / (2 * s(3)), -s(5) / 2, 1 / s(6), 1 / s(6), -s(5) / 2, 5 / (2 * s(3))]
        v2 = [s(5 / 6), -s(5 / 3), s(2), -s(5 / 3), s(5 / 6)]
        v0 = [5 / (2 * s(3)), 0.0, -s(3) / 2, s(2 / 3), -s(3) / 2, 0.0, 5 / (2 * s(3))]
        for m, v, at in ((-2, v2, 2), (-1, v1, 1), (0, v0, 0), (1, v1, 0), (2, v2, 0)):
            Q = np.zeros((7, 7), complex)
            for k, x in enumerate(v):
                i = at + k
                Q[i, 6 - m - i] = x / s(7)
            quint.append(Q)
    t = lambda a: None if a is None else torch.tensor(a, device=DEV, dtype=torch.complex128)  # noqa: E731
    return [t(a) for a in f], t(A), [t(a) for a in quint]


def _apply(Mx, X):
    """(M X)_i = sum_j M_ij X_j for a sparse (K, K) matrix."""
    out = torch.zeros_like(X)
    for i in range(X.shape[0]):
        for j in range(X.shape[0]):
            c = complex(Mx[i, j])
            if c:
                out[i] += c * X[j]
    return out


class _Plain:
    """E, its gradient and its Hessian-vector product by FFTs over the grid and dense spin matrices."""

    def __init__(self, F, n, L, beta):
        self.F, self.n, self.d = F, n, len(n)
        self.h = float(np.prod([2.0 * L / m for m in n]))
        self.beta = list(beta) + [0.0] * (4 - len(beta))
        self.V = sum(0.5 * x * x + 10.0 * torch.sin(0.25 * math.pi * x) ** 2
                     for x in (_axis(n, L, a, self.d) for a in range(self.d)))
        self.sym = 0.0
        for a in range(self.d):
            p = torch.fft.fftfreq(n[a], 1.0 / n[a], device=DEV, dtype=torch.float64)
            lam = (math.pi / L * p) ** 2
            self.sym = self.sym + lam.reshape([n[a] if b == self.d - 1 - a else 1 for b in range(self.d)])
        self.f, self.A, self.Q = _spin(F)

    def lap(self, X):
        ax = tuple(range(1, self.d + 1))
        return torch.fft.ifftn(torch.fft.fftn(X, dim=ax) * self.sym, dim=ax)

    def _fields(self, X):
        rho = (X * X.conj()).real.sum(0)
        fx = [_apply(m, X) for m in self.f]
        pair = ([(2, self.A)] if self.A is not None else []) + [(3, q) for q in self.Q]
        return rho, fx, pair

    def energy(self, X):
        rho, fx, pair = self._fields(X)
        b, h = self.beta, self.h
        E = 0.5 * _dot(X, self.lap(X)) + float((self.V * rho).sum()) + b[0] / (2 * h) * float((rho * rho).sum())
        for y in fx:
            E += b[1] / (2 * h) * float(((X.conj() * y).real.sum(0) ** 2).sum())
        for k, m in pair:
            a = (X * _apply(m, X)).sum(0)
            E += b[k] / (2 * h) * float((a.abs() ** 2).sum())
        return E

    def grad(self, X):
        rho, fx, pair = self._fields(X)
        b, h = self.beta, self.h
        G = self.lap(X) + 2 * self.V * X + (2 * b[0] / h) * rho * X
        for y in fx:
            G += (2 * b[1] / h) * (X.conj() * y).real.sum(0) * y
        for k, m in pair:
            G += (2 * b[k] / h) * (X * _apply(m, X)).sum(0) * _apply(m, X.conj())
        return G

    def hvp(self, X, Z):
        rho, fx, pair = self._fields(X)
        b, h = self.beta, self.h
        H = self.lap(Z) + 2 * self.V * Z
        H += (2 * b[0] / h) * (rho * Z + 2 * (Z * X.conj()).real.sum(0) * X)
        for m, y in zip(self.f, fx):
            H += (2 * b[1] / h) * ((X.conj() * y).real.sum(0) * _apply(m, Z)
                                   + 2 * (Z.conj() * y).real.sum(0) * y)
        for k, m in pair:
            H += (2 * b[k] / h) * ((X * _apply(m, X)).sum(0) * _apply(m, Z.conj())
                                   + 2 * (Z * _apply(m, X)).sum(0) * _apply(m, X.conj()))
        return H

    def rhess(self, X, Z, sigma):
        G = self.grad(X)
        l = _lv(self.F, self.d)
        lX = l * X
        a11, a12, a22 = _dot(X, X), _dot(X, lX), _dot(lX, lX)
        r1, r2 = _dot(X, G), _dot(lX, G)
        det = a11 * a22 - a12 * a12
        ag, bg = (a22 * r1 - a12 * r2) / det, (a11 * r2 - a12 * r1) / det
        return _project(self.F, X, self.hvp(X, Z) + (sigma - ag) * Z - bg * l * Z)


def _sigma(F, M, kind, a):
    """Factors of the three retractions from the component norms a (storage order l = F..-F)."""
    l = np.arange(F, -F - 1, -1).astype(float)
    if kind == 3:
        ww, g1, g2 = a.sum(), (l * a).sum(), (l * l * a).sum()
        return np.sqrt((g2 - (M + l) * g1 + M * l * ww) / (ww * g2 - g1 * g1))
    if kind == 2:
        value = lambda s: float(((l - M) * a * np.exp(l * s)).sum())  # noqa: E731
        lo, hi = -60.0, 60.0
    else:
        value = lambda t: float(((l - M) * a / (1 - (l - M) * t) ** 2).sum())  # noqa: E731
        lo, hi = 1 / (-F - M), 1 / (F - M)
    for _ in range(200):
        mid = 0.5 * (lo + hi)
        lo, hi = (lo, mid) if value(mid) > 0 else (mid, hi)
    t = 0.5 * (lo + hi)
    w = np.exp(0.5 * l * t) if kind == 2 else 1 / (1 - (l - M) * t)
    return w / math.sqrt(float((a * w * w).sum()))


def _interpolate(X, n, a, d):
    """Trigonometric interpolant along axis a (x first) onto twice the nodes, Nyquist split evenly."""
    dim = 1 + d - 1 - a
    m = n[a]
    C = torch.fft.fft(X, dim=dim)
    lo, ny, hi = C.narrow(dim, 0, m // 2), 0.5 * C.narrow(dim, m // 2, 1), C.narrow(dim, m // 2 + 1, m // 2 - 1)
    shape = list(C.shape)
    shape[dim] = m - 1
    zero = torch.zeros(shape, device=DEV, dtype=C.dtype)
    return 2.0 * torch.fft.ifft(torch.cat([lo, ny, zero, ny, hi], dim=dim), dim=dim)


def exact(case, seed):
    op = case["op"]
    if op == "solve":
        return None
    wd = torch.complex128 if case["prec"] == "fp64" else torch.complex64
    if op == "batch":
        us, zs = _batch_inputs(case, seed)
        out, kap = [], []
        for (n, b1, M), u, z in zip(_batch_problems(case), us, zs):
            e = _Plain(case["F"], (n, n), case["L"], _batch_beta(case["F"], b1))
            z = z.to(wd).to(torch.complex128)
            H = e.rhess(u, z, 0.01) if case["riem"] else e.hvp(u, z)
            out.append(H.reshape(-1))
            kap.append(_dot(z, H))
        return (torch.cat(out), np.array(kap)) if case["kappa"] else torch.cat(out)
    u, z = _inputs(case, seed)
    n = _n(case)
    if op == "prolong":
        for a in range(len(n)):
            u = _interpolate(u, n, a, len(n))
        return u * 2.0 ** (-0.5 * len(n))
    if op == "retract":
        w = u + case["t"] * z
        a = torch.view_as_real(w).reshape(w.shape[0], -1).square().sum(1).cpu().numpy()
        s = torch.tensor(_sigma(case["F"], case["M"], case["kind"], a), device=DEV)
        return w * s.reshape((-1,) + (1,) * len(n))
    e = _Plain(case["F"], n, case["L"], BETA[case["F"]])
    if op == "hvp":
        z = z.to(wd).to(torch.complex128)
        H = e.rhess(u, z, case["sigma"]) if case["riem"] else e.hvp(u, z)
        return (H, np.float64(_dot(z, H))) if case["dot"] else H
    if op == "energy":
        return np.float64(e.energy(u))
    G = e.grad(u)
    if op == "grad":
        E = np.float64(e.energy(u))
        if case["riem"]:
            G = _project(case["F"], u, G)
        return G, E, np.float64(math.sqrt(_dot(G, G)))
    return torch.tensor(e.energy(u), device=DEV, dtype=torch.float64), G, e.hvp(u, z.to(wd).to(torch.complex128))
