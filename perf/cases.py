"""The work a user of the library has it do, as timed cases.

``listed()`` names the cases, ``draw(rng)`` gives further ones of the same
ranges, ``prepare(case, seed)`` makes a case's inputs on the GPU, ``run(state)``
is one pass through the public entry points, ``work(case)`` the bytes and
operations a pass cannot do without, and ``exact(case, seed)`` the same outputs
in FP64 from plain torch and numpy.

A case is ``{"entry", "matrix", "size", "degree", "cols", "dtype"}``:

entry   ``logdet``, ``logdet_adaptive``, ``logdet_with_grad`` (cols = queries),
        ``apply_log``, ``apply_log_adaptive`` (cols = columns of V),
        ``spectral_bounds`` (degree = Lanczos steps)
matrix  ``grid2d``    kappa^2 I + 5-point Laplacian, size x size points
        ``gmrf``      tau (kappa^2 I + 5-point Laplacian)
        ``theta``     I + theta Adj on a size x size grid (the likelihood sweep)
        ``grid3d``    kappa^2 I + 7-point Laplacian, size^3 points
        ``penta``     random pentadiagonal matrix plus about n I, n = size
        ``mesh``      irregular sparse matrix of a mesh in a banded order, n = size
        ``chunglu``   weighted Laplacian of a power-law graph plus 0.01 I, n = size

The coefficients and the probe seed come from the seed.
"""
import decimal
import math

import numpy as np
import torch

import paper_2603_02207_amd as ld

DEV = "cuda:0"
DTYPES = {"f32": torch.float32, "f64": torch.float64}
MESH_WINDOW, MESH_DENSITY = 40, 0.18   # about 15 stored entries a row


def _case(name, entry, matrix, size, degree, cols, dtype):
    return dict(name=name, entry=entry, matrix=matrix, size=size, degree=degree, cols=cols, dtype=dtype)


def listed():
    return [
        # the smallest estimate: a 32 x 32 grid in a serving loop, all latency
        _case("logdet_grid32_f32", "logdet", "grid2d", 32, 40, 30, "f32"),
        # a finite-element matrix of the size the method is usually quoted on
        # (tens of thousands of rows, about 15 entries each), FP64, few queries
        _case("logdet_mesh36k_f64", "logdet", "mesh", 36441, 81, 12, "f64"),
        # the benchmark: a million-point grid precision matrix, 60 queries
        _case("logdet_grid1024_f32", "logdet", "grid2d", 1024, 80, 60, "f32"),
        # one evaluation of the likelihood sweep over theta: 25 million points
        _case("logdet_theta5000_f32", "logdet", "theta", 5000, 80, 30, "f32"),
        # a 3-D grid at full precision with many queries
        _case("logdet_grid128c_f64", "logdet", "grid3d", 128, 120, 96, "f64"),
        # a power-law graph: irregular rows from one entry to thousands
        _case("logdet_chunglu1M_f32", "logdet", "chunglu", 1 << 20, 150, 64, "f32"),
        # the pentadiagonal study at its largest size, low degree
        _case("logdet_penta1e7_f32", "logdet", "penta", 10_000_000, 8, 30, "f32"),
        # the estimate with a degree of its own for every column
        _case("adaptive_gmrf2048_f32", "logdet_adaptive", "gmrf", 2048, 100, 32, "f32"),
        # log(A) V for a ragged block of vectors on a ragged grid (sampling)
        _case("apply_grid500_17_f32", "apply_log", "grid2d", 500, 60, 17, "f32"),
        # log(A) V to a tolerance on an irregular matrix, full precision
        _case("apply_adaptive_mesh36k_f64", "apply_log_adaptive", "mesh", 36441, 120, 10, "f64"),
        # a step of hyperparameter fitting: the estimate and its derivative
        _case("grad_gmrf1024_f32", "logdet_with_grad", "gmrf", 1024, 100, 32, "f32"),
        # the spectral interval before an estimate, upper end from Lanczos
        _case("bounds_mesh200k_f32", "spectral_bounds", "mesh", 200_000, 64, 0, "f32"),
    ]


def draw(rng):
    """One more case of the ranges above; odd sizes among them, spread over their logarithm."""
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    dtype = rng.choice(["f32", "f64"])
    kind = rng.choice(["small", "mesh", "grid2d", "theta", "grid3d", "chunglu", "penta", "adaptive", "apply",
                       "apply_adaptive", "grad", "bounds"])
    c = dict(dtype=dtype)
    if kind == "small":
        c.update(entry="logdet", matrix="grid2d", size=size(20, 120), degree=rng.randint(20, 80), cols=rng.randint(9, 60))
    elif kind == "mesh":
        c.update(entry="logdet", matrix="mesh", size=size(4000, 400_000), degree=rng.randint(40, 120),
                 cols=rng.randint(9, 60))
    elif kind in ("grid2d", "theta"):
        c.update(entry="logdet", matrix=kind, size=size(150, 2200), degree=rng.randint(40, 110), cols=rng.randint(9, 72))
    elif kind == "grid3d":
        c.update(entry="logdet", matrix="grid3d", size=size(16, 120), degree=rng.randint(40, 120),
                 cols=rng.randint(12, 96))
    elif kind == "chunglu":
        c.update(entry="logdet", matrix="chunglu", size=size(8000, 500_000), degree=rng.randint(50, 150),
                 cols=rng.randint(12, 64))
    elif kind == "penta":
        c.update(entry="logdet", matrix="penta", size=size(20_000, 8_000_000), degree=rng.randint(6, 12),
                 cols=rng.randint(9, 45))
    elif kind == "adaptive":
        c.update(entry="logdet_adaptive", matrix=rng.choice(["gmrf", "mesh"]), degree=rng.randint(60, 110),
                 cols=rng.randint(9, 48))
        c["size"] = size(100, 1500) if c["matrix"] == "gmrf" else size(5000, 200_000)
    elif kind == "apply":
        c.update(entry="apply_log", matrix=rng.choice(["grid2d", "mesh"]), degree=rng.randint(30, 100),
                 cols=rng.randint(1, 64))
        c["size"] = size(50, 1200) if c["matrix"] == "grid2d" else size(4000, 300_000)
    elif kind == "apply_adaptive":
        c.update(entry="apply_log_adaptive", matrix=rng.choice(["gmrf", "mesh"]), degree=rng.randint(60, 150),
                 cols=rng.randint(1, 40))
        c["size"] = size(50, 1000) if c["matrix"] == "gmrf" else size(4000, 200_000)
    elif kind == "grad":
        c.update(entry="logdet_with_grad", matrix=rng.choice(["gmrf", "mesh"]), degree=rng.randint(30, 100),
                 cols=rng.randint(9, 36))
        c["size"] = size(60, 900) if c["matrix"] == "gmrf" else size(4000, 60_000)
    else:
        c.update(entry="spectral_bounds", matrix=rng.choice(["mesh", "grid2d"]), degree=rng.randint(20, 100), cols=0)
        c["size"] = size(5000, 1_000_000) if c["matrix"] == "mesh" else size(60, 1500)
    return c


# ---- inputs ------------------------------------------------------------------------------

def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _stencil(dims, centre, neighbour):
    """CSR of the Dirichlet stencil: `centre` on the diagonal, `neighbour` on the 2 len(dims) neighbours."""
    n = math.prod(dims)
    idx = torch.arange(n, device=DEV, dtype=torch.int32)
    strides = [math.prod(dims[a + 1:]) for a in range(len(dims))]
    offsets = sorted([(s * d, a, d) for a, s in enumerate(strides) for d in (-1, 1)] + [(0, -1, 0)])
    ok = torch.empty((n, len(offsets)), dtype=torch.bool, device=DEV)
    for q, (_, axis, step) in enumerate(offsets):
        if axis < 0:
            ok[:, q] = True
        else:
            at = torch.div(idx, strides[axis], rounding_mode="floor") % dims[axis]
            ok[:, q] = (at > 0) if step < 0 else (at < dims[axis] - 1)
    row_ptr = torch.zeros(n + 1, dtype=torch.int32, device=DEV)
    row_ptr[1:] = ok.sum(1, dtype=torch.int32).cumsum(0, dtype=torch.int32)
    off = torch.tensor([o for o, _, _ in offsets], dtype=torch.int32, device=DEV)
    col_idx = (idx[:, None] + off[None, :])[ok]
    val = torch.where(off == 0, float(centre), float(neighbour)).to(torch.float64).expand(n, -1)[ok]
    return row_ptr, col_idx, val, n


def _from_edges(n, u, v, w, shift):
    """CSR of diag(sum of a row's weights + shift) - W for the edges (u, v, w), u != v, each pair once."""
    key = torch.cat([u * n + v, v * n + u])
    ww = torch.cat([w, w])
    deg = torch.zeros(n, dtype=torch.float64, device=DEV).index_add_(0, torch.div(key, n, rounding_mode="floor"), ww)
    i = torch.arange(n, device=DEV, dtype=torch.int64)
    key = torch.cat([key, i * (n + 1)])
    val = torch.cat([-ww, deg + shift])
    key, order = torch.sort(key)
    val = val[order]
    rows = torch.div(key, n, rounding_mode="floor")
    row_ptr = torch.zeros(n + 1, dtype=torch.int32, device=DEV)
    row_ptr[1:] = torch.bincount(rows, minlength=n).cumsum(0).to(torch.int32)
    return row_ptr, (key - rows * n).to(torch.int32), val, n


def _matrix(case, seed):
    """(row_ptr, col_idx, val FP64, n), lmin, lmax."""
    g = _generator(seed)
    kind, size = case["matrix"], case["size"]
    shake = 1.0 + 0.02 * torch.rand(1, generator=g, device=DEV, dtype=torch.float64).item()
    if kind in ("grid2d", "gmrf"):
        kappa2, tau = (0.5 if size <= 64 else 0.1) * shake, 1.5 if kind == "gmrf" else 1.0
        return _stencil([size, size], tau * (4.0 + kappa2), -tau), 0.999 * tau * kappa2, tau * (kappa2 + 8.0)
    if kind == "theta":
        theta = -0.22 / shake
        return _stencil([size, size], 1.0, theta), 1.0 - 4.0 * abs(theta), 1.0 + 4.0 * abs(theta)
    if kind == "grid3d":
        kappa2 = 0.05 * shake
        return _stencil([size] * 3, 6.0 + kappa2, -1.0), 0.999 * kappa2, kappa2 + 12.0
    if kind == "penta":
        n = size
        r = [torch.rand(n, generator=g, device=DEV, dtype=torch.float64) for _ in range(5)]
        s1, s2 = r[1] + r[3], r[2] + r[4]   # (i, i+1) and (i, i+2), mirrored below
        shift = n * shake
        vals = torch.stack([s2.roll(2), s1.roll(1), 2.0 * r[0] + shift, s1, s2], 1)
        idx = torch.arange(n, device=DEV, dtype=torch.int32)
        col = idx[:, None] + torch.arange(-2, 3, device=DEV, dtype=torch.int32)[None, :]
        ok = (col >= 0) & (col < n)
        row_ptr = torch.zeros(n + 1, dtype=torch.int32, device=DEV)
        row_ptr[1:] = ok.sum(1, dtype=torch.int32).cumsum(0, dtype=torch.int32)
        return (row_ptr, col[ok], vals[ok], n), shift - 8.0, shift + 10.0
    if kind == "mesh":
        n = size
        us, vs = [], []
        for off in range(1, MESH_WINDOW + 1):
            u = torch.nonzero(torch.rand(n - off, generator=g, device=DEV) < MESH_DENSITY).flatten()
            us.append(u)
            vs.append(u + off)
        u, v = torch.cat(us), torch.cat(vs)
        w = 0.5 + torch.rand(u.numel(), generator=g, device=DEV, dtype=torch.float64)
        csr, shift = _from_edges(n, u, v, w, 0.5), 0.5
    elif kind == "chunglu":
        n, mean = size, 16.0
        p = (torch.arange(n, device=DEV, dtype=torch.float64) + 1.0) ** (-1.0 / 1.5)
        p = torch.clamp(p * (mean * n / p.sum()), max=math.sqrt(n * mean))
        cdf = torch.cumsum(p / p.sum(), 0)
        edges = int(n * mean // 2)
        a, b = (torch.searchsorted(cdf, torch.rand(edges, generator=g, device=DEV, dtype=torch.float64)).clamp_(max=n - 1)
                for _ in range(2))
        key = torch.unique((torch.minimum(a, b) * n + torch.maximum(a, b))[a != b])
        u = torch.div(key, n, rounding_mode="floor")
        w = 0.5 + torch.rand(key.numel(), generator=g, device=DEV, dtype=torch.float64)
        csr, shift = _from_edges(n, u, key - u * n, w, 0.01), 0.01
    else:
        raise ValueError(kind)
    rows = torch.repeat_interleave(torch.arange(n, device=DEV), csr[0].diff().long())
    top = 2.0 * csr[2][csr[1] == rows].max().item() - shift   # Gershgorin: twice the largest weight sum + shift
    return csr, 0.999 * shift, top


def _block(case, n, seed):
    g = _generator(seed + 1)
    return torch.randn((n, case["cols"]), generator=g, device=DEV, dtype=torch.float64).to(DTYPES[case["dtype"]])


def _tolerance(case, n):
    return (1e-7 if case["dtype"] == "f32" else 1e-10) * math.sqrt(n)


def prepare(case, seed):
    (row_ptr, col_idx, val, n), lmin, lmax = _matrix(case, seed)
    state = dict(case=case, seed=seed, lmin=lmin, lmax=lmax,
                 A=ld.CSR(row_ptr, col_idx, val.to(DTYPES[case["dtype"]]), n))
    if case["entry"].startswith("apply"):
        state["V"] = _block(case, n, seed)
    return state


def run(state):
    c, A = state["case"], state["A"]
    lo, hi, m, seed = state["lmin"], state["lmax"], c["degree"], state["seed"]
    if c["entry"] == "logdet":
        return ld.logdet(A, lo, hi, m, c["cols"], seed)
    if c["entry"] == "logdet_adaptive":
        return ld.logdet_adaptive(A, lo, hi, m, _tolerance(c, A.n), c["cols"], seed)
    if c["entry"] == "logdet_with_grad":
        return ld.logdet_with_grad(A, lo, hi, m, c["cols"], seed)
    if c["entry"] == "apply_log":
        return ld.apply_log(A, lo, hi, m, state["V"])
    if c["entry"] == "apply_log_adaptive":
        return ld.apply_log_adaptive(A, lo, hi, m, _tolerance(c, A.n), state["V"])
    return ld.spectral_bounds(A, m)


# ---- what a pass cannot do without -------------------------------------------------------

def _shape(case):
    """(n, stored entries)"""
    s, kind = case["size"], case["matrix"]
    if kind in ("grid2d", "gmrf", "theta"):
        return s * s, 5 * s * s - 4 * s
    if kind == "grid3d":
        return s**3, 7 * s**3 - 6 * s * s
    if kind == "penta":
        return s, 5 * s - 6
    return s, int(s * (1 + 2 * MESH_WINDOW * MESH_DENSITY)) if kind == "mesh" else 17 * s


def work(case):
    """Inputs read and outputs written once; the products of A with the columns the method needs (the
    quadratic forms take half the degree), the k-column products of the basis and the deflation."""
    n, nnz = _shape(case)
    e = 4 if case["dtype"] == "f32" else 8
    m, cols, entry = case["degree"], case["cols"], case["entry"]
    matrix = nnz * (e + 4) + 4 * (n + 1)
    k = cols // 3
    kg = cols - 2 * k
    dense = 2.0 * n * (4 * k * k + 2 * k * kg)
    if entry == "logdet":
        return dict(bytes=matrix, flops=2.0 * nnz * (m * k + (m + 1) // 2 * (k + kg)) + dense)
    if entry == "logdet_adaptive":   # about half of the degree is used
        return dict(bytes=matrix, flops=2.0 * nnz * (m // 2) * (2 * k + kg) + dense)
    if entry == "logdet_with_grad":
        return dict(bytes=matrix + nnz * e,
                    flops=2.0 * nnz * (3 * m * k + 3 * ((m + 1) // 2) * (k + kg)) + 2.5 * dense)
    if entry == "apply_log":
        return dict(bytes=matrix + 2 * n * cols * e, flops=2.0 * nnz * m * cols)
    if entry == "apply_log_adaptive":
        return dict(bytes=matrix + 2 * n * cols * e, flops=2.0 * nnz * (m // 2) * cols)
    return dict(bytes=matrix, flops=2.0 * nnz * m + 10.0 * n * m)


# ---- the same in FP64, plainly -----------------------------------------------------------

class _Product(torch.autograd.Function):
    """A X for A in CSR with differentiable values."""

    @staticmethod
    def forward(ctx, val, X, rows, cols, row_ptr):
        ctx.save_for_backward(val, X, rows, cols, row_ptr)
        n = row_ptr.numel() - 1
        return torch.sparse_csr_tensor(row_ptr, cols, val, (n, n)) @ X

    @staticmethod
    def backward(ctx, G):
        val, X, rows, cols, row_ptr = ctx.saved_tensors
        n = row_ptr.numel() - 1
        gval = torch.empty_like(val)
        for b in range(0, val.numel(), 4_000_000):
            s = slice(b, b + 4_000_000)
            gval[s] = (G[rows[s]] * X[cols[s]]).sum(1)
        return gval, torch.sparse_csr_tensor(row_ptr, cols, val, (n, n)) @ G, None, None, None   # A is symmetric


def _points(count):
    """Fast Leja points on [-2, 2] (largest product over the midpoints; ties within 1e-12 to the larger)."""
    pts = [2.0, -2.0][:count]
    while len(pts) < count:
        s = np.sort(pts)
        mid = 0.5 * (s[:-1] + s[1:])
        prod = np.ones_like(mid)
        for p in pts:
            prod *= np.abs(mid - p)
        pts.append(float(mid[prod >= prod.max() * (1.0 - 1e-12)].max()))
    return pts


class _Plan:
    def __init__(self, lmin, lmax, degree):
        self.sigma = lmin if lmin < 1.0 else 1.0
        lo, hi = lmin / self.sigma, lmax / self.sigma
        c, gamma = (lo + hi) / 2.0, (hi - lo) / 4.0
        xi = _points(degree + 1)
        with decimal.localcontext() as ctx:
            ctx.prec = max(120, 3 * degree + 60)
            D = decimal.Decimal
            X = [D(x) for x in xi]
            table = [(D(c) + D(gamma) * x).ln() for x in X]
            d = [table[0]]
            for level in range(1, degree + 1):
                table = [(table[j + 1] - table[j]) / (X[j + level] - X[j]) for j in range(len(table) - 1)]
                d.append(table[0])
        self.d = [float(v) for v in d]
        self.alpha, self.beta, self.m = 1.0 / (self.sigma * gamma), [c / gamma + x for x in xi[:degree]], degree

    def apply(self, mul, V):
        W, P = V, self.d[0] * V
        for j in range(self.m):
            W = self.alpha * mul(W) - self.beta[j] * W
            P = P + self.d[j + 1] * W
        return P

    def apply_adaptive(self, mul, V, tol):
        W, P = V, self.d[0] * V
        on = abs(self.d[0]) * W.square().sum(0).sqrt() > tol
        for j in range(self.m):
            if not on.any():
                break
            W = self.alpha * mul(W) - self.beta[j] * W
            P = P + self.d[j + 1] * W * on
            on = on & (abs(self.d[j + 1]) * W.square().sum(0).sqrt() > tol)
        return P


def _signs(seed, stream, n, cols):
    """+-1 entries: the top bit of SplitMix64 output column * n + row + 1 of the stream's key."""
    wrap = lambda x: (x + 2**63) % 2**64 - 2**63   # noqa: E731

    def mix(z):
        for shift, mul in ((30, 0xBF58476D1CE4E5B9), (27, 0x94D049BB133111EB), (31, None)):
            z = z ^ ((z >> shift) & ((1 << (64 - shift)) - 1))
            z = z if mul is None else z * wrap(mul)
        return z

    golden = 0x9E3779B97F4A7C15
    key = mix(torch.tensor([wrap(seed + (stream + 1) * golden)], dtype=torch.int64, device=DEV))
    i = torch.arange(n, dtype=torch.int64, device=DEV) + 1
    out = torch.empty((n, cols), dtype=torch.float64, device=DEV)
    for c in range(cols):
        out[:, c] = torch.where(mix(key + (i + c * n) * wrap(golden)) < 0, -1.0, 1.0)
    return out


def _basis(Y):
    for _ in range(2):   # Cholesky QR, twice
        L = torch.linalg.cholesky(Y.T @ Y)
        Y = Y @ torch.linalg.inv(L).T
    return Y


def _estimate(case, seed, n, plan, apply):
    k = case["cols"] // 3
    kg = case["cols"] - 2 * k
    Q = _basis(apply(_signs(seed, 0, n, k)))
    G = _signs(seed, 1, n, kg)
    U = G - Q @ (Q.T @ G)
    low = (Q * apply(Q)).sum()
    return n * math.log(plan.sigma) + low + (U * apply(U)).sum() / kg


def _lanczos_upper(mul, n, steps, lo, hi):
    v, prev, beta = _signs(0, 2, n, 1) / math.sqrt(n), None, 0.0
    a, b = [], []
    for j in range(min(steps, n)):
        w = mul(v)
        a.append((v * w).sum().item())
        w = w - a[-1] * v - (beta * prev if prev is not None else 0.0)
        beta = w.norm().item()
        if j + 1 == min(steps, n) or beta <= 1e-14 * max(abs(a[-1]), abs(lo), abs(hi)):
            break
        b.append(beta)
        prev, v = v, w / beta
    theta, s = np.linalg.eigh(np.diag(a) + np.diag(b, 1) + np.diag(b, -1))
    return min(hi, theta[-1] + beta * abs(s[-1, -1]))


def exact(case, seed):
    entry = case["entry"]
    if entry == "logdet_with_grad" and _shape(case)[0] * case["degree"] * case["cols"] > 4e9:
        return None
    (row_ptr, col_idx, val, n), lmin, lmax = _matrix(case, seed)
    val = val.to(DTYPES[case["dtype"]]).double()
    rows = torch.repeat_interleave(torch.arange(n, device=DEV), row_ptr.diff().long())
    cols = col_idx.long()
    if entry == "spectral_bounds":
        own = cols == rows
        radius = torch.zeros(n, dtype=torch.float64, device=DEV).index_add_(0, rows[~own], val[~own].abs())
        lo, hi = (val[own] - radius).min().item(), (val[own] + radius).max().item()
    val.requires_grad_(entry == "logdet_with_grad")
    mul = lambda X: _Product.apply(val, X, rows, col_idx, row_ptr)   # noqa: E731
    if entry == "spectral_bounds":
        return lo, _lanczos_upper(mul, n, case["degree"], lo, hi)
    plan = _Plan(lmin, lmax, case["degree"])
    tol = _tolerance(case, n)
    if entry == "apply_log":
        V = _block(case, n, seed).double()
        return plan.apply(mul, V) + math.log(plan.sigma) * V
    if entry == "apply_log_adaptive":
        V = _block(case, n, seed).double()
        return plan.apply_adaptive(mul, V, tol) + math.log(plan.sigma) * V, None
    if entry == "logdet_adaptive":
        return _estimate(case, seed, n, plan, lambda X: plan.apply_adaptive(mul, X, tol)).item(), None
    est = _estimate(case, seed, n, plan, lambda X: plan.apply(mul, X))
    if entry == "logdet":
        return est.item()
    est.backward()
    return est.item(), val.grad
