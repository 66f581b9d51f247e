"""Performance cases of the RA-FEAST library: what a program calls, at the sizes it calls it with.

A case is a dict of plain values.  `kind` names the call:

  spmm     Plan.spmm             the FP64 operator product of Phase 1 and of Rayleigh-Ritz
  power    Plan.spmm + cholqr2   one power step of Phase 1: operator application, orthonormalisation
  syev     Plan.syev             the reduced eigenproblem of Rayleigh-Ritz
  gemm     gemm                  the dense operators' product
  solve    warmstart + solve     a whole eigensolve of a sparse matrix
  kernel   warmstart + solve     a whole eigensolve of a dense kernel matrix (kernel PCA)
  shifted  Plan.shifted_solve    the shifted systems of one filter application
  pc       Plan.pc_solve         the same with a polynomial preconditioner

Matrices: k-nearest-neighbour graph Laplacians (2D with 10 neighbours, 3D with 16, Gaussian
weights, + 1e-3 I), random geometric graph Laplacians, 7-point grid Laplacians and Gaussian
kernel matrices, the families of the benchmark and of the tests, drawn anew for each seed.
"""

from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2512_01257_amd import native

# Smallest eigenvalues of the graph families grow as 1e-3 + c (j / n)^(2 / dim); c measured on
# graphs of 1,000 to 12,000 points.
GROWTH = {"knn2d": 9.4, "knn3d": 13.0}
DEGREE = {"knn2d": 12.4, "knn3d": 19.2, "rgg": 67.0, "grid3d": 6.94}  # nonzeros per row


def listed():
    return [
        # Rayleigh-Ritz product W = A Q on a 100^3 grid: the benchmark's SpMM, the largest block
        dict(name="spmm grid 1e6 x 64", kind="spmm", graph="grid3d", n=1_000_000, k=64),
        # a Phase-1 power step of the headline eigensolve (m0 = 64, p = 20): latency counts
        dict(name="power knn 8000 x 84", kind="power", graph="knn2d", n=8000, k=84),
        # the same step at n = 1e6, where the tall-skinny products stream from memory
        dict(name="power grid 1e6 x 84", kind="power", graph="grid3d", n=1_000_000, k=84),
        # Rayleigh-Ritz at the end of Phase 1: a full reduced matrix of m0 + p = 84
        dict(name="syev 84", kind="syev", k=84, mix=1.0),
        # a dense operator's product inside FP32 COCG: K (8192) times 8 shifts x 30 columns, re and im
        dict(name="gemm f32 8192 x 480", kind="gemm", m=8192, n=480, k=8192, a_cols=True, dtype="float32"),
        # the smallest whole eigensolve: one small graph, a few eigenpairs; launches and waits count
        dict(name="solve knn 1000", kind="solve", graph="knn2d", n=1000, m0=24, nc=4, q=2, engine="auto",
             precision="fp32"),
        # the headline eigensolve: 50 eigenpairs of a graph of 8,000 points
        dict(name="solve knn 8000", kind="solve", graph="knn2d", n=8000, m0=64, nc=4, q=2, engine="auto",
             precision="fp32"),
        # a larger graph with FP64 solves, as the batching form runs its larger members
        dict(name="solve knn3d 30000 f64", kind="solve", graph="knn3d", n=30000, m0=64, nc=4, q=1,
             engine="multishift", precision="fp64"),
        # kernel PCA: leading eigenpairs of a Gaussian kernel matrix
        dict(name="kernel 4096", kind="kernel", n=4096, m0=30, nc=16, q=2),
        # one filter application past the on-chip engine's size, dense rows: the paper's largest graph
        dict(name="shifted rgg 16000 f32", kind="shifted", graph="rgg", n=16000, k=40, nc=4, engine="stream",
             precision="fp32"),
        # exact solves: factorizations and substitutions for the nodes of one window
        dict(name="shifted knn 8000 direct", kind="shifted", graph="knn2d", n=8000, k=64, nc=8, engine="direct",
             precision="fp64"),
        # one filter application with a polynomial preconditioner
        dict(name="pc knn 8000", kind="pc", graph="knn2d", n=8000, k=32, nc=4),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("spmm", "power", "syev", "gemm", "solve", "solve", "kernel", "shifted", "shifted", "shifted", "pc"))
    if kind in ("spmm", "power"):
        graph = rng.choice(("knn2d", "knn3d", "grid3d"))
        k = rng.randint(9, 148)
        n = _log(rng, 1500, 60_000 if graph != "grid3d" else min(1_000_000, 64_000_000 // k))
        if graph == "grid3d":
            n = max(12, round(n ** (1 / 3))) ** 3
        return dict(kind=kind, graph=graph, n=n, k=k)
    if kind == "syev":
        return dict(kind=kind, k=rng.randint(8, 148), mix=rng.choice((1.0, 1e-2)))
    if kind == "gemm":
        a_cols = rng.random() < 0.5
        m, k = _log(rng, 500, 8192), _log(rng, 500, 8192)
        return dict(kind=kind, m=m, n=rng.randint(16, 480), k=k, a_cols=a_cols,
                    dtype=rng.choice(("float32", "float64")))
    if kind == "solve":
        engine = rng.choice(("auto", "auto", "multishift", "direct"))
        graph = "knn2d" if engine == "direct" else rng.choice(("knn2d", "knn3d"))
        n = _log(rng, 700, 8000 if engine == "auto" else 16000)
        return dict(kind=kind, graph=graph, n=n, m0=rng.randint(16, 64), nc=rng.choice((2, 4, 8)), q=rng.randint(1, 2),
                    engine=engine, precision="fp64" if engine != "auto" or n < 4000 and rng.random() < 0.5 else "fp32")
    if kind == "kernel":
        return dict(kind=kind, n=_log(rng, 700, 4096), m0=rng.randint(28, 36), nc=16, q=rng.randint(1, 2))
    if kind == "shifted":
        engine = rng.choice(("auto", "stream", "multishift", "direct"))
        graph = rng.choice(("knn2d", "rgg") if engine == "direct" else ("knn2d", "knn3d", "rgg"))
        n = _log(rng, 700, dict(auto=8000, stream=16000, multishift=16000, direct=8000)[engine])
        precision = "fp32" if engine == "auto" else rng.choice(("fp32", "fp64")) if engine == "stream" else "fp64"
        return dict(kind=kind, graph=graph, n=n, k=rng.randint(5, 40), nc=rng.choice((2, 4)), engine=engine,
                    precision=precision)
    return dict(kind="pc", graph=rng.choice(("knn2d", "knn3d")), n=_log(rng, 700, 8000), k=rng.randint(5, 32),
                nc=rng.choice((2, 4)))


# ---------------------------------------------------------------------------- inputs

def _generator(seed, what):
    return torch.Generator().manual_seed(1_000_003 * (int(seed) % 1_000_003) + what)


def _csr(n, i, j, v):
    """CSR arrays on the host from unique (row, column, value) triples on the GPU."""
    order = torch.argsort(i * n + j)
    i, j, v = i[order], j[order], v[order]
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device=i.device)
    rowptr[1:] = torch.cumsum(torch.bincount(i, minlength=n), 0)
    return SimpleNamespace(n=n, rowptr=rowptr.to(torch.int32).cpu().numpy(), colind=j.to(torch.int32).cpu().numpy(),
                           values=v.cpu().numpy())


def _laplacian(n, a, b, w, shift):
    """D - W + shift I of the undirected edges a < b."""
    i, j = torch.cat((a, b)), torch.cat((b, a))
    ww = torch.cat((w, w))
    deg = torch.zeros(n, dtype=torch.float64).index_add_(0, i.cpu(), ww.cpu()).to(i.device)
    d = torch.arange(n, device=i.device)
    return _csr(n, torch.cat((i, d)), torch.cat((j, d)), torch.cat((-ww, deg + shift)))


def _matrix(graph, n, seed):
    if graph == "grid3d":  # 7-point Dirichlet Laplacian, the seed in the diagonal shift
        m = round(n ** (1 / 3))
        idx = torch.arange(n, device="cuda")
        x, y, z = idx // (m * m), idx // m % m, idx % m
        parts = [(idx, idx, torch.full((n,), 6.0 + 1e-3 * (1 + int(seed) % 97), dtype=torch.float64, device="cuda"))]
        for c, s in ((x, m * m), (y, m), (z, 1)):
            up = idx[c < m - 1]
            e = torch.full((len(up),), -1.0, dtype=torch.float64, device="cuda")
            parts += [(up, up + s, e), (up + s, up, e)]
        return _csr(n, *(torch.cat(p) for p in zip(*parts)))
    dim = 3 if graph == "knn3d" else 2
    pts = torch.rand((n, dim), generator=_generator(seed, 1), dtype=torch.float64).cuda()
    step = max(1, 40_000_000 // n)
    if graph == "rgg":
        r = 1.5 * math.sqrt(math.log(n) / n)
        pairs = [torch.nonzero(torch.cdist(pts[s:s + step], pts) < r) + torch.tensor([s, 0], device="cuda")
                 for s in range(0, n, step)]
        a, b = torch.cat(pairs).T
        keep = a < b
        a, b = a[keep], b[keep]
        return _laplacian(n, a, b, torch.ones(len(a), dtype=torch.float64, device="cuda"), 0.0)
    kk = 16 if graph == "knn3d" else 10
    near = [torch.topk(torch.cdist(pts[s:s + step], pts), kk + 1, largest=False) for s in range(0, n, step)]
    j = torch.cat([t.indices[:, 1:] for t in near]).reshape(-1)
    sigma = float(torch.cat([t.values[:, 1:] for t in near]).reshape(-1).median())
    i = torch.arange(n, device="cuda").repeat_interleave(kk)
    key = torch.unique(torch.minimum(i, j) * n + torch.maximum(i, j))
    a, b = key // n, key % n
    keep = a != b
    a, b = a[keep], b[keep]
    w = torch.exp(-((pts[a] - pts[b]) ** 2).sum(1) / sigma ** 2)
    return _laplacian(n, a, b, w, 1e-3)


def _window(case, count):
    """A window [0, u] with about `count` eigenvalues of a neighbour graph; [0, 5] of a geometric graph."""
    if case["graph"] == "rgg":
        return 0.0, 5.0
    d = 3 if case["graph"] == "knn3d" else 2
    return 0.0, 1e-3 + GROWTH[case["graph"]] * (count / case["n"]) ** (2 / d)


def _block(rows, cols, seed, what=2, dtype=torch.float64):
    return torch.randn((rows, cols), generator=_generator(seed, what), dtype=dtype).cuda()


def _reduced(case, seed):
    """A symmetric matrix with a spread spectrum: rotated fully (mix 1), or nearly diagonal as in
    the later Rayleigh-Ritz steps (mix << 1)."""
    k = case["k"]
    g = torch.randn((k, k), generator=_generator(seed, 3), dtype=torch.float64)
    jitter = torch.rand(k, generator=_generator(seed, 4), dtype=torch.float64)
    lam = (torch.arange(k, dtype=torch.float64) + 1 + 0.5 * jitter) / k
    q = torch.linalg.qr(g if case["mix"] == 1.0 else torch.eye(k, dtype=torch.float64) + case["mix"] * g / math.sqrt(k))[0]
    h = (q * lam) @ q.T
    return (0.5 * (h + h.T)).cuda()


def _kernel(case, seed):
    """Gaussian kernel matrix of a mixture of six clusters in the unit cube."""
    n = case["n"]
    centres = torch.rand((6, 3), generator=_generator(seed, 5), dtype=torch.float64)
    x = centres[torch.randint(0, 6, (n,), generator=_generator(seed, 6))]
    x = (x + 0.15 * torch.randn((n, 3), generator=_generator(seed, 7), dtype=torch.float64)).cuda()
    d2 = (x * x).sum(1)[:, None] + (x * x).sum(1)[None, :] - 2.0 * (x @ x.T)
    k = torch.exp(-torch.clamp(0.5 * (d2 + d2.T), min=0.0) / 0.32)
    k.fill_diagonal_(1.0)
    return 0.5 * (k + k.T)


def _operands(case, seed):
    dt = getattr(torch, case["dtype"])
    a = _block(case["k"], case["m"], seed, 8, dt) if case["a_cols"] else _block(case["m"], case["k"], seed, 8, dt)
    return a, _block(case["k"], case["n"], seed, 9, dt)


def _kernel_window(a):
    """From 0.6% of the trace to above the largest eigenvalue."""
    n = a.shape[0]
    v = torch.ones((n, 1), dtype=torch.float64, device=a.device)
    for _ in range(60):
        v = a @ (v / v.norm())
    return 0.006 * n, 1.05 * float(v.norm())


def _count(case):
    return case["m0"] * 3 // 4 if case["kind"] == "solve" else case["k"] * 3 // 4


def _gersh(csr):
    """The Gershgorin interval."""
    row = np.repeat(np.arange(csr.n), np.diff(csr.rowptr))
    diag = csr.values[row == csr.colind]
    r = np.bincount(row, weights=np.abs(csr.values), minlength=csr.n) - np.abs(diag)
    return float((diag - r).min()), float((diag + r).max())


def _coefficients(csr, z):
    """Coefficients of the degree-7 Chebyshev polynomials p_j(A) that leave the least residual
    1 - (z_j - x) p_j(x) over the Gershgorin interval."""
    lo, hi = _gersh(csr)
    t = np.cos(np.pi * (np.arange(600) + 0.5) / 600)
    x = 0.5 * (hi - lo) * t + 0.5 * (hi + lo)
    T = np.polynomial.chebyshev.chebvander(t, 7)
    return np.stack([np.linalg.lstsq((zj - x)[:, None] * T, np.ones(600, dtype=complex), rcond=None)[0] for zj in z])


# ---------------------------------------------------------------------------- the calls

TOL = {"fp32": 1e-8, "fp64": 1e-11}  # relative residual of the step-level solves


def prepare(case, seed):
    s = SimpleNamespace(case=case)
    kind = case["kind"]
    if kind == "syev":
        s.plan = _step_plan()
        s.h = _reduced(case, seed)
        s.theta, s.s = torch.empty(case["k"], dtype=torch.float64, device="cuda"), torch.empty_like(s.h)
        return s
    if kind == "gemm":
        s.a, s.b = _operands(case, seed)
        s.c = torch.empty((case["m"], case["n"]), dtype=s.a.dtype, device="cuda")
        return s
    if kind == "kernel":
        a = _kernel(case, seed)
        lo, hi = _kernel_window(a)
        s.plan = native.Plan.from_dense(a.cpu().numpy(), lo, hi, case["m0"], nc=case["nc"], q=case["q"],
                                        ws_op="literal", max_iter=40, seed=int(seed) % 1000)
    else:
        csr = _matrix(case["graph"], case["n"], seed)
        kw = dict(seed=int(seed) % 1000)
        if kind in ("spmm", "power"):
            lo, hi, m0 = 0.0, 1.0, 8
            kw.update(nc=1, engine="multishift", precision="fp64")
        else:
            lo, hi = _window(case, _count(case))
            m0 = case.get("m0", 8)
            kw.update(nc=case["nc"], engine=case.get("engine", "auto"), precision=case.get("precision", "fp64"))
            if kind == "solve":
                kw.update(q=case["q"], max_iter=40)
        s.plan = native.Plan(csr, lo, hi, m0, **kw)
    n = case["n"]
    if kind in ("spmm", "power"):
        s.x = _block(n, case["k"], seed)
        s.y = torch.empty_like(s.x)
    elif kind in ("solve", "kernel"):
        # room for m0 pairs; those past the number found stay zero
        s.lam = torch.zeros(case["m0"], dtype=torch.float64, device="cuda")
        s.res = torch.zeros_like(s.lam)
        s.x = torch.zeros((case["m0"], n), dtype=torch.float64, device="cuda")
    else:
        s.z = _nodes(lo, hi, case["nc"])
        s.b = _block(n, case["k"], seed)
        wide = torch.complex64 if case.get("precision", "fp64") == "fp32" else torch.complex128
        s.x = torch.empty((n, len(s.z) * case["k"]), dtype=wide, device="cuda")
        if kind == "pc":
            s.coef = _coefficients(csr, s.z)
    return s


def _step_plan():
    n = 256  # a plan's handle for the calls that use no matrix
    i = torch.arange(n)
    return native.Plan(_csr(n, i, i, torch.linspace(1.0, 2.0, n, dtype=torch.float64)), 0.0, 1.5, 8, nc=1)


def run(s):
    kind = s.case["kind"]
    if kind == "spmm":
        s.plan.spmm(s.x, s.y)
        return s.y
    if kind == "power":  # C = I - A / s, as the flip operator of a bottom window
        s.plan.spmm(s.x, s.y, alpha=-0.07, beta=1.0)
        s.plan.cholqr2(s.y)
        return s.y
    if kind == "syev":
        s.plan.syev(s.h, s.theta, s.s)
        return s.theta, s.s
    if kind == "gemm":
        native.gemm(s.a, s.b, s.c, a_cols=s.case["a_cols"])
        return s.c
    if kind in ("solve", "kernel"):
        s.plan.warmstart()
        out = s.plan.solve_device(s.lam, s.res, s.x)
        return out["M"], s.lam, s.x
    if kind == "shifted":
        s.plan.shifted_solve(s.z, s.b, s.x, TOL[s.case["precision"]])
        return s.x
    s.plan.pc_solve(s.z, s.b, s.x, TOL["fp64"], coef=s.coef)
    return s.x


# ---------------------------------------------------------------------------- bytes and operations

def work(case):
    kind = case["kind"]
    if kind == "syev":  # read H, write theta and S; tridiagonal reduction and eigenvectors: about 9 k^3
        k = case["k"]
        return {"bytes": 8 * (2 * k * k + k), "flops": 9 * k ** 3}
    if kind == "gemm":
        m, n, k, e = case["m"], case["n"], case["k"], 4 if case["dtype"] == "float32" else 8
        return {"bytes": e * (m * k + k * n + m * n), "flops": 2 * m * n * k}
    n = case["n"]
    if kind == "kernel":  # some 10 filter applications, in each some 5 products with K for a complex column
        return {"bytes": 8 * n * n + 8 * n * case["m0"], "flops": 4 * n * n * 10 * case["nc"] * case["m0"] * 5}
    nnz = DEGREE[case["graph"]] * n
    mat = 12 * nnz + 4 * (n + 1)
    if kind in ("spmm", "power"):
        k = case["k"]
        # CholQR2: twice a symmetric Gram matrix and a product with a triangle
        return {"bytes": mat + 16 * n * k, "flops": 2 * nnz * k + (4 * n * k * k if kind == "power" else 0)}
    # Krylov iterations of a shift at distance d from the spectrum: 1/2 sqrt(norm / d) ln(2 / tol)
    lo, hi = _window(case, _count(case))
    norm = {"knn2d": 12.0, "knn3d": 16.0, "rgg": 130.0}[case["graph"]]
    theta = math.pi / (2 * case["nc"])
    its = 0.5 * math.sqrt(norm / (0.5 * (hi - lo) * math.sin(theta)))
    if kind == "solve":
        m0, rounds = case["m0"], 6 if case["nc"] <= 4 else 4
        cols = case["nc"] * m0
        return {"bytes": mat + 8 * n * m0, "flops": rounds * cols * its * math.log(2e6) / 2 * (4 * nnz + 30 * n)}
    cols = case["nc"] * case["k"]
    out = (8 if case.get("precision") == "fp32" else 16) * n * cols
    if case.get("engine") == "direct":  # band L D L^T, complex: band width about 2.9 sqrt(n)
        b = 2.9 * math.sqrt(n) * (1 if case["graph"] == "knn2d" else 2.5)
        return {"bytes": mat + 8 * n * case["k"] + out, "flops": case["nc"] * 4 * n * b * b + cols * 16 * n * b}
    return {"bytes": mat + 8 * n * case["k"] + out,
            "flops": cols * its * math.log(2 / TOL[case.get("precision", "fp64")]) / 2 * (4 * nnz + 30 * n)}


# ---------------------------------------------------------------------------- the same in plain torch, 64 bits

def _sparse(csr):
    return torch.sparse_csr_tensor(torch.from_numpy(csr.rowptr.astype(np.int64)), torch.from_numpy(csr.colind.astype(np.int64)),
                                   torch.from_numpy(csr.values), (csr.n, csr.n)).cuda()


def _nodes(lo, hi, nc):
    """Gauss-Legendre nodes on the upper half circle over [lo, hi], by increasing imaginary part."""
    t = np.polynomial.legendre.leggauss(nc)[0]
    z = 0.5 * (lo + hi) + 0.5 * (hi - lo) * np.exp(0.5j * math.pi * (1 + t))
    return z[np.argsort(np.abs(z.imag), kind="stable")]


def _cocg(csr, z, b):
    """(z I - A)^{-1} b by conjugate orthogonal conjugate gradients in complex128, all columns at once."""
    a = _sparse(csr)
    r = torch.complex(b, torch.zeros_like(b))
    x, p = torch.zeros_like(r), r.clone()
    rho, stop, best = (r * r).sum(0), 1e-14 * b.norm(dim=0), math.inf
    for it in range(6000):
        w = z * p - torch.complex(a @ p.real.contiguous(), a @ p.imag.contiguous())
        alpha = rho / (p * w).sum(0)
        alpha = torch.where(torch.isfinite(alpha.abs()), alpha, torch.zeros_like(alpha))
        x += alpha * p
        r -= alpha * w
        new = (r * r).sum(0)
        beta = new / rho
        p = r + torch.where(torch.isfinite(beta.abs()), beta, torch.zeros_like(beta)) * p
        rho = new
        if it % 25 == 24:
            if bool((r.abs().square().sum(0).sqrt() <= stop).all()):
                break
    return x


def _smallest(csr, lo, hi, count):
    """Eigenpairs in [lo, hi] at the bottom of a positive definite matrix: inverse subspace iteration."""
    a = _sparse(csr).to_dense()
    chol = torch.linalg.cholesky(a)
    q = torch.linalg.qr(_block(csr.n, min(csr.n, 2 * count + 40), 1, 10))[0]
    last = None
    for _ in range(80):
        q = torch.linalg.qr(torch.cholesky_solve(q, chol))[0]
        lam, u = torch.linalg.eigh((lambda h: 0.5 * (h + h.T))(q.T @ (a @ q)))
        q = q @ u
        inside = (lam >= lo) & (lam <= hi)
        res = float((a @ q - q * lam)[:, inside].norm())
        if last is not None and res > 0.5 * last and res < 1e-10:
            break
        last = res
    return lam[inside], q[:, inside]


def _largest(a, lo):
    q = torch.linalg.qr(_block(a.shape[0], min(a.shape[0], 120), 1, 10))[0]
    for _ in range(60):
        q = torch.linalg.qr(a @ q)[0]
    lam, u = torch.linalg.eigh((lambda h: 0.5 * (h + h.T))(q.T @ (a @ q)))
    return lam[lam >= lo], (q @ u)[:, lam >= lo]


def _pairs(m0, lam, q):
    """Eigenvalues and unit eigenvectors as rows, the largest entry of each positive, and zeros up to m0."""
    x = (q / q.norm(dim=0)).T.contiguous()
    big = x.gather(1, x.abs().argmax(1, keepdim=True))
    full, rows = torch.zeros(m0, dtype=torch.float64), torch.zeros((m0, x.shape[1]), dtype=torch.float64)
    full[:len(lam)], rows[:len(lam)] = lam.cpu(), (x * torch.sign(big)).cpu()
    return len(lam), full, rows


def exact(case, seed):
    kind, n = case["kind"], case.get("n")
    if kind == "syev":  # an eigenvector's sign is free
        return torch.linalg.eigvalsh(_reduced(case, seed).cpu()), None
    if kind == "gemm":
        a, b = _operands(case, seed)
        return (a.double().T if case["a_cols"] else a.double()) @ b.double()
    if kind == "kernel":
        a = _kernel(case, seed)
        return _pairs(case["m0"], *_largest(a, _kernel_window(a)[0]))
    csr = _matrix(case["graph"], n, seed)
    if kind in ("spmm", "power"):
        x = _block(n, case["k"], seed)
        ax = _sparse(csr) @ x
        if kind == "spmm":
            return ax
        y = x - 0.07 * ax
        for _ in range(3):  # the orthonormal factor whose triangle has a positive diagonal
            r = torch.linalg.cholesky(y.T @ y)
            y = y @ torch.linalg.inv(r).T.contiguous()
        return y
    lo, hi = _window(case, _count(case))
    if kind == "solve":
        return None if n > 12000 else _pairs(case["m0"], *_smallest(csr, lo, hi, _count(case)))
    b = _block(n, case["k"], seed)
    return torch.cat([_cocg(csr, complex(z), b) for z in _nodes(lo, hi, case["nc"])], dim=1)
