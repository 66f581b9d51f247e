"""Forward errors of the direct engine against solutions refined with residuals in
extended precision: as large as those of the same block elimination carried out
with plain sums on the host, on average over graphs and shifts."""

import numpy as np
import pytest
import scipy.sparse as sp
import scipy.sparse.linalg as spla

from oracle.contour import half_circle
from workloads import knn_laplacian

pytestmark = pytest.mark.gpu

K = 32


def _refined(A, z, B):
    """Solutions of (z I - A) X = B to about 1e-17, rounded."""
    lu = spla.splu((z * sp.identity(A.shape[0], format="csc") - A.tocsc()).astype(complex))
    X = lu.solve(B.astype(complex)).astype(np.clongdouble)
    data, ptr = A.data.astype(np.longdouble)[:, None], A.indptr[:-1]
    zr, zi = np.longdouble(z.real), np.longdouble(z.imag)
    for _ in range(4):
        re, im = X.real, X.imag
        ar = np.add.reduceat(data * re[A.indices], ptr, axis=0)
        ai = np.add.reduceat(data * im[A.indices], ptr, axis=0)
        r = (B - (zr * re - zi * im - ar)).astype(float) - 1j * (zr * im + zi * re - ai).astype(float)
        X = X + lu.solve(r)
    return X.astype(complex)


def _block_solve(M, b, B):
    """Block L D L^T with inverses of the 32 x 32 blocks, in the band of M."""
    n, W, inv = len(M), M.copy(), []
    starts = range(0, n, K)
    for c in starts:
        e, r = min(c + K, n), min(n, min(c + K, n) + b)
        inv.append(np.linalg.inv(W[c:e, c:e]))
        W[e:r, e:r] -= (W[e:r, c:e] @ inv[-1]) @ W[e:r, c:e].T
    Y, V = B.astype(complex), np.zeros(B.shape, dtype=complex)
    for i, c in enumerate(starts):
        e, lo = min(c + K, n), max(0, c - b - K)
        Y[c:e] -= W[c:e, lo:c] @ V[lo:c]
        V[c:e] = inv[i] @ Y[c:e]
    X = np.zeros_like(Y)
    for i, c in reversed(list(enumerate(starts))):
        e, r = min(c + K, n), min(n, min(c + K, n) + b)
        X[c:e] = inv[i] @ (Y[c:e] - W[e:r, c:e].T @ X[e:r])
    return X


def test_direct_errors(gpu_lib):
    import torch

    n, k, ratios = 1500, 6, []
    z = half_circle(0.0, 0.05, 4)[0]
    for seed in range(4):
        csr = knn_laplacian(n, 2, 10, seed=seed, weighted=True, shift=1e-3)
        A = csr.to_scipy().tocsr()
        B = np.random.default_rng(seed + 1).standard_normal((n, k))
        with gpu_lib.Plan(csr, 0.0, 0.05, 4, nc=1, q=0, p=4, precision="fp64",
                          engine="direct") as plan:
            X = torch.empty((n, len(z) * k), dtype=torch.complex128, device="cuda")
            plan.shifted_solve(z, torch.from_numpy(B).cuda(), X, 1e-10)
            X = X.cpu().numpy()
        perm = gpu_lib.rcm_order(csr)
        P = A[perm][:, perm].toarray()
        i, j = np.nonzero(P)
        b = int((i - j).max())
        for t, zt in enumerate(z):
            R = _refined(A, zt, B)
            host = np.empty_like(R)
            host[perm] = _block_solve(zt * np.eye(n) - P, b, B[perm])
            err = [np.linalg.norm(Y - R) / np.linalg.norm(R)
                   for Y in (X[:, t * k:(t + 1) * k], host)]
            ratios.append(err[0] / err[1])
    # single ratios scatter between about a half and two
    mean = float(np.exp(np.mean(np.log(ratios))))
    print("ratios", ratios, "mean", mean)
    assert mean <= 1.35, (mean, ratios)
