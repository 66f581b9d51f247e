"""Preconditioned and plain lock-step FP64 COCG (rafeast_pc_solve) at the edges of its
work split: column chunks of 16 and 64 and their remainders, rows longer than a chunk's
lanes, fewer rows than a workgroup's step.  Every system's true residual is recomputed on
the host in FP64; the solver stops at its own FP64 true residual <= tol, and the two
evaluations differ by rounding only (at most a few row lengths of ulps of |z I - A| |x|)."""

import numpy as np
import pytest

from workloads import grid_laplacian, knn_laplacian, random_symmetric

pytestmark = pytest.mark.gpu

CASES = [
    ("tiny", 1, 3), ("tiny", 2, 9), ("dense rows", 3, 5), ("dense rows", 2, 16),
    ("knn", 1, 17), ("knn", 4, 8), ("knn", 3, 43), ("wide", 1, 33), ("wide", 2, 40),
]


def _matrix(name):
    if name == "tiny":
        return random_symmetric(5, seed=3, density=0.6)
    if name == "dense rows":  # rows of 16 to about 100 entries
        return random_symmetric(300, seed=4, density=0.12)
    if name == "knn":
        return knn_laplacian(1501, 2, 10, seed=5, weighted=True, shift=1e-3)
    return grid_laplacian((113, 113), 0.1)  # n > 12288: a wave per row


@pytest.mark.parametrize("name,nz,k", CASES)
@pytest.mark.parametrize("pre", [False, True])
def test_pc_solve_residuals(name, nz, k, pre):
    import torch

    from paper_2512_01257_amd import native

    csr = _matrix(name)
    A = csr.to_scipy()
    rng = np.random.default_rng(7)
    hi = float(abs(A).sum(axis=1).max())
    z = (0.1 + 0.1 * np.arange(nz)) * hi + 1j * (0.2 + 0.1 * np.arange(nz)) * hi
    B = rng.standard_normal((csr.n, k))
    if k > 2:
        B[:, 1] = 0.0  # a system that is done at once
    tol = 1e-10
    with native.Plan(csr, 0.0, 0.5 * hi, min(2, csr.n), nc=2, precision="fp64",
                     p=-1 if csr.n > 20 else 4) as plan:
        info = plan.info()
        lo, up = info["sig_lo"], info["sig_hi"]
        coef = None
        if pre:
            t = np.cos(np.pi * (np.arange(400) + 0.5) / 400)
            x = 0.5 * (up - lo) * t + 0.5 * (up + lo)
            T = np.polynomial.chebyshev.chebvander(t, 7)
            coef = np.stack([np.linalg.lstsq((zj - x)[:, None] * T, np.ones(400, complex),
                                             rcond=None)[0] for zj in z])
        X = torch.zeros((csr.n, nz * k), dtype=torch.complex128, device="cuda")
        it, rs = plan.pc_solve(z, torch.from_numpy(B).cuda(), X, tol, coef=coef)
        Xh = X.cpu().numpy()
    bn = np.linalg.norm(B, axis=0)
    for j in range(nz):
        x = Xh[:, j * k:(j + 1) * k]
        R = B - (z[j] * x - A @ x)
        rel = np.linalg.norm(R, axis=0) / np.where(bn > 0, bn, 1.0)
        assert rel.max() <= tol + 1e-13
        assert np.abs(rel - rs[j * k:(j + 1) * k]).max() <= 1e-13
        if k > 2:
            assert it[j * k + 1] == 0 and not x[:, 1].any()
    assert it.max() > 0
