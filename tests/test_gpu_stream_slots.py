"""The streaming engine keeps the columns that are not done side by side and
moves them together as others finish: shifts that need very different numbers
of iterations, column counts around the unit that moves (8 columns in FP64, 16
in FP32), row counts around a wave's rows, systems that finish at the start,
and a dense operator whose checks multiply the waiting columns alone."""

import numpy as np
import pytest

from workloads import grid_laplacian

pytestmark = pytest.mark.gpu

Z = np.array([0.3 + 1e-3j, 6.0 + 3.0j, 0.5 + 0.1j, 20.0 + 10.0j])  # slow, fast, medium, at once


def check(A, B, X, its, rs, z, tol, u):
    """The engine accepts a column when its FP64 residual meets tol; the output
    rounds the solution once (u) and the residual is recomputed here."""
    n, k = B.shape
    norm_m = np.abs(z).max() + np.abs(A).sum(1).max()
    for j in range(len(z)):
        for c in range(k):
            x, b = X[:, j * k + c], B[:, c]
            if not b.any():
                assert not x.any() and its[j * k + c] == 0
                continue
            assert rs[j * k + c] <= tol
            bound = 1.01 * tol * np.linalg.norm(b) + 2 * u * norm_m * np.linalg.norm(x)
            assert np.linalg.norm(b - (z[j] * x - A @ x)) <= bound


def rhs(n, k, seed):
    B = np.random.default_rng(seed).standard_normal((n, k))
    if k > 2:
        B[:, 1] = 0.0
        B[:, 2] *= 1e-7
    return B


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("dims,k", [((5, 1), 1), ((3, 3), 2), ((31, 33), 4), ((13, 11, 7), 5),
                                    ((32, 32), 8), ((25, 41), 17), ((10, 10, 10), 33)])
def test_columns_move_together(gpu_lib, precision, dims, k):
    import torch

    csr = grid_laplacian(dims, 0.01)
    B = rhs(csr.n, k, k)
    ct, u = (torch.complex64, 2.0 ** -24) if precision == "fp32" else (torch.complex128, 2.0 ** -53)
    m0 = min(4, csr.n - 4)
    with gpu_lib.Plan(csr, 0.0, 0.6, m0, nc=2, q=1, p=4, precision=precision,
                      engine="stream") as plan:
        X = torch.zeros((csr.n, len(Z) * k), dtype=ct, device="cuda")
        its, rs = plan.shifted_solve(Z, torch.from_numpy(B).cuda(), X, 1e-10)
    check(csr.to_scipy().toarray(), B, X.cpu().numpy().astype(complex), its, rs, Z, 1e-10, u)
    if csr.n > 900:
        assert its.max() > 2 * its[3 * k] > 0  # the shifts finish apart


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n,k", [(97, 1), (300, 5), (513, 16), (401, 40)])
def test_dense_columns_move_together(gpu_lib, precision, n, k):
    import torch

    rng = np.random.default_rng(n)
    Q = np.linalg.qr(rng.standard_normal((n, n)))[0]
    K = (Q * np.linspace(0.0, 5.0, n)) @ Q.T
    K = 0.5 * (K + K.T)
    B = rhs(n, k, n)
    z = np.array([1.0 + 5e-3j, 2.0 + 2.0j, 3.0 + 0.2j])
    ct, u = (torch.complex64, 2.0 ** -24) if precision == "fp32" else (torch.complex128, 2.0 ** -53)
    with gpu_lib.Plan.from_dense(K, 1.0, 2.0, 8, nc=2, q=1, p=4,
                                 precision=precision) as plan:
        X = torch.zeros((n, len(z) * k), dtype=ct, device="cuda")
        its, rs = plan.shifted_solve(z, torch.from_numpy(B).cuda(), X, 1e-9)
    check(K, B, X.cpu().numpy().astype(complex), its, rs, z, 1e-9, u)
