"""The GEMM's split of the inner dimension: lengths around the smallest chunks
and around the length from which chunks are longer, few and many output tiles,
covariance operators whose rows are not whole vectors."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("a_cols", [False, True])
@pytest.mark.parametrize("shape", [(130, 33, 127), (130, 33, 128), (257, 100, 255), (64, 7, 256),
                                   (883, 131, 883), (700, 480, 1023), (129, 65, 2559),
                                   (129, 65, 2560), (515, 20, 5000)])
def test_split_products(gpu_lib, dtype, a_cols, shape):
    import torch

    M, N, K = shape
    rng = np.random.default_rng(M + N + K)
    A = rng.standard_normal((K, M) if a_cols else (M, K)).astype(dtype)
    B = rng.standard_normal((K, N)).astype(dtype)
    C0 = rng.standard_normal((M, N)).astype(dtype)
    C = torch.tensor(C0, device="cuda")
    gpu_lib.gemm(torch.tensor(A, device="cuda"), torch.tensor(B, device="cuda"), C, alpha=0.75,
                 beta=-1.25, a_cols=a_cols)
    opA = (A.T if a_cols else A).astype(np.float64)
    B64, u = B.astype(np.float64), np.finfo(dtype).eps / 2
    want = 0.75 * (opA @ B64) - 1.25 * C0
    # any order of a sum of K products
    bound = (K + 4) * u * (0.75 * np.abs(opA) @ np.abs(B64) + 1.25 * np.abs(C0))
    assert (np.abs(C.cpu().numpy().astype(np.float64) - want) <= bound).all()


@pytest.mark.parametrize("rows,n", [(61, 130), (203, 97), (130, 1031)])
def test_covariance_with_odd_rows(gpu_lib, rows, n):
    import torch

    X = np.random.default_rng(rows).standard_normal((rows, n))
    A = X.T @ X / (rows - 1)
    B = np.random.default_rng(n).standard_normal((n, 3))
    lam = np.linalg.eigvalsh(A)
    z = np.array([0.5 * lam[-1] + 0.2j * lam[-1], lam[-1] + 1.0j])
    with gpu_lib.Plan.from_covariance(X, 0.5 * lam[-1], 1.1 * lam[-1], 8, nc=2, q=1, p=4,
                                      precision="fp64") as plan:
        Xd = torch.zeros((n, 6), dtype=torch.complex128, device="cuda")
        its, rs = plan.shifted_solve(z, torch.from_numpy(B).cuda(), Xd, 1e-10)
    x = Xd.cpu().numpy()
    assert rs.max() <= 1e-10
    for j in range(2):
        for c in range(3):
            v = x[:, 3 * j + c]
            r = B[:, c] - (z[j] * v - A @ v)
            bound = 1.01e-10 * np.linalg.norm(B[:, c]) + 1e-13 * abs(z[j]) * np.linalg.norm(v)
            assert np.linalg.norm(r) <= bound
