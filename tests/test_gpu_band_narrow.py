"""The direct engine's factors of bands below 31 at their own width (matrices whose
widened factors would take more than 32 GiB): the kernels at the edges of their
blocks against dense solves, and the engine on both sides of the line."""

import ctypes as C

import numpy as np
import pytest
import scipy.sparse as sp

from workloads import csr_from_scipy

pytestmark = pytest.mark.gpu

U = 2.0 ** -53


def _calls(gpu_lib):
    """band_factor and band_solve of the library (C++ functions)."""
    L = gpu_lib.lib()
    factor = L["_ZN7rafeast11band_factorEP12ihipStream_tiiiPNS_3cpxIdEEPi"]
    solve = L["_ZN7rafeast10band_solveEP12ihipStream_tiiiPKNS_3cpxIdEEPKiPKdiiPS3_l"]
    p, i = C.c_void_p, C.c_int
    factor.argtypes, solve.argtypes = [p, i, i, i, p, p], [p, i, i, i, p, p, p, i, i, p, C.c_int64]
    return factor, solve


def _bands(A, z, b):
    """W[j][r][d] = (z_j I - A)(r, r - d)."""
    n = len(A)
    W = np.zeros((len(z), n, b + 1), dtype=complex)
    for d in range(min(b, n - 1) + 1):
        W[:, d:, d] = -np.diagonal(A, -d)
    W[:, :, 0] += np.asarray(z)[:, None]
    return W


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 32, 33, 130])
@pytest.mark.parametrize("b", [0, 1, 2, 7, 8, 29, 30])
def test_narrow_kernels(gpu_lib, n, b):
    import torch

    factor, solve = _calls(gpu_lib)
    rng = np.random.default_rng(100 * n + b)
    A = rng.standard_normal((n, n))
    A = np.tril(np.triu(A, -b), b)
    A = A + A.T
    z = np.array([0.3 + 0.7j, -1.0 - 0.5j, 0.2 + 2.0j])
    perm = rng.permutation(n).astype(np.int32)
    W = torch.from_numpy(_bands(A, z, b)).cuda()
    info = torch.full((3,), -1, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    assert factor(None, n, b, 3, W.data_ptr(), info.data_ptr()) == 0
    pd = torch.from_numpy(perm).cuda()
    for k in (1, 2, 64, 65):
        Bm = rng.standard_normal((n, k))
        x = torch.full((n, 3 * k), float("nan"), dtype=torch.complex128, device="cuda")
        bd = torch.from_numpy(Bm).cuda()
        torch.cuda.synchronize()
        assert solve(None, n, b, 3, W.data_ptr(), pd.data_ptr(), bd.data_ptr(), k, k, x.data_ptr(),
                     3 * k) == 0
        torch.cuda.synchronize()
        assert info.cpu().tolist() == [0, 0, 0]
        X = x.cpu().numpy()
        for j, zj in enumerate(z):
            M = zj * np.eye(n) - A
            # row r of the matrix is row perm[r] of the blocks
            want = np.empty((n, k), dtype=complex)
            want[perm] = np.linalg.solve(M, Bm[perm].astype(complex))
            err = np.linalg.norm(X[:, j * k:(j + 1) * k] - want) / np.linalg.norm(want)
            assert err <= 1e3 * np.linalg.cond(M) * U, (j, k, err)


def test_narrow_vanishing_pivot(gpu_lib):
    import torch

    factor, _ = _calls(gpu_lib)
    n, b = 50, 3
    A = np.diag(np.arange(1.0, n + 1))
    W = torch.from_numpy(_bands(A, [37.0, 0.5j], b)).cuda()
    info = torch.full((2,), -1, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    assert factor(None, n, b, 2, W.data_ptr(), info.data_ptr()) == 0
    torch.cuda.synchronize()
    assert info.cpu().tolist() == [37, 0]


def test_both_sides_of_the_line(gpu_lib):
    # 64 shifts of 2^20 rows at b = 31 take 32 GiB, one row more takes more
    import torch

    n, k = 1_048_577, 1
    r = np.random.default_rng(1)
    e1, e2 = r.standard_normal(n - 1), r.standard_normal(n - 2)
    A = sp.diags([e2, e1, r.uniform(1, 5, n), e1, e2], [-2, -1, 0, 1, 2]).tocsr()
    z = 1.0 + 0.8 * np.exp(1j * np.pi * (np.arange(64) + 0.5) / 64)
    B = r.standard_normal((n, k))
    free = torch.cuda.mem_get_info()[0]
    with gpu_lib.Plan(csr_from_scipy(A), 0.0, 2.0, 4, nc=64, q=0, p=4, precision="fp64",
                      engine="direct") as plan:
        # the plan's factors: 64 n (b + 1) numbers of 16 bytes, b <= 4 in the
        # reverse Cuthill-McKee order, and blocks of 64 x 4 columns
        assert free - torch.cuda.mem_get_info()[0] <= 64 * n * 5 * 16 + 64 * 4 * n * 16 + 1e9
        b = torch.from_numpy(B).cuda()
        X = torch.empty((n, 64 * k), dtype=torch.complex128, device="cuda")
        plan.shifted_solve(z, b, X, 1e-10)
        Y = torch.empty((n, 63 * k), dtype=torch.complex128, device="cuda")
        _, rs = plan.shifted_solve(z[:63], b, Y, 1e-10)
    # |z - lambda| >= Im z_j >= 0.019, ||z I - A|| <= 30: kappa <= 1,600
    assert rs.max() <= 1e3 * 1600 * U
    diff = (X[:, :63 * k] - Y).abs().max().item()
    assert diff <= 1e3 * 1600 * U * Y.abs().max().item()
    for j in (0, 31, 63):
        x = X[:, j * k:(j + 1) * k].cpu().numpy()
        res = B - (z[j] * x - A @ x)
        assert np.linalg.norm(res) <= 1e3 * 1600 * U * np.linalg.norm(B)
