"""Band factorization and solves of the direct engine at the edges of their blocks of 32:
fewer rows than a block, one row past a block, bands below a block and past the entries
held in registers, odd numbers of right-hand sides.  The reference is a dense complex
solve; the tolerance is that of backward stable elimination, a modest multiple of the
condition number times the unit roundoff (as in the other direct-engine tests)."""

import numpy as np
import pytest
import scipy.sparse as sp

from workloads import csr_from_scipy, grid_laplacian, random_symmetric

pytestmark = pytest.mark.gpu

U = 2.0 ** -53


def _banded(n, b, seed):
    """A symmetric matrix with a full band, so that no ordering narrows it much."""
    rng = np.random.default_rng(seed)
    offs = range(1, min(b, n - 1) + 1)
    L = sp.diags([rng.standard_normal(n - o) for o in offs], [-o for o in offs], shape=(n, n))
    return csr_from_scipy(L + L.T + sp.diags(rng.standard_normal(n) * 4))


CASES = [
    ("dense", 1, 1), ("dense", 20, 3), ("dense", 32, 2), ("dense", 33, 1), ("dense", 97, 5),
    ("band31", 160, 3), ("band32", 161, 2), ("band33", 191, 4), ("band304", 700, 3),
    ("band500", 1100, 1), ("path", 1000, 2), ("grid", 41 * 17, 7),
]


@pytest.mark.parametrize("name,n,k", CASES)
def test_band_solve_edges(gpu_lib, name, n, k):
    import torch

    if name == "dense":
        csr = random_symmetric(n, seed=n, density=0.9)
    elif name == "path":
        csr = grid_laplacian((n,), 0.1)
    elif name == "grid":
        csr = grid_laplacian((41, 17), 0.1)
    else:
        csr = _banded(n, int(name[4:]), n)
    A = csr.to_scipy().toarray()
    lam = np.linalg.eigvalsh(A)
    c = 0.5 * (lam[0] + lam[-1])
    z = np.array([c + 0.2j, lam[0] - 0.5 + 0.5j, c + 2.0 + 5.0j])
    B = np.random.default_rng(1).standard_normal((n, k))
    with gpu_lib.Plan(csr, lam[0] - 1.0, lam[-1] + 1.0, 1, nc=2, precision="fp64",
                      engine="direct") as plan:
        X = torch.zeros((n, len(z) * k), dtype=torch.complex128, device="cuda")
        its, rs = plan.shifted_solve(z, torch.from_numpy(B).cuda(), X, 1e-10)
    Xh = X.cpu().numpy()
    for j, zj in enumerate(z):
        M = zj * np.eye(n) - A
        ref = np.linalg.solve(M, B.astype(complex))
        kappa = np.abs(zj - lam).max() / np.abs(zj - lam).min()
        x = Xh[:, j * k:(j + 1) * k]
        err = np.linalg.norm(x - ref, axis=0) / np.linalg.norm(ref, axis=0)
        rel = np.linalg.norm(B - M @ x, axis=0) / np.linalg.norm(B, axis=0)
        assert err.max() <= 1e3 * kappa * U + 1e-14, (j, err, kappa)
        assert np.abs(rel - rs[j * k:(j + 1) * k]).max() <= 1e3 * kappa * U
