"""The SpMM on both sides of the lines between its forms: widths around 64, 120,
128 and 192 on rows of a few and of many entries, and narrow blocks on few and
many rows, against a host product."""

import numpy as np
import pytest
import scipy.sparse as sp

from workloads import csr_from_scipy

pytestmark = pytest.mark.gpu


def _band(n, half, seed):
    """Rows of 2 half + 1 entries within 4 half + 1 of the diagonal, a short first row."""
    r = np.random.default_rng(seed)
    i = np.repeat(np.arange(1, n), half)
    j = np.clip(i + r.integers(1, 4 * half + 2, len(i)), 0, n - 1)
    A = sp.coo_matrix((r.standard_normal(len(i)), (i, j)), (n, n)).tocsr()
    A = A + A.T + sp.diags(r.uniform(1, 2, n))
    A.sum_duplicates()
    A.sort_indices()
    return A.tocsr()


@pytest.mark.parametrize("n,half,ks", [
    (16500, 1, (65, 119, 121, 129, 191, 193)), (16500, 3, (65, 129, 159)),
    (16500, 9, (129, 137, 177, 179)), (16384, 1, (129, 161)), (16384, 9, (2, 3, 8, 15, 17)),
    (16385, 9, (2, 3, 8, 15, 17)), (700, 30, (1, 2, 3, 4, 5, 6, 7, 9))])
def test_spmm_forms(gpu_lib, n, half, ks):
    import torch

    A = _band(n, half, n + half)
    csr = csr_from_scipy(A)
    absA, most = abs(A), np.diff(A.indptr).max()
    with gpu_lib.Plan(csr, 0.0, 1.0, 4, nc=1, q=0, p=4, engine="multishift",
                      precision="fp64") as plan:
        for k in ks:
            X = np.random.default_rng(k).standard_normal((n, k))
            x = torch.from_numpy(X).cuda()
            y = torch.full_like(x, float("nan"))
            plan.spmm(x, y, alpha=-0.5, beta=2.0)
            want = -0.5 * (A @ X) + 2.0 * X
            bound = (most + 4) * 2.0 ** -53 * (0.5 * (absA @ np.abs(X)) + 2.0 * np.abs(X))
            assert np.all(np.abs(y.cpu().numpy() - want) <= bound), k
