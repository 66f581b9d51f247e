"""Direct engine on matrices whose entries squared leave the range of a double:
the factorization depends on the matrix's scale by powers of two alone, so the
solutions of 2^s A at 2^s z are those of A at z times 2^-s."""

import numpy as np
import pytest

from workloads import CSR, knn_laplacian

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("s", [-560, -300, 300, 500])
@pytest.mark.parametrize("n", [40, 500])
def test_direct_solves_scale(gpu_lib, n, s):
    import torch

    csr = knn_laplacian(n, 2, 6, seed=3, weighted=True, shift=1e-3)
    z = np.array([0.05 + 0.02j, 0.4 - 0.3j])
    B = np.random.default_rng(n).standard_normal((n, 3))
    out = []
    for e in (0, s):
        f = 2.0 ** e
        A = CSR(csr.n, csr.rowptr, csr.colind, csr.values * f)
        with gpu_lib.Plan(A, 0.0, 0.5 * f, 4, nc=1, q=0, p=4, precision="fp64",
                          engine="direct") as plan:
            X = torch.zeros((n, 2 * 3), dtype=torch.complex128, device="cuda")
            _, rs = plan.shifted_solve(z * f, torch.from_numpy(B).cuda(), X, 1e-10)
        out.append(X.cpu().numpy() * f)
        assert rs.max() <= 1e-11
    # the two forms of the pivots' inverse round differently: both solutions are
    # within kappa times a modest multiple of u (kappa <= 400: |z - lambda| in
    # [0.02, 8])
    assert np.abs(out[1] - out[0]).max() <= 1e3 * 400 * 2.0 ** -53 * np.abs(out[0]).max()
