"""The multi-shift engine applies the shifted updates of four seed iterations in
one pass: iteration counts that leave a pass of one, two or three, several
launches per pass (more shifts than one holds), and FEAST runs whose weighted
sum is accumulated over such passes."""

import numpy as np
import pytest

from oracle.cocg import cocg
from oracle.contour import half_circle
from tests.closed_forms import grid_eigs, window_basis
from tests.feast_checks import check_against, gap_out
from workloads import gaussian, grid_laplacian

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cap,nz,k", [(1, 1, 3), (2, 3, 3), (3, 5, 64), (4, 2, 65), (5, 9, 3),
                                      (8, 4, 3), (11, 6, 130)])
def test_capped_solves_match_single_shift(gpu_lib, cap, nz, k):
    """At the cap every system holds the iterate of single-shift COCG after as
    many steps (the same Krylov space, the same Galerkin condition): a dozen
    steps of a well-conditioned recurrence, a few hundred roundings each."""
    import torch

    csr = grid_laplacian((9, 7, 5), 0.01)
    A, n = csr.to_scipy(), csr.n
    z = np.concatenate([half_circle(0.0, 0.5, max(2, nz))[0]])[:nz]
    B = np.random.default_rng(cap).standard_normal((n, k))
    B[:, 1] = 0.0
    with gpu_lib.Plan(csr, 0.0, 0.5, 8, nc=2, q=1, p=4, precision="fp64", engine="multishift",
                      max_cocg=cap) as plan:
        X = torch.zeros((n, nz * k), dtype=torch.complex128, device="cuda")
        its, _ = plan.shifted_solve(z, torch.from_numpy(B).cuda(), X, 1e-15)
    X = X.cpu().numpy()
    for j in range(nz):
        for c in sorted({0, 1, 2, k - 1}):
            ref, it, _ = cocg(A, z[j], B[:, c], tol=1e-15, maxiter=cap)
            assert its[j * k + c] == it
            assert np.linalg.norm(X[:, j * k + c] - ref) <= 1e-11 * np.linalg.norm(ref)


@pytest.mark.parametrize("nc", [2, 3, 9, 13])
def test_feast_over_several_launches(gpu_lib, nc):
    dims, shift = (20, 20), 0.01
    csr = grid_laplacian(dims, shift)
    lmin, lmax = 0.0, 0.5
    vals, V = window_basis(dims, shift, lmin, lmax)
    allv, _ = grid_eigs(dims, shift)
    m0 = int(1.5 * len(vals))
    with gpu_lib.Plan(csr, lmin, lmax, m0, nc=nc, q=2, p=10, precision="fp64",
                      engine="multishift", tol_solve=1e-6) as plan:
        plan.warmstart(omega=gaussian(csr.n, m0 + 10, 0))
        out = plan.solve()
    assert out["status"] == "OK" and out["M"] == len(vals)
    check_against(out, csr.to_scipy(), vals, V, lmin, lmax, 1e-10, gap_out(allv, lmin, lmax))
