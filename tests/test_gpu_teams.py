"""Resident engine: systems that are expected to run long after the others are
continued by four workgroups each.  Solves against their FP64 residuals and
exact solutions, the same bits on every run, systems that are done before the
teams take over, numbers of teams that do not fill a group."""

import numpy as np
import pytest

from oracle.contour import half_circle
from tests.closed_forms import grid_eigs
from workloads import grid_laplacian

pytestmark = pytest.mark.gpu


# n = 4225 (slots with few slices), 8190 (a partial last slice, nearly all
# slots); k systems of the hardest shift get teams; 64 * 2 > one round of teams
@pytest.mark.parametrize("dims,k", [((65, 65), 1), ((65, 65), 7), ((90, 91), 9), ((90, 91), 64),
                                    ((80, 80), 100)])
@pytest.mark.parametrize("wait", [None, "0"])
def test_team_solves(gpu_lib, monkeypatch, dims, k, wait):
    # wait 0: a team whose members do not all run at once does not set out, and
    # its system is solved by a launch of its own
    import torch

    if wait is not None:
        monkeypatch.setenv("RAFEAST_TEAM_WAIT", wait)

    csr = grid_laplacian(dims, 0.01)
    A, n = csr.to_scipy(), csr.n
    z = np.concatenate([[0.5 + 4e-3j], half_circle(0.0, 1.0, 4)[0]])
    lam = grid_eigs(dims, 0.01)[0]
    B = np.random.default_rng(k).standard_normal((n, k))
    if k > 2:
        B[:, 1] = 0.0
        B[:, 2] *= 1e-7
    tol = 1e-8
    runs = []
    with gpu_lib.Plan(csr, 0.0, 0.6, 8, nc=2, q=1, p=4, precision="fp32") as plan:
        assert plan.engine == "resident"
        for _ in range(2):
            X = torch.zeros((n, len(z) * k), dtype=torch.complex64, device="cuda")
            its, rs = plan.shifted_solve(z, torch.from_numpy(B).cuda(), X, tol)
            runs.append((X.cpu().numpy(), its, rs))
    if wait is None:
        assert all(np.array_equal(a, b) for a, b in zip(*runs))
    X, its, rs = runs[1]
    u = 2.0 ** -24
    norm_m = np.abs(z).max() + 8.02
    for j in range(len(z)):
        for c in range(k):
            x, b = X[:, j * k + c].astype(complex), B[:, c]
            if not b.any():
                assert not x.any() and its[j * k + c] == 0 and rs[j * k + c] == 0
                continue
            assert rs[j * k + c] <= tol
            bound = 1.01 * tol * np.linalg.norm(b) + 2 * u * norm_m * np.linalg.norm(x)
            assert np.linalg.norm(b - (z[j] * x - A @ x)) <= bound
            dist = np.abs(z[j] - lam).min()
            assert np.linalg.norm(x) <= 1.01 * np.linalg.norm(b) / dist
    assert its[0] > 2 * its[k:].max() > 0  # the first shift's systems run on
