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


def test_two_plans_at_once(gpu_lib):
    """Teams of two plans on two threads and streams share the device: each
    solve ends and has the residuals it has alone."""
    import threading

    import torch

    csr = grid_laplacian((70, 70), 0.01)
    A, n, k = csr.to_scipy(), csr.n, 24
    z = np.concatenate([[0.5 + 4e-3j], half_circle(0.0, 1.0, 4)[0]])
    B = np.random.default_rng(5).standard_normal((n, k))
    tol, out, errors = 1e-8, {}, []

    def work(i):
        try:
            stream = torch.cuda.Stream()
            with gpu_lib.Plan(csr, 0.0, 0.6, 8, nc=2, q=1, p=4, precision="fp32",
                              stream=stream.cuda_stream) as plan:
                b = torch.from_numpy(B).cuda()
                X = torch.zeros((n, len(z) * k), dtype=torch.complex64, device="cuda")
                torch.cuda.synchronize()
                for _ in range(3):
                    its, rs = plan.shifted_solve(z, b, X, tol)
                torch.cuda.synchronize()
                out[i] = (X.cpu().numpy().astype(complex), rs)
        except Exception as e:  # the main thread reports it
            errors.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for X, rs in out.values():
        assert rs.max() <= tol
        for j in range(len(z)):
            for c in (0, k - 1):
                x, b = X[:, j * k + c], B[:, c]
                bound = 1.01 * tol * np.linalg.norm(b) + 2 * 2.0 ** -24 * 30 * np.linalg.norm(x)
                assert np.linalg.norm(b - (z[j] * x - A @ x)) <= bound


def test_left_systems_keep_their_solution(gpu_lib):
    """A workgroup that leaves a system to its team goes on with other items:
    with more systems than workgroups the ones with teams take the iterations
    that they take among few (a lost x_hi would cost them what they had)."""
    import torch

    csr = grid_laplacian((80, 80), 0.01)
    n, k = csr.n, 100
    z = np.concatenate([[0.5 + 4e-3j], half_circle(0.0, 1.0, 4)[0]])
    B = np.random.default_rng(11).standard_normal((n, k))
    its = {}
    with gpu_lib.Plan(csr, 0.0, 0.6, 8, nc=2, q=1, p=4, precision="fp32") as plan:
        for m in (k, 10):
            X = torch.zeros((n, len(z) * m), dtype=torch.complex64, device="cuda")
            b = torch.from_numpy(np.ascontiguousarray(B[:, :m])).cuda()
            for rep in range(3):
                its[m], rs = plan.shifted_solve(z, b, X, 1e-8)
                assert rs.max() <= 1e-8
    # one FP32 system's count varies by several percent with the rounding of its
    # sums, the mean of ten by two or three
    assert its[k][:10].mean() <= 1.15 * its[10][:10].mean()
