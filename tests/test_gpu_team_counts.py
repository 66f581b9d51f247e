"""Teams of the resident engine are formed, set out, and are solved for where they
do not (rafeast_plan_teams): a changed rule or a lost workspace would leave every
solution right and every system with one workgroup."""

import numpy as np
import pytest

from oracle.contour import half_circle
from workloads import grid_laplacian, knn_laplacian

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("wait", [None, "-1"])
@pytest.mark.parametrize("dims,k", [((65, 65), 3), ((90, 91), 64)])
def test_shifted_solve_teams(gpu_lib, monkeypatch, dims, k, wait):
    import torch

    if wait is not None:  # no team sets out
        monkeypatch.setenv("RAFEAST_TEAM_WAIT", wait)
    # four slots a thread at n = 4225, eight at 8190: only the latter have teams
    csr = grid_laplacian(dims, 0.01)
    z = np.concatenate([[0.5 + 4e-3j], half_circle(0.0, 1.0, 4)[0]])
    B = torch.randn((csr.n, k), dtype=torch.float64, device="cuda")
    X = torch.empty((csr.n, len(z) * k), dtype=torch.complex64, device="cuda")
    with gpu_lib.Plan(csr, 0.0, 0.6, 8, nc=2, q=1, p=4, precision="fp32") as plan:
        assert plan.teams["set_out"] == plan.teams["redone"] == 0
        for calls in (1, 2):
            its, rs = plan.shifted_solve(z, B, X, 1e-8)
            assert rs.max() <= 1e-8
            t = plan.teams
            if plan.tuning["chosen"] != 8:
                assert t["set_out"] == t["redone"] == 0
            elif wait is None:  # the hardest shift's systems, on a free device
                assert t["set_out"] >= calls and t["redone"] == 0
            else:
                assert t["redone"] >= calls and t["set_out"] == 0


@pytest.mark.parametrize("wait", [None, "-1"])
def test_solve_teams(gpu_lib, monkeypatch, wait):
    if wait is not None:
        monkeypatch.setenv("RAFEAST_TEAM_WAIT", wait)
    csr = knn_laplacian(8000, 2, 10, seed=1, weighted=True, shift=1e-3)
    with gpu_lib.Plan(csr, 0.0, 1e-3 + 9.4 * 24 / 8000, 32, nc=4, q=1) as plan:
        assert plan.tuning["chosen"] == 8
        t = plan.teams
        assert 0 < t["planned"] <= 128 and t["set_out"] == t["redone"] == 0
        plan.warmstart()
        out = plan.solve(want_vectors=False)
        assert out["status"] == "OK"
        t = plan.teams
        assert t["planned"] > 0
        left = t["redone"] if wait else t["set_out"]
        assert out["iters"] <= left <= out["iters"] * t["planned"]
        assert t["set_out" if wait else "redone"] == 0
    monkeypatch.setenv("RAFEAST_RESIDENT_SLOTS", "8")
    with gpu_lib.Plan(csr, 0.0, 1e-3 + 9.4 * 24 / 8000, 32, nc=4, q=1) as plan:
        plan.warmstart()
        plan.solve(want_vectors=False)
        assert plan.teams == dict(planned=0, set_out=0, redone=0)
