"""Device memory of plans: a small plan's fixed part, whatever its subspace."""

import numpy as np
import pytest

from workloads import grid_laplacian

pytestmark = pytest.mark.gpu


def test_small_plans_are_small(gpu_lib):
    import torch

    torch.cuda.synchronize()
    csr, plans = grid_laplacian((6, 6), 0.1), []
    plans.append(gpu_lib.Plan(csr, 0.0, 0.5, 4, nc=1, q=0, p=4, engine="stream"))
    before = torch.cuda.mem_get_info()[0]
    for _ in range(16):
        plans.append(gpu_lib.Plan(csr, 0.0, 0.5, 4, nc=1, q=0, p=4, engine="stream"))
    used = (before - torch.cuda.mem_get_info()[0]) / 16
    # three matrices of 192 x 192 doubles and small arrays, each rounded up by the
    # runtime; the list of rotations for 192 columns alone would be 11.7 MB
    assert used <= 6e6, used
    # the reduced eigenproblem takes any k <= 192 all the same, also after smaller ones
    for k in (192, 9, 192):
        H = np.random.default_rng(k).standard_normal((k, k))
        H = H + H.T
        theta = torch.empty(k, dtype=torch.float64, device="cuda")
        S = torch.empty((k, k), dtype=torch.float64, device="cuda")
        plans[3].syev(torch.from_numpy(H).cuda(), theta, S)
        lam = np.linalg.eigvalsh(H)
        assert np.abs(theta.cpu().numpy() - lam).max() <= 1e-12 * np.abs(lam).max()
    for p in plans:
        p.close()
