"""The multi-shift engine without memory for the residuals of four iterations: it
runs with one, to the same bits."""

import numpy as np
import pytest

from workloads import grid_laplacian

pytestmark = pytest.mark.gpu


def test_multishift_without_room(gpu_lib):
    import torch

    csr = grid_laplacian((700, 700), 0.01)
    n, k = csr.n, 64
    z = np.array([0.05 + 0.2j, 0.3 + 0.1j])
    B = torch.randn((n, k), dtype=torch.float64, device="cuda",
                    generator=torch.Generator(device="cuda").manual_seed(3))
    X = torch.empty((n, 2 * k), dtype=torch.complex128, device="cuda")
    block = n * k * 8  # 251 MB
    # p, w (1 each), X, P (4 each) and the residuals (4, or 1)
    with gpu_lib.Plan(csr, 0.0, 0.2, 4, nc=1, q=0, p=4, engine="multishift",
                      precision="fp64") as plan:
        its, rs = plan.shifted_solve(z, B, X, 1e-9)
        want = X.clone()
    assert rs.max() <= 2e-9
    with gpu_lib.Plan(csr, 0.0, 0.2, 4, nc=1, q=0, p=4, engine="multishift",
                      precision="fp64") as plan:
        X.fill_(float("nan"))
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        fill = []
        for _ in range(4):
            over = torch.cuda.mem_get_info()[0] - int(12.5 * block)
            if over > block // 8:
                fill.append(torch.empty(over, dtype=torch.uint8, device="cuda"))
        assert 12 * block < torch.cuda.mem_get_info()[0] < 13 * block
        try:
            its2, rs2 = plan.shifted_solve(z, B, X, 1e-9)
        finally:
            del fill
            torch.cuda.empty_cache()
    assert np.array_equal(its, its2) and np.array_equal(rs, rs2)
    assert torch.equal(X.view(torch.float64), want.view(torch.float64))
