"""The reduced eigenproblem of one and two columns, over scales and gaps: the
spectrum and the factorization H S = S diag(theta) to rounding, S orthogonal."""

import numpy as np
import pytest

from workloads import grid_laplacian

pytestmark = pytest.mark.gpu

U = 2.0 ** -53


def test_syev_one_and_two(gpu_lib):
    import torch

    mats = [[[3.0]], [[-1e-200]]]
    for scale in (1.0, 1e-140, 1e140):
        for a, b, d in ((1, 0, 2), (2, 0, 1), (1, 0, 1), (1, 0.5, 1), (1, -0.5, 1), (1, 1e-17, 1),
                        (1, 1e-9, 2), (-3, 2, 5), (5, 2, -3), (0, 1, 0), (0, 0, 0), (1, 1e3, 1.5)):
            mats.append(scale * np.array([[a, b], [b, d]], dtype=float))
    mats.append(np.array([[1.0, 2.0], [0.0, 1.0]]))  # the symmetric part counts
    with gpu_lib.Plan(grid_laplacian((6, 6), 0.1), 0.0, 0.5, 4, nc=1, q=0, p=4) as plan:
        for H in mats:
            H = np.ascontiguousarray(H, dtype=float)
            k = len(H)
            th = torch.full((k,), float("nan"), dtype=torch.float64, device="cuda")
            S = torch.full((k, k), float("nan"), dtype=torch.float64, device="cuda")
            plan.syev(torch.from_numpy(H).cuda(), th, S)
            th, S, G = th.cpu().numpy(), S.cpu().numpy(), 0.5 * (H + H.T)
            size = np.abs(G).max()
            # a few operations on each entry
            assert np.all(np.diff(th) >= 0)
            assert np.abs(th - np.linalg.eigvalsh(G)).max() <= 16 * U * size, H
            assert np.abs(G @ S - S * th).max() <= 32 * U * size, H
            assert np.abs(S.T @ S - np.eye(k)).max() <= 16 * U, H
