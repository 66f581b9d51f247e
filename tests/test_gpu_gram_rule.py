"""The Gram product of one block on both sides of the rule that chooses between
the symmetric and the general kernel, and its allocation-free form, which gives
the same bits as long as its scratch holds as many row chunks."""

import numpy as np
import pytest

from workloads import grid_laplacian

pytestmark = pytest.mark.gpu


# rows and widths at the rule's lines: 3 | 4, 32 | 33, 64 | 65, 96 | 97 columns,
# 2^14, 2^17, 4096, 8192 rows
@pytest.mark.parametrize("n,k", [
    (16384, 3), (16385, 3), (16385, 4), (131072, 32), (131073, 32), (131073, 33), (300, 64),
    (4096, 65), (4097, 65), (4097, 96), (8192, 97), (8193, 97), (8193, 192), (200_000, 80),
    (200_000, 90), (200_000, 96), (140_000, 17)])
def test_gram_of_one_block(gpu_lib, n, k):
    import torch

    st = torch.cuda.Stream()
    with torch.cuda.stream(st), gpu_lib.Plan(grid_laplacian((6, 6), 0.1), 0.0, 0.5, 4, nc=1, q=0,
                                             p=4, stream=st.cuda_stream) as plan:
        X = torch.from_numpy(np.random.default_rng(n + k).standard_normal((n, k))).cuda()
        G = torch.full((k, k), float("nan"), dtype=torch.float64, device="cuda")
        F = torch.full_like(G, float("nan"))
        plan.gram(X, X, G)
        gpu_lib.gram_noalloc(X, X, F, stream=st)
        torch.cuda.synchronize()
        ref = X.T @ X
        # sums of n products in some order
        bound = 2.0 * n * 2.0 ** -53 * (X.abs().T @ X.abs())
        assert bool(((G - ref).abs() <= bound).all())
        assert torch.equal(G, G.T)
        if k <= 96:
            assert torch.equal(F, G)
        else:
            assert bool(((F - ref).abs() <= bound).all())
