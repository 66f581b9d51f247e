"""A step-level call that fails after it has put work on the plan's stream
returns, like any other, only when that work is done: its host arrays and device
workspaces are the caller's and the next call's again."""

import numpy as np
import pytest

from workloads import grid_laplacian

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw,z,k,status", [
    # real shifts are refused by the multi-shift engine, too many columns by both
    (dict(engine="multishift", precision="fp64"), [0.3 + 0j], 4, "INVALID_ARG"),
    (dict(engine="multishift", precision="fp64"), [0.3 + 0.1j], 193, "UNSUPPORTED"),
    (dict(engine="stream", precision="fp32"), [0.3 + 0.1j], 16385, "UNSUPPORTED")])
def test_failed_shifted_solve_has_waited(gpu_lib, kw, z, k, status):
    import torch

    csr = grid_laplacian((8, 8), 0.01)
    stream = torch.cuda.Stream()
    with gpu_lib.Plan(csr, 0.0, 0.2, 4, nc=1, q=1, p=4, stream=stream.cuda_stream, **kw) as plan:
        B = torch.zeros((csr.n, k), dtype=torch.float64, device="cuda")
        X = torch.zeros((csr.n, k), dtype=torch.complex64 if kw["precision"] == "fp32"
                        else torch.complex128, device="cuda")
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            torch.cuda._sleep(200_000_000)  # about 0.1 to 2 s of the stream's time
        with pytest.raises(gpu_lib.RafeastError) as e:
            plan.shifted_solve(np.array(z), B, X, 1e-8)
        done = stream.query()
        stream.synchronize()
        assert status in str(e.value)
        assert done
