"""Registers of the matrix-core GEMM, from the gfx950 assembly of this source
tree: every instance leaves room for two waves a SIMD (256 registers a wave),
spills nothing, and in FP64 and in the element forms keeps its accumulators in
the registers that the MFMAs write (no AGPRs, so no copies in the steps)."""

import os
import re
import subprocess

import pytest

from tests.test_kernel_structure import _hipcc


@pytest.mark.skipif(_hipcc() is None, reason="hipcc not available")
def test_two_waves_and_no_copies(tmp_path):
    from paper_2512_01257_amd import build

    out = os.path.join(str(tmp_path), "k_gemm.s")
    flags = [f for f in build.FLAGS if f != "-fPIC"]
    r = subprocess.run([_hipcc(), *flags, "--cuda-device-only", "-S",
                        os.path.join(build.CSRC, "k_gemm.hip"), "-o", out],
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-4000:]
    meta = open(out).read().split("amdhsa.kernels:")[1]
    seen = 0
    for entry in meta.split("\n  - ")[1:]:
        m = re.search(r"6k_gemmI(d|f)Lb(\d)ELi\d+ELi(\d)ELi(\d)E", entry)
        if not m:
            continue
        seen += 1
        count = {k: int(re.search(rf"\.{k}:\s+(\d+)", entry).group(1))
                 for k in ("agpr_count", "vgpr_count", "vgpr_spill_count")}
        assert count["vgpr_count"] <= 256 and count["vgpr_spill_count"] == 0, (m.group(0), count)
        if m.group(1) == "d" or m.group(3) == "1":
            assert count["agpr_count"] == 0, (m.group(0), count)
    assert seen == 20
