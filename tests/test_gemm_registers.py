"""Registers of the matrix-core GEMM, from the gfx950 assembly of this source
tree: every instance leaves room for two waves a SIMD (256 registers a wave),
spills nothing, and in FP64 and in the element forms keeps its accumulators in
the registers that the MFMAs write (no AGPRs, so no copies in the steps).  Blocks of
up to 64 columns in FP32 with A by rows leave LDS for three workgroups a CU."""

import os
import re
import subprocess

import pytest

from tests.test_kernel_structure import _hipcc


@pytest.fixture(scope="module")
def instances(tmp_path_factory):
    """(type, A by columns, vector length, tiles) -> the kernel's metadata."""
    from paper_2512_01257_amd import build

    out = os.path.join(str(tmp_path_factory.mktemp("gemm")), "k_gemm.s")
    flags = [f for f in build.FLAGS if f != "-fPIC"]
    r = subprocess.run([_hipcc(), *flags, "--cuda-device-only", "-S",
                        os.path.join(build.CSRC, "k_gemm.hip"), "-o", out],
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-4000:]
    found = {}
    for entry in open(out).read().split("amdhsa.kernels:")[1].split("\n  - ")[1:]:
        m = re.search(r"6k_gemmI(d|f)Lb(\d)ELi\d+ELi(\d)ELi(\d)E", entry)
        if m:
            key = (m.group(1), m.group(2) == "1", int(m.group(3)), int(m.group(4)))
            found[key] = {k: int(re.search(rf"\.{k}:\s+(\d+)", entry).group(1))
                          for k in ("agpr_count", "vgpr_count", "vgpr_spill_count",
                                    "group_segment_fixed_size")}
    assert len(found) == 20
    return found


@pytest.mark.skipif(_hipcc() is None, reason="hipcc not available")
def test_two_waves_and_no_copies(instances):
    for key, count in instances.items():
        assert count["vgpr_count"] <= 256 and count["vgpr_spill_count"] == 0, (key, count)
        if key[0] == "d" or key[2] == 1:
            assert count["agpr_count"] == 0, (key, count)


@pytest.mark.skipif(_hipcc() is None, reason="hipcc not available")
def test_three_narrow_workgroups_share_lds(instances):
    # 160 KiB of LDS a CU, given out in pieces of 1280 bytes
    for key, count in instances.items():
        if key[0] == "f" and not key[1] and key[3] <= 2:
            lds = -(-count["group_segment_fixed_size"] // 1280) * 1280
            assert 3 * lds <= 160 * 1024, (key, count)
