"""The kernels of the resident engine's teams, read from the gfx950 assembly of
this source tree: the launch that leaves systems to teams keeps the uniform work
loop of the plain one (fetch, then barrier), and no loop of it or of the team
kernel is latched by the execution mask (a wave would wait at a workgroup
barrier with part of its lanes)."""

import os
import re
import subprocess

import pytest

from tests.test_kernel_structure import _hipcc


@pytest.mark.skipif(_hipcc() is None, reason="hipcc not available")
def test_team_loops_are_uniform(tmp_path):
    from paper_2512_01257_amd import build

    out = os.path.join(str(tmp_path), "k_cocg.s")
    flags = [f for f in build.FLAGS if f != "-fPIC"]
    r = subprocess.run([_hipcc(), *flags, "--cuda-device-only", "-S",
                        os.path.join(build.CSRC, "k_cocg.hip"), "-o", out],
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-4000:]
    parts = re.split(r"\n(_ZN7rafeast(?:14k_cocg_leaving|11k_cocg_team)I\S+):", open(out).read())
    kernels = {parts[i]: parts[i + 1][: parts[i + 1].find(".Lfunc_end")]
               for i in range(1, len(parts), 2)}
    assert len(kernels) == 2
    for name, body in kernels.items():
        lines = body.split("\n")
        assert not [ln for ln in lines if re.search(r"s_andn2_b64\s+exec,\s*exec", ln)], name
        if "leaving" not in name:
            continue
        top = next(k for k, ln in enumerate(lines) if "=>This Loop Header: Depth=1" in ln)
        seq = []
        for ln in lines[top + 1:]:
            if "This Loop Header: Depth=2" in ln:
                break
            if "global_atomic_add" in ln:
                seq.append("fetch")
            elif "s_barrier" in ln:
                seq.append("barrier")
        assert seq[:2] == ["fetch", "barrier"], (name, seq)
