"""Rules of the launchers that are plain host functions, on devices and sizes
that the tests' GPU does not have: small C++ programs against the library's
internal headers (CPU only, no device is touched)."""

import os
import subprocess

import pytest

from tests.test_kernel_structure import _hipcc

pytestmark = pytest.mark.skipif(_hipcc() is None, reason="hipcc not available")


def run(tmp_path, body):
    """Compiles body as main's text, links the library and returns its output lines."""
    from paper_2512_01257_amd import build

    src = tmp_path / "rule.cpp"
    src.write_text('#include "kernels.h"\n#include <cstdio>\n#include <vector>\n'
                   "using namespace rafeast;\nint main() {\n" + body + "\nreturn 0;\n}\n")
    exe = str(tmp_path / "rule")
    cmd = [_hipcc(), "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-I", build.CSRC,
           "-x", "hip", str(src), "-o", exe, "-L", build.HERE, "-l:librafeast.so",
           "-Wl,-rpath," + build.HERE]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stderr[-2000:])
    return r.stdout.split("\n")[:-1]


def test_shifted_updates_take_every_row_once(tmp_path):
    # the updates are in place: a row that two workgroups reach is updated twice.
    # Row block r of workgroup b: stripe b mod 8, swept with a stride of grid / 8
    # workgroups, from workgroup b / 8 on
    out = run(tmp_path, """
  for (int cu : {1, 3, 7, 8, 60, 104, 110, 228, 252, 255, 256, 304})
    for (int nz : {2, 4, 8})
      for (int n : {1, 31, 255, 4000, 30001}) std::printf("%d %d\\n", n, ms_shift_blocks(n, cu, nz));
""")
    rows_of_step = 32  # eight waves of four rows
    for line in out:
        n, grid = map(int, line.split())
        count = [0] * n
        stripe, stride = (n + 7) // 8, (grid >> 3) * rows_of_step
        assert stride > 0
        for b in range(grid):
            hi = min(n, ((b & 7) + 1) * stripe)
            for r0 in range((b & 7) * stripe + (b >> 3) * rows_of_step, hi, stride):
                for r in range(r0, min(hi, r0 + rows_of_step)):
                    count[r] += 1
        assert count == [1] * n, (n, grid)
