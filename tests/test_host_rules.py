"""Rules of the launchers that are plain host functions, on devices and sizes
that the tests' GPU does not have: small C++ programs against the library's
internal headers (CPU only, no device is touched)."""

import os
import subprocess

import pytest

from tests.test_kernel_structure import _hipcc

pytestmark = pytest.mark.skipif(_hipcc() is None, reason="hipcc not available")


def run(tmp_path, body, before=""):
    """Compiles body as main's text, links the library and returns its output lines.
    before: definitions, of HIP functions among others: the program's own take
    the place of the runtime's in the library, too."""
    from paper_2512_01257_amd import build

    src = tmp_path / "rule.cpp"
    src.write_text('#include "kernels.h"\n#include "../../include/rafeast.h"\n#include <cstdio>\n'
                   "#include <vector>\nusing namespace rafeast;\n" + before +
                   "\nint main() {\n" + body + "\nreturn 0;\n}\n")
    exe = str(tmp_path / "rule")
    cmd = [_hipcc(), "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-I", build.CSRC,
           "-x", "hip", str(src), "-o", exe, "-rdynamic", "-L", build.HERE, "-l:librafeast.so",
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


# a device without memory on which every launch succeeds and does nothing
NO_MEMORY = """
static std::vector<dim3> grids;
static std::vector<const void*> kernels;
static dim3 next_grid;
extern "C" {
hipError_t hipMalloc(void** p, size_t) { *p = nullptr; return hipErrorOutOfMemory; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3 g, dim3, size_t, hipStream_t) {
  next_grid = g;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3*, dim3*, size_t*, hipStream_t*) { return hipSuccess; }
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void**, size_t, hipStream_t) {
  kernels.push_back(f);
  grids.push_back(next_grid);
  return hipSuccess;
}
}
"""


@pytest.mark.parametrize("m,n,k", [(602, 350, 1391), (300, 24, 4096), (64, 32, 300)])
def test_gemm_runs_unsplit_without_memory(tmp_path, m, n, k):
    # split for speed where there is room, in one launch of one chunk where not
    out = run(tmp_path, f"""
  std::printf("%zu\\n", gemm_work_elems(true, {m}, {n}, {k}));
  double* p = reinterpret_cast<double*>(4096);
  int s = rafeast_gemm(nullptr, RAFEAST_FP64, 1, {m}, {n}, {k}, p, {m}, p, {n}, p, {n}, 1.0, 0.0);
  std::printf("%d %zu %u\\n", s, grids.size(), grids.empty() ? 0 : grids[0].z);
""", NO_MEMORY)
    assert int(out[0]) > 0
    assert out[1] == "0 1 1"  # OK, one launch, one chunk


@pytest.mark.parametrize("f64", [0, 1])
@pytest.mark.parametrize("m,n,a_cols", [(512, 29, 0), (512, 29, 1), (97, 64, 1), (97, 27, 1)])
def test_gemm_takes_vectors_only_where_none_is_cut(tmp_path, f64, m, n, a_cols):
    # C is smaller than a tile and cuts a vector: the vector form has no whole
    # step, and alignment of the operands does not change that
    prec = "RAFEAST_FP64" if f64 else "RAFEAST_FP32_REFINED"
    out = run(tmp_path, f"""
  const int lda[2] = {{600, 601}}, ldb[2] = {{128, 129}};
  for (int i = 0; i < 2; ++i) {{
    void* p = reinterpret_cast<void*>(4096 + i * {8 if f64 else 4});
    std::printf("%d\\n", rafeast_gemm(nullptr, {prec}, {a_cols}, {m}, {n}, 100, p, lda[i], p,
                                       ldb[i], p, {n}, 1.0, 0.0));
  }}
  std::printf("%zu %d\\n", kernels.size(), kernels.size() == 2 && kernels[0] == kernels[1]);
""", NO_MEMORY)
    assert out == ["0", "0", "2 1"]


def test_spmm_form(tmp_path):
    # the one-column form (the kernel that a single column takes) or the number of
    # workgroups of the two-column one, for (rows, entries a row, span, columns)
    cases = {(20000, 3, 1, 65): "one", (20000, 3, 1, 119): "one", (20000, 3, 1, 121): "pairs",
             (20000, 5, 2, 65): "pairs", (20000, 3, 1, 129): "one", (20000, 3, 1, 66): "pairs",
             (250000, 3, 1, 73): "one", (250000, 3, 1, 81): "pairs", (20000, 3, 1, 193): "pairs",
             (64000, 40, 120, 137): "one", (64000, 40, 60000, 137): "pairs",
             (64000, 40, 120, 191): "one", (64000, 40, 120, 193): "pairs",
             (64000, 20, 60, 191): "pairs", (64000, 7, 1600, 147): "pairs",
             (9402, 19, 9000, 147): "one", (50000, 19, 49000, 33): "one",
             # eight lanes a row on few rows: 32 rows a workgroup
             (4000, 67, 3900, 3): 128, (4000, 67, 3900, 2): 128, (16384, 70, 200, 5): 512,
             (16384, 13, 200, 64): 1024, (16384, 40, 200, 64): 2048, (70000, 3, 1, 128): 8752,
             (16385, 70, 200, 5): 264, (16385, 70, 200, 9): 520}
    calls = "".join(f"""
  launch_spmm_f64(nullptr, {n}, {k}, nullptr, nullptr, nullptr, {n * d}LL, nullptr, {k}, nullptr,
                  {k}, 1.0, 0.0, nullptr, 0, 0.0, {s});""" for n, d, s, k in cases)
    out = run(tmp_path, """
  launch_spmm_f64(nullptr, 100, 1, nullptr, nullptr, nullptr, 100, nullptr, 1, nullptr, 1, 1.0,
                  0.0, nullptr, 0, 0.0, 0);""" + calls + """
  for (size_t i = 1; i < kernels.size(); ++i)
    std::printf("%d %u\\n", kernels[i] == kernels[0], grids[i].x);
""", NO_MEMORY)
    assert len(out) == len(cases)
    for line, (case, want) in zip(out, cases.items()):
        one, grid = map(int, line.split())
        if want in ("one", "pairs"):
            assert bool(one) == (want == "one"), case
        else:
            assert not one and grid == want, (case, grid)


def test_band_width(tmp_path):
    # 64 shifts: widened up to 2^20 rows (32 GiB), at its own width above
    got = run(tmp_path, """
  for (long long n : {100LL, 1048576LL, 1048577LL, 70000000LL})
    for (int b : {0, 1, 30, 31, 500}) std::printf("%d\\n", band_width(n, 64, b));
""")
    wide, own = ["31", "31", "31", "31", "500"], ["0", "1", "30", "31", "500"]
    assert got == wide + wide + own + own


def test_team_planning(tmp_path):
    # shifts of a half circle around the low end of [0, 20]: the one nearest the
    # spectrum takes four times the others' steps
    out = run(tmp_path, """
  const double zs[] = {0.0567, 0.0062, 0.0007, 0.0062, 0.0141, 0.0247, 0.0433, 0.0247};
  const int order[] = {0, 1, 3, 2};
  auto plan = [&](int shifts, int k, int cu, int rpt, bool same) {
    std::vector<int> items, of;
    for (int j = 0; j < shifts; ++j)
      for (int i = 0; i < k; ++i) {
        items.push_back(0);
        items.push_back(same ? 0 : order[j]);
        items.push_back(i);
      }
    double done = -1.0;
    const int n = cocg_plan_teams(items, zs, 0.001, 19.76, cu, rpt, of, done);
    int bad = n > 0 && (int)of.size() != shifts * k;
    for (size_t i = 0; i < of.size(); ++i) bad += of[i] != ((int)i < n ? (int)i : -1);
    std::printf("%d %d %d %d\\n", n, bad, done > 0.0,
                done > 0.0 ? cocg_team_iteration(done, 1e-6) : 0);
  };
  plan(4, 64, 256, 8, false);
  plan(4, 10, 256, 8, false);
  plan(4, 64, 256, 4, false);
  plan(4, 64, 32, 8, false);
  plan(4, 64, 256, 8, true);
  plan(4, 200, 256, 8, false);
  plan(1, 1, 256, 8, false);
""")
    rows = [tuple(map(int, ln.split())) for ln in out]
    assert all(bad == 0 for _, bad, _, _ in rows)
    full, few, slots, small, alike, many, single = rows
    # the hardest shift's systems, left when the others are done (343 to 377 steps)
    assert full[0] == 64 and 300 <= full[3] <= 420
    # few systems: CUs for teams of all at once
    assert few[0] == 40
    # four slots a thread, a small device, equal shifts: no teams; more systems of
    # the hardest shift than half the CUs: none either; one system: its team starts
    # at once or there is none
    assert slots[0] == small[0] == alike[0] == many[0] == 0
    assert single[0] in (0, 1)


def test_plan_teams_refuses_null_pointers():
    import ctypes as C

    from paper_2512_01257_amd import native

    n = C.c_int32()
    assert native.lib().rafeast_plan_teams(None, C.byref(n), C.byref(n), C.byref(n)) == 1
