"""The caches of device workspaces, against a device of a given capacity that
lives in host memory (CPU only): blocks are used again, what is kept stays
within the caches' and the pool's bounds with the oldest blocks freed first, an
allocation that does not fit gets everything idle back from every cache, and
nothing is lost or freed twice, also with several threads."""

import shutil
import subprocess

import pytest

SRC = r"""
#include "work_cache.h"
#include <assert.h>
#include <stdio.h>
#include <stdlib.h>
#include <atomic>
#include <map>
#include <thread>
#undef NDEBUG
#include <assert.h>
using namespace rafeast;
static std::mutex mu;
static std::map<void*, size_t> live;
static size_t used = 0, capacity = 0, calls = 0;
static int alloc(void** q, size_t bytes) {
  std::lock_guard<std::mutex> lock(mu);
  ++calls;
  if (used + bytes > capacity) return 2;
  *q = malloc(1);
  live[*q] = bytes;
  used += bytes;
  return 0;
}
static void release(void* q) {
  std::lock_guard<std::mutex> lock(mu);
  assert(live.count(q));  // not freed twice
  used -= live[q];
  live.erase(q);
  free(q);
}
int main() {
  const size_t K = 1024;
  void *a, *b, *c;
  size_t sa, sb, sc;
  {
    capacity = 100 * K;
    WorkPool pool({alloc, release, 2}, 32 * K);
    WorkCache x(pool, 32 * K), y(pool, 32 * K);
    // used again for at most half of a block and more
    sa = 10 * K;
    assert(x.get(&a, sa) == 0 && sa == 10 * K);
    x.put(a, sa);
    sb = 6 * K;
    assert(x.get(&b, sb) == 0 && b == a && sb == 10 * K && pool.idle_bytes() == 0);
    x.put(b, sb);
    sb = 4 * K;
    assert(x.get(&b, sb) == 0 && b != a && sb == 4 * K);
    x.put(b, sb);
    // another cache's blocks are not this one's
    sc = 10 * K;
    assert(y.get(&c, sc) == 0 && c != a);
    y.put(c, sc);
    assert(pool.idle_bytes() == 24 * K && used == 24 * K);
    // past the pool's bound the oldest goes, whichever cache holds it
    sc = 12 * K;
    assert(y.get(&c, sc) == 0);
    y.put(c, sc);
    assert(pool.idle_bytes() == 26 * K && used == 26 * K && !live.count(a));
    // a block above the bound is not kept
    sc = 40 * K;
    assert(y.get(&c, sc) == 0);
    y.put(c, sc);
    assert(pool.idle_bytes() == 26 * K && used == 26 * K);
    // a cache full of blocks that do not serve makes room for one that does
    for (int i = 0; i < 2; ++i) {
      sc = 30 * K;
      const size_t before = calls;
      assert(x.get(&c, sc) == 0);
      x.put(c, sc);
      assert(calls - before == (i == 0 ? 1 : 0));
    }
    assert(pool.idle_bytes() == 30 * K && used == 30 * K);
    // an allocation that does not fit: all caches give back, then it does
    sa = 2 * K;
    assert(y.get(&a, sa) == 0);
    y.put(a, sa);
    assert(pool.idle_bytes() == 32 * K);
    assert(pool.alloc(&b, 90 * K) == 0 && pool.idle_bytes() == 0 && used == 90 * K);
    sc = 20 * K;
    assert(x.get(&c, sc) == 2 && c == nullptr);
    release(b);
    assert(x.get(&c, sc) == 0);
    x.put(c, sc);
  }
  assert(used == 0);  // the caches freed theirs
  {
    capacity = 150 * K;
    WorkPool pool({alloc, release, 2}, 140 * K);
    std::atomic<int> failed{0};
    std::vector<std::thread> t;
    for (int i = 0; i < 6; ++i)
      t.emplace_back([&, i] {
        for (int round = 0; round < 50; ++round) {
          WorkCache own(pool, 140 * K);
          unsigned r = 7 * i + round;
          for (int s = 0; s < 40; ++s) {
            r = r * 1103515245u + 12345u;
            void* q;
            size_t bytes = 256 + (r >> 8) % (6 * K);
            if (own.get(&q, bytes) != 0) {
              ++failed;
              continue;
            }
            assert(q);
            own.put(q, bytes);
          }
        }
      });
    for (auto& th : t) th.join();
    assert(used == 0 && pool.idle_bytes() == 0);
    assert(failed < 6 * 50 * 40 / 10);  // only beside blocks that a thread is just freeing
  }
  puts("ok");
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_work_cache(tmp_path):
    from paper_2512_01257_amd import build

    src = tmp_path / "cache.cpp"
    src.write_text(SRC)
    exe = str(tmp_path / "cache")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", build.CSRC, str(src), "-o", exe],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout == "ok\n", (r.returncode, r.stderr[-2000:])
