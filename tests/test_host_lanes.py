"""fade_lanes.h, compiled for the host: work shared by several threads, some of which may not start."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LANES = """
#include <stdio.h>
#include <stdlib.h>
#include <atomic>
#include <new>
#include "fade_lanes.h"
static std::atomic<int> left{1 << 30};  // allocations until there is no memory
void *operator new(size_t n) {
  if (left.fetch_sub(1) <= 0) throw std::bad_alloc();
  return malloc(n);
}
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }
int main(int, char **argv) {
  const int threads = atoi(argv[1]), n = atoi(argv[2]);
  std::atomic<int> next{0}, done{0}, lanes{0};
  left = threads;  // one allocation per thread that starts
  fade_on_lanes<4>(n, [&](int) noexcept {
    ++lanes;
    for (int k; (k = next.fetch_add(1)) < 1000;) ++done;
  });
  left = 1 << 30;
  const int want = 1 + (n - 1 < threads ? n - 1 : threads);
  if (done != 1000 || lanes != want) { printf("%d of 1000 done by %d lanes, not %d\\n", done.load(), lanes.load(), want); return 1; }
  return 0;
}
"""


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    d = tmp_path_factory.mktemp("lanes")
    (d / "lanes.cpp").write_text(LANES)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-pthread", "-I", os.path.join(ROOT, "paper_2604_07239_amd", "csrc"), str(d / "lanes.cpp"),
                    "-o", str(d / "lanes")], check=True)
    return str(d / "lanes")


@pytest.mark.parametrize("threads", [0, 1, 2, 3])
@pytest.mark.parametrize("n", [1, 2, 4])
def test_work_is_done_by_the_threads_there_are(exe, threads, n):
    r = subprocess.run([exe, str(threads), str(n)], capture_output=True, text=True)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)
