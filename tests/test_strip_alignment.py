"""The lane geometry of the fused weight-gradient + Adam kernel, compiled for the host: a lane that takes its four columns as one
16-byte piece does so on 16-byte boundaries, and the lanes of a matrix cover every element exactly once."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = """
#include <stdio.h>
#include <vector>
#include "fade_rules.h"
int main() {
  const size_t off = 12;
  for (int N = 1; N <= 200; ++N) {
    const int M = 21;
    std::vector<int> seen(M * N, 0);
    for (int n0 = 0; n0 < N; n0 += 64)
      for (int m = 0; m < M; ++m)
        for (int q = 0; q < 16; ++q) {
          const FadeStripLane at = fade_strip_lane(off, N, n0, m, q);
          if (at.left <= 0) continue;
          if (at.vec && (at.left != 4 || at.idx % 4 != 0)) { printf("N=%d row %d lane %d: piece at %zu, %d left\\n", N, m, q, at.idx, at.left); return 1; }
          if (N % 4 == 0 && !at.vec) { printf("N=%d: no pieces\\n", N); return 1; }
          for (int i = 0; i < at.left; ++i) ++seen[at.idx - off + i];
        }
    for (int i = 0; i < M * N; ++i)
      if (seen[i] != 1) { printf("N=%d: element %d covered %d times\\n", N, i, seen[i]); return 1; }
  }
  return 0;
}
"""


def test_strip_pieces_are_aligned_and_cover_the_matrix(tmp_path):
    src, exe = tmp_path / "strip.cpp", tmp_path / "strip"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2604_07239_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
