"""The rules and the index arithmetic of fade_rules.h, compiled for the host."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
STRIP = """
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


def _run(text, tmp_path):
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text(text)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2604_07239_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_strip_pieces_are_aligned_and_cover_the_matrix(tmp_path):
    """The fused weight-gradient + Adam kernel: a lane that takes its four columns as one 16-byte piece does so on 16-byte
    boundaries, and the lanes of a matrix cover every element exactly once."""
    _run(STRIP, tmp_path)


STREAMED = """
#include <stdio.h>
#include "fade_rules.h"
static size_t params(size_t B, size_t T, size_t D, size_t H) {  // the matrices
  const size_t Dh = T * D;
  return B * 4096 + 4 * H * Dh + 2 * Dh * Dh + 2 * 64 * Dh + 256 * Dh + 256 * D;
}
static int wrong = 0;
static void want(bool streamed, bool bf16, bool online, size_t B, size_t T, size_t D, size_t H) {
  if (fade_streamed(bf16, online, params(B, T, D, H), B, T * D) == streamed) return;
  printf("%s %s B=%zu T=%zu D=%zu H=%zu\\n", bf16 ? "bf16" : "fp32", online ? "adapting" : "frozen", B, T, D, H);
  ++wrong;
}
int main() {
  // either side of the line as measured, and far from it
  want(false, true, true, 16, 64, 32, 128);
  want(false, true, true, 128, 64, 32, 128);
  want(false, true, true, 16, 64, 32, 256);
  want(true, true, true, 256, 64, 32, 128);
  want(true, true, true, 16, 64, 32, 512);
  want(false, true, true, 128, 16, 32, 512);
  want(false, true, true, 1024, 16, 32, 512);
  want(true, true, true, 2048, 16, 32, 512);
  want(true, true, true, 1024, 64, 32, 256);
  want(true, true, true, 16384, 64, 32, 512);
  want(false, true, false, 8192, 16, 32, 256);
  want(true, true, false, 16384, 16, 32, 256);
  // fp32 never, however large
  want(false, false, true, 300, 64, 32, 512);
  want(false, false, true, 16384, 32, 16, 128);
  want(false, false, false, 16384, 64, 32, 512);
  return wrong != 0;
}
"""


def test_which_sizes_go_past_the_caches(tmp_path):
    _run(STREAMED, tmp_path)


TILE_PLAN = """
#include <stdio.h>
#include <vector>
#include "fade_rules.h"
int main() {
  for (int tiles = 1; tiles <= 1100; tiles = tiles < 300 ? tiles + 1 : tiles + 37)
    for (int units : {1, 2, 7, 64, 129, 256}) {
      const FadeTilePlan p = fade_tile_plan(tiles, units);
      if (p.wgs < 1 || p.wgs > 8 || p.wgs * p.groups > 32) { printf("tiles=%d units=%d: %d x %d workgroups on an XCD\\n", tiles, units, p.groups, p.wgs); return 1; }
      std::vector<int> steps((size_t)tiles * units, 0), slices((size_t)tiles * 64, 0);
      for (int x = 0; x < 8; ++x)
        for (int s = 0; s < 32; ++s) {  // as a workgroup goes through its share
          const int g = s / p.wgs, member = s % p.wgs;
          if (g >= p.groups) continue;
          for (int u = member * p.per_wg; u < fade_tile_end(p, tiles, x, g, member); ++u) {
            const int j = u / units, seq = fade_tile_seq(p, x, g, j), slice = member - fade_tile_first(p, j);
            if (seq >= tiles || fade_tile_of_seq(p, seq) != j || slice < 0 || slice >= fade_tile_parts(p, j)) {
              printf("tiles=%d units=%d: tile %d slice %d of %d\\n", tiles, units, seq, slice, fade_tile_parts(p, j)); return 1;
            }
            ++steps[(size_t)seq * units + u % units];
            slices[(size_t)seq * 64 + slice] = 1;
          }
        }
      for (size_t i = 0; i < steps.size(); ++i)
        if (steps[i] != 1) { printf("tiles=%d units=%d: step %zu of tile %zu taken %d times\\n", tiles, units, i % units, i / units, steps[i]); return 1; }
      for (int t = 0; t < tiles; ++t)
        for (int k = 0; k < fade_tile_parts(p, fade_tile_of_seq(p, t)); ++k)
          if (!slices[(size_t)t * 64 + k]) { printf("tiles=%d units=%d: tile %d has no slice %d\\n", tiles, units, t, k); return 1; }
    }
  return 0;
}
"""


def test_tile_plan_takes_every_step_once(tmp_path):
    """Weight gradients at large batches: the workgroups' shares cover every step of every tile exactly once, and a tile's partial
    sums are the slices that the optimiser adds."""
    _run(TILE_PLAN, tmp_path)


TILE_RANGES = """
#include <stdio.h>
#include "fade_rules.h"
// ranges of a launch per matrix or of equal ranges over all of them (what the sums were formed in by launches of equal workgroups)
static int by_launch(int tiles, int least, int count, int units) {
  double best = 0.0;
  int ranges = 0;
  for (int sp = 1; count >= 2 && sp <= 16; sp *= 2) {
    if (units % sp || units / sp < 8 || tiles * sp < 512) continue;
    const int blocks = tiles * sp;
    const double fill = (double)blocks / (((blocks + 255) / 256) * 256);
    if (fill > best + 1e-9) { best = fill; ranges = sp; }
  }
  if (ranges) return ranges;
  int sp = 1;
  while (sp < 16 && least * sp * 2 <= 256 && units % (sp * 2) == 0 && units / (sp * 2) >= 8) sp *= 2;
  return sp;
}
int main() {
  const int sets[][3] = {{192, 16, 5}, {144, 16, 3}, {152, 24, 3}, {128, 64, 2}, {48, 16, 3}, {32, 16, 2}, {16, 16, 1}, {20, 20, 1}, {24, 24, 1}, {224, 32, 3}, {512, 64, 5}};
  for (const auto &q : sets)
    for (int units = 32; units <= 16384; units = units < 300 ? units + 1 : units + 97) {
      const int r = fade_tile_ranges(q[0], q[1], q[2], units);
      const int least = units < 128 ? (units % 2 == 0 ? 2 : 1) : by_launch(q[0], q[1], q[2], units);
      if (r < least || r > 16 || units % r) { printf("%d tiles, %d blocks of rows: %d ranges, %d before\\n", q[0], units, r, least); return 1; }
      const FadeTilePlan p = fade_tile_plan(q[0] * r, units / r);  // partial sums of a tile: counted in 8 bits
      int most = 0;
      for (int j = 0; j < p.tpg; ++j) most = fade_tile_parts(p, j) > most ? fade_tile_parts(p, j) : most;
      if (most * r > 255) { printf("%d tiles, %d blocks of rows: %d x %d partial sums\\n", q[0], units, r, most); return 1; }
    }
  return 0;
}
"""


def test_tile_ranges_keep_the_sums_short(tmp_path):
    """Weight gradients at large batches: no fp32 chain is longer than with a launch of equal ranges for every workgroup."""
    _run(TILE_RANGES, tmp_path)


TALL_RANGES = """
#include <stdio.h>
#include "fade_rules.h"
int main() {
  for (size_t De = 2048; De <= 8192; De += 64)
    for (size_t Dh = 128; Dh <= 2048; Dh += 128)
      for (size_t B = 1; B <= 20000; B += B % 256 == 1 ? 255 : 1) {
        const int r = fade_tall_ranges(B, Dh, 2 * De);
        if (r == 0) continue;
        const size_t tiles = B / 256 * (Dh / 256), wgs = tiles * r;
        const bool whole = B % 256 == 0 && Dh % 256 == 0 && 2 * De % (64 * r) == 0 && 2 * De / r >= 1024 && r <= 16;
        // one round of the chip, more than half full; two from 128 tiles on
        if (!whole || wgs <= 128 || (wgs > 256 && !(tiles > 128 && r == 2)) || tiles >= 256) {
          printf("B=%zu D_h=%zu D_e=%zu: %zu tiles x %d ranges\\n", B, Dh, De, tiles, r); return 1;
        }
      }
  return fade_tall_ranges(4096, 512, 16384) != 8 || fade_tall_ranges(4096, 256, 16384) != 16 || fade_tall_ranges(8448, 512, 16384) != 2;
}
"""


def test_ranges_of_the_wide_refiners_gradient_fit_a_round(tmp_path):
    _run(TALL_RANGES, tmp_path)
