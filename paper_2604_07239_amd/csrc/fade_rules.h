// fade_rules.h — index arithmetic of the kernels as plain constexpr C++ (usable in device code, and by a host compiler alone).
#pragma once
#include <stddef.h>

// Columns of one lane in a strip of 64 columns (from n0) of a row-major matrix with N columns whose first element is at `off`, a
// multiple of four, of the state arrays: four neighbouring columns from n0 + 4 q (q < 16) of row m. `left`: how many of them exist
// (0 or less: none). `vec`: they may be accessed as one 16-byte piece in every row, which takes rows that are whole pieces: with
// 5 or 6 columns most rows start between two pieces, also where four columns are left.
struct FadeStripLane {
  size_t idx;
  int left;
  bool vec;
};
constexpr FadeStripLane fade_strip_lane(size_t off, int N, int n0, int m, int q) {
  const int n = n0 + 4 * q, left = N - n < 4 ? N - n : 4;
  return FadeStripLane{off + (size_t)m * (size_t)N + (size_t)n, left, N % 4 == 0};
}
