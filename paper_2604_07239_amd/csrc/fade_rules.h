// fade_rules.h — rules on sizes and index arithmetic as plain constexpr C++ (usable in device code, and by a host compiler alone).
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

// Whether a step's weights and optimiser state are accessed past the caches (nt), given the parameter count, the streams and D_h:
// they are when they do not survive in the 256 MB Infinity Cache from one step to the next. Same bits either way.
//   * bf16, adapting: weight, gradient and two moments, and some twenty activation rows of D_h per stream, 184 MB and more. Step in
//     us with plain and nt accesses (state + activations in MB): B = 128 / 256, D_h = 2048, H = 128 262 -> 270 (174), 313 -> 299 (192);
//     B = 128, H = 192 275 -> 279 (182); B = 256, H = 64 306 -> 295 (184); B = 16, H = 128 / 256 / 512 251 -> 266 (158),
//     264 -> 275 (174), 315 -> 301 (206); D_h = 512, B = 1024 / 1536 / 2048 250 -> 257 (111), 286 -> 288 (153), 350 -> 332 (195);
//     D_h = 2048, B = 1024, H = 256 443 -> 396 (317).
//   * bf16, frozen: the one copy of the weights, from 128 MB on. D_h = 512, B = 8192 / 16384 (64 / 128 MB of them per-stream):
//     146.6 -> 147.0, 233.4 -> 220.7.
//   * fp32: never. B = 300 / 512, D_h = 2048, H = 512 3452 -> 3655, 3894 -> 4275: its products fetch the masters themselves, so the
//     optimiser's accesses are what brings them into the cache (D_h = 512, B = 2048 / 4096, where W_U is most of it: 2452 -> 2478,
//     4313 -> 4245).
constexpr bool fade_streamed(bool bf16, bool online, size_t params, size_t B, size_t Dh) {
  const size_t MB = (size_t)1 << 20;
  return bf16 && (online ? 16 * params + 20 * 2 * B * Dh >= 184 * MB : 2 * params >= 128 * MB);
}
