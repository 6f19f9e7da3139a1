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

// Whether the weight gradients that can be 256 x 256 tiles (`tiles` of them together) leave the grouped launches of their phases, 64 / 128-wide
// tiles beside an activation gradient, and become one launch of equal shares: with 8192 rows of the batch and more, whatever the tiles, and
// from 2048 on when they are three quarters of the compute units or more. Adapting step in us, grouped | in one launch (ranges below):
// D_h = 2048, H = 512 (192 tiles): 2048 rows 648 | 624, 4096 937 | 935, 7000 1550 | 1482, 8192 1537 | 1442, 10001 2212 | 2035, 16384 2780 | 2518;
// D_h = 512, D_cache = 4096, D_e = 8192 (224), 4096 rows 1118 | 1073. Fewer tiles from 8192 rows on: D_h = 2048, H = 384 (152) 8192 1592 | 1590,
// 16384 2908 | 2790; D_h = 1024, H = 512 (48) 8192 990 | 1004, 16384 1678 | 1602; H = 256 (32) 16384 1531 | 1479, 8200 1288 | 1343;
// D_h = 512, D_e = 1024 (16) 8192 780 | 784, 16384 1281 | 1260. D_h = 2048, H = 256 (144) 10001 2056 | 1981, but 8192 1441 | 1553 and 16384
// 2584 | 2636: there the launch sums in 16 ranges, the groups in 2 and 4. Fewer tiles below 8192 rows, with no ranges yet (the better case):
// H = 384 2048 rows 627 | 632; H = 256 4096 867 | 918, 6144 1244 | 1252; H = 128 (128) 4096 843 | 906; D_h = 1024, H = 512 4096 615 | 622.
constexpr bool fade_tile_launch(int rows, int tiles) { return tiles > 0 && (rows >= 8192 || (rows >= 2048 && tiles >= 192)); }

// Equal ranges of the batch that every tile's contraction over `units` blocks of 64 rows is summed in, each from zero, and added up by
// the Adam pass in their order: a sum over thousands of rows in one fp32 accumulator drifts with its length (16384 rows of bf16 operands
// against 64 bits: one chain 8.2e-7 of the result's norm, 12288 + 4096 rows 6.5e-7, four of 4096 4.1e-7). `count` matrices with `tiles`
// tiles together, `least` in the smallest. Below 8192 rows two: what the grouped launches cut W_f and W_fg | W_fv into there.
// From there on the smallest count, of eight blocks or more each, with two pieces or more per compute unit that leaves least of the last round
// of the chip empty; where none divides the batch so, as many as give the smallest matrix a piece per unit. What the shorter chains
// cost, adapting step in us with shares that cut whole tiles | shares of these ranges: D_h = 2048, H = 512, 16384 rows (4 ranges)
// 2578 | 2601, 8192 (4) 1457 | 1485, 4096 (2) 927 | 935; H = 256, 16384 rows (16) 2478 | 2625; D_h = 1024, H = 512, 16384 rows (16)
// 1595 | 1642; D_h = 512, D_cache = 4096, D_e = 8192, 4096 rows (2) 1069 | 1073.
constexpr int fade_tile_ranges(int tiles, int least, int count, int units) {
  if (units < 128) return units % 2 == 0 ? 2 : 1;
  int best = 0, best_rounds = 1;
  for (int r = 1; count >= 2 && r <= 16; r *= 2) {
    const int rounds = (tiles * r + 255) / 256;
    if (units % r != 0 || units / r < 8 || tiles * r < 512) continue;
    if (best == 0 || r * best_rounds > best * rounds) { best = r; best_rounds = rounds; }  // ranges per round: the fill
  }
  if (best > 0) return best;
  int r = 1;
  while (r < 16 && least * r * 2 <= 256 && units % (r * 2) == 0 && units / (r * 2) >= 8) r *= 2;
  return r;
}

// How `tiles` equal contractions of `units` steps each (every range of a weight gradient's tile is one) are shared out over 256
// workgroups, 32 on each of 8 XCDs. On an XCD, `groups` groups of `wgs` workgroups take `tpg` tiles each: the group's tiles lie end to end
// and its members take per_wg steps each, so a tile is cut where a member's share ends and arrives as one partial sum per member that
// worked on it. Small groups (at most eight members) keep the members' starting points few, so that the same members of an XCD's
// groups read the same operand rows at the same time; among them the one that takes the least steps. Tile j of group g of XCD x is
// tile (x tpg + j) groups + g of the order: the g-th neighbours of one another.
struct FadeTilePlan {
  int tpg, wgs, groups, units, per_wg;
};
constexpr FadeTilePlan fade_tile_plan(int tiles, int units) {
  FadeTilePlan best{0, 1, 32, units, 0};
  for (int wgs = 1; wgs <= 8; ++wgs) {
    const int groups = 32 / wgs, tpg = (tiles + 8 * groups - 1) / (8 * groups), per = (tpg * units + wgs - 1) / wgs;
    if (best.tpg == 0 || per < best.per_wg) best = FadeTilePlan{tpg, wgs, groups, units, per};
  }
  return best;
}
constexpr int fade_tile_seq(const FadeTilePlan &p, int xcd, int group, int j) { return (xcd * p.tpg + j) * p.groups + group; }
constexpr int fade_tile_of_seq(const FadeTilePlan &p, int seq) { return seq / p.groups % p.tpg; }  // its place j in its group
constexpr int fade_tile_first(const FadeTilePlan &p, int j) { return j * p.units / p.per_wg; }  // first member on tile j of a group
constexpr int fade_tile_parts(const FadeTilePlan &p, int j) {  // members on it = partial sums of it
  return ((j + 1) * p.units - 1) / p.per_wg - fade_tile_first(p, j) + 1;
}
// end of a member's steps (its first is member * per_wg); the last groups may have fewer tiles than tpg
constexpr int fade_tile_end(const FadeTilePlan &p, int tiles, int xcd, int group, int member) {
  int have = 0;
  while (have < p.tpg && fade_tile_seq(p, xcd, group, have) < tiles) ++have;
  const int end = (member + 1) * p.per_wg;
  return end < have * p.units ? end : have * p.units;
}

// Ranges of the contraction over K = 2 D_e that the gradient at H_coarse (B x D_h of them) is cut into on 256 x 256 tiles, as fp32
// partials that the kernel behind adds; 0: no such tiles (then 128 x 128, cut or not). As many as one round of the chip has workgroups
// for, of 1024 or more each: a few workgroups past a round cost another round, and every range is written and read again. Over half
// the chip, or 128-wide tiles are as fast. From 128 tiles on two, where a range is 4096 or the rows are narrow (D_h <= 512: the
// narrower tiles read the long operand once per 128 columns). The product and the kernel behind in us, 128 x 128 tiles | this rule,
// and (with so many ranges) the first power of two that gives 256 workgroups where that is another:
// D_h = 512, D_e = 8192: 18 tiles 107 | 89, (16) 95; 32 146 | 123; 34 162 | 151, (8) 155; 48 218 | 182, (8) 196; 66 331 | 261, (4) 294;
// 96 404 | 274, (4) 355; 120 397 | 307, (4) 368; 128 398 | 300. D_e = 2048: 32 90 | as that, (4) 94; 66 134 | 118, (4) 137; 96 147 | 130, (4) 155;
// 128 169 | 150. D_h = 1024, D_e = 4096: 64 138 | 107; 136 291 | 260; 200 346 | 291. D_h = 2048, D_e = 4096: 136 235 | 226; 200 272 | 263.
// D_e = 2048, 128 tiles: D_h = 1024 145 | as that, (2) 145; D_h = 2048 106 | as that, (2) 110.
constexpr int fade_tall_ranges(size_t B, size_t Dh, size_t K) {
  if (B % 256 != 0 || Dh % 256 != 0) return 0;
  const size_t tiles = B / 256 * (Dh / 256);
  if (tiles == 0 || tiles >= 256) return 0;
  size_t r = 2;
  while (r < 16 && tiles * r * 2 <= 256 && K % (64 * r * 2) == 0 && K / (r * 2) >= 1024) r *= 2;
  if (K % (64 * r) != 0 || K / r < 1024 || tiles * r <= 128) return 0;
  return tiles < 128 || K / r >= 4096 || Dh <= 512 ? (int)r : 0;
}
