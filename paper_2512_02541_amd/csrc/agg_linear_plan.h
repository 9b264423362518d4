// Launch plan of the projection kernels: which tiles a layer's token rows go to.  Plain host code,
// without the HIP runtime.
#pragma once

#include <stdint.h>

namespace agg {

constexpr int kGemmXcds = 8;
constexpr int kGemmCus = 256;

// Token rows 0 .. split-1 go to tiles of kLargeEdge in a launch of their own (split = 0: there is none),
// the rows from split on to tiles of `edge`: 256 and 128 are linear_kernel's, 64 linear_few_kernel's.
constexpr int kLargeEdge = 256, kSmallEdge = 128, kFewEdge = 64;
struct LinearPlan {
  int64_t split;
  int edge;
};

static inline int64_t few_tiles(int64_t rows, int N, int count) {
  return (rows + kFewEdge - 1) / kFewEdge * (N / kFewEdge) * count;
}

// Times of a launch in microseconds, from what a round of tiles took at K = 1024: 256-wide tiles 33,
// one to a CU; 128-wide ones 20.6 two to a CU and 14 alone, 7 where a CU's last one runs alone behind
// others.  They are taken to follow K, which stores and starts do not; at K = 128 to 4096 and 261 to
// 137 400 rows (184 launches) the choice below took 0.85 to 1.03 of the better single size, once 1.07
// (K = 512, 21 984 rows, three matrices: 46.3 against 43.4 us with small tiles alone).
static inline double linear_time(int64_t rows, int edge, int N, int K, int count) {
  const int64_t tiles = (rows + edge - 1) / edge * ((N + edge - 1) / edge) * count;
  const int64_t mine = (tiles + kGemmXcds - 1) / kGemmXcds;  // of one XCD, which has 32 CUs
  const double k = K / 1024.0;
  if (edge == kLargeEdge) return k * 33.0 * ((mine + 31) / 32);
  const int64_t full = mine / 64, rest = mine % 64;
  return k * (20.6 * full + (rest == 0 ? 0.0 : rest > 32 ? 20.6 : full ? 7.0 : 14.0));
}

// The plan for `count` weight matrices [N, K] applied to the same rows.
static inline LinearPlan plan_linear(int64_t rows, int N, int K, int count) {
  // Up to two 64-wide tiles per CU.  Tiles of 128 / of 64, us, by the number of the latter at C = 1024: 144
  // 13.3 / 6.8; 288 13.3 / 9.7; 352 13.2 / 10.2; 432 13.7 / 10.9; beyond the line 688 14.1 / 16.7; 864 14.8 / 17.8.
  // C = 1280: 260 15.5 / 10.8; 780 17.0 / 20.7.  C = 512: 216 8.7 / 5.7; 344 8.8 / 7.7; 1032 12.9 / 14.9.
  if (few_tiles(rows, N, count) <= 2 * kGemmCus) return {0, kFewEdge};
  // Large tiles move half the bytes per product, small ones fill the chip and its last round: the
  // rows of whole rounds of large tiles go to them and the others to small tiles, if that is at
  // least 6 % ahead of large tiles alone and 3 % of small ones (a second launch costs 4 us).  Measured for the Q/K/V and
  // the output projection at C = 1024, large / small / chosen, us:
  // 5 496 rows 58 + 32 / 46 + 20 / 45 + 21; 10 992 rows 90 + 35 / 85 + 32 / 82 + 31; 32 976 rows
  // 232 + 110 / 270 + 104 / 229 + 105; 137 400 rows 817 + 325 / 1022 + 374 / large.
  const int64_t per_m = (int64_t)((N + 255) / 256) * count;
  const int64_t gm = (rows + 255) / 256;
  const int64_t whole = gm * per_m / kGemmCus * kGemmCus / per_m;  // token tiles that fill whole rounds
  const int64_t split = whole * 256 < rows ? whole * 256 : 0;
  const double large = linear_time(rows, kLargeEdge, N, K, count);
  const double small = linear_time(rows, kSmallEdge, N, K, count);
  // The others take tiles of 64 where these are few enough: 7.5 us up to one per CU, 11 up to two, where a
  // single round of small tiles takes 14 to 20.  Whole block, others in small tiles / in tiles of 64 (and
  // then also where that makes two launches the better choice): 16 frames of 37x37, 239 others, 731.5 /
  // 722.3; per-frame, 8 frames 188.5 / 181.3; 96 frames, 832, 1879 / 1864; 42 frames of 28x37 622 / 607;
  // 167 frames of 16x16, 12 heads, 364 / 353.
  const int64_t few_rest = few_tiles(rows - split, N, count);
  const double rest_time = few_rest > 2 * kGemmCus ? linear_time(rows - split, kSmallEdge, N, K, count)
                                                   : K / 1024.0 * (few_rest > kGemmCus ? 11.0 : 7.5);
  const double both = split ? linear_time(split, kLargeEdge, N, K, count) + rest_time + 4.0 : large;
  if (small < 0.97 * large && small <= 1.03 * both) return {0, kSmallEdge};
  if (both >= 0.94 * large) return {0, kLargeEdge};
  return {split, few_rest <= 2 * kGemmCus ? kFewEdge : kSmallEdge};
}

}  // namespace agg
