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

// Time of one launch for `count` weight matrices [N, K], in microseconds.  A launch goes by rounds: a
// CU runs one 256-wide tile or two of the others at a time, and an XCD has 32 CUs.  What a round costs has
// a part that follows K (the steps) and one that does not (the stores, the residual's loads), and a round of at
// most one small tile per CU is cheaper than a full one.
//
// The constants are fitted to 5 137 sizes timed with every choice of tiles, on three boxes, with what
// surrounds a projection in a block: its input has just been written, the residual a while ago.  N = K = 64 to
// 4096 in 19 widths, one matrix with the residual and three without, up to 300 000 rows.  Nine launches in ten
// take 0.73 to 1.20 (tiles of 128) and 0.90 to 1.13 (of 256) of the time given here.
static inline double linear_time(int64_t rows, int edge, int N, int K, int count, bool residual) {
  const int64_t across = (N + edge - 1) / edge;
  const int64_t tiles = (rows + edge - 1) / edge * across * count;
  const int64_t mine = (tiles + kGemmXcds - 1) / kGemmXcds;  // of one XCD
  const int64_t at_once = edge == kLargeEdge ? 32 : 64;
  const int64_t full = mine / at_once, last = mine % at_once;
  const double part = (double)last / at_once, rounds = full + part;
  const double k = K / 1024.0;
  if (edge == kLargeEdge) {
    // channels past the end of a tile are not stored
    const double stored = rounds * N / (double)(across * edge);
    return 2.7 + (full + (last > 0)) * (0.6 + 24.6 * k) + stored * (residual ? 9.1 : 3.9);
  }
  const bool half = last > 0 && last <= 32;  // at most one tile per CU in the last round
  const int64_t whole = full + (last > 32);
  if (edge == kFewEdge) return 2.0 + whole * (1.5 + 6.0 * k) + half * (0.7 + 4.4 * k);
  // Beyond what the last cache level holds, every 128-wide column of tiles reads the rows again.
  const bool far = 2.0 * rows * (K + (count + residual) * (double)N) > 300e6;
  return 2.5 + rounds * (1.4 + (residual ? 1.7 : 0.0) + (far ? 1.1 : 0.0)) +
         k * (full * 17.3 + part * 5.3 + (last > 32 ? 11.7 : !half ? 0.0 : full ? 6.0 : 10.7));
}

// The plan for `count` weight matrices [N, K] applied to the same rows.
static inline LinearPlan plan_linear(int64_t rows, int N, int K, int count, bool residual) {
  // Up to two 64-wide tiles per CU: the best choice, or within 1 % of it, at all of 957 sizes.  Tiles of 128 / of
  // 64, us, by the number of the latter at C = 1024, launches back to back: 144 13.3 / 6.8; 288 13.3 / 9.7; 432 13.7 /
  // 10.9; beyond the line 688 14.1 / 16.7; 864 14.8 / 17.8.  (Exceptions there: launches that would just begin their
  // second half round of tiles of 128, 1065 rows of 1280 channels, three matrices, 22.5 / 19.7; 398 of 3072 49.6 / 39.9.)
  if (few_tiles(rows, N, count) <= 2 * kGemmCus) return {0, kFewEdge};
  // Large tiles move half the bytes per product, small ones fill the chip and its last round; or the rows of
  // whole rounds of large tiles go to them and the others to small ones, or to tiles of 64 where these are few
  // enough, by a second launch.  At the 5 137 sizes, where a second launch was taken when 2 % ahead, the choice was
  // 1.003 of the best one on average and 1.15 at worst (23 983 rows of 768 channels, 42.0 us in two launches, 36.5 in
  // tiles of 128); times that only followed K, 6 % ahead, gave 1.009.  Whole blocks gain less by a second launch than
  // the projections' own times say (idle CUs leave the others more power, which may be why).  In per-frame blocks of
  // 130 drawn sizes, each projection with and without its second launch, a predicted lead of 8 us over large
  // tiles was mostly between a gain of 7 and a loss of 9, one of 16 us and more a gain of 4 to 20; 2 % ahead took 1.0012 of the best choice (11 220 rows of
  // 512 channels 68.6 us, 66.6 without; 51 678 of 1024 636 / 624; 59 337 of 768 558 / 548), the leads asked for
  // here 1.0006.  At C = 1024, tiles of 256 / of 128 / two launches, us: Q/K/V 5 651 rows 52 / 39 / 36; 21 960 135 / 141 /
  // 119; 92 600 488 / 625 / 499; output 5 651 rows 29 / 16; 21 960 64 / 57 / 60; 103 206 240 / 264 / 236 (within
  // a block the same).
  const int64_t per_m = (int64_t)((N + 255) / 256) * count;
  const int64_t gm = (rows + 255) / 256;
  const int64_t whole = gm * per_m / kGemmCus * kGemmCus / per_m;  // token tiles that fill whole rounds
  const int64_t split = whole * 256 < rows ? whole * 256 : 0;
  const double large = linear_time(rows, kLargeEdge, N, K, count, residual);
  const double small = linear_time(rows, kSmallEdge, N, K, count, residual);
  if (split) {
    const int rest = few_tiles(rows - split, N, count) <= 2 * kGemmCus ? kFewEdge : kSmallEdge;
    const double two = linear_time(split, kLargeEdge, N, K, count, residual) +
                       linear_time(rows - split, rest, N, K, count, residual);
    if (two + (residual ? 5 : 2) < small && 1.02 * two + 5 < large) return {split, rest};
  }
  return {0, small < large ? kSmallEdge : kLargeEdge};
}

}  // namespace agg
