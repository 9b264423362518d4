// Launch plan of the attention kernels: which workgroups a (batch, head) pair's queries are cut into
// and where rows that leave the fast path's range are redone.  Plain host code, without the HIP
// runtime.
#pragma once

#include <stdint.h>

namespace agg {

constexpr int kWaves = 4;  // wavefronts per workgroup
constexpr int kCus = 256;

// How many queries a wavefront owns: kQB blocks (the units of the key loop's pipeline) of kJ
// tiles of 16.  The full width is kQB = kJ = 2; narrower workgroups finish a launch (plan_tiles).
constexpr int wave_queries(int qb, int j) { return 16 * qb * j; }
constexpr int kQTile = kWaves * wave_queries(2, 2);  // queries of a full-width workgroup (256)

// How a pair's queries are cut: n_full workgroups of kQTile queries, then n_tail of tail_q.
// The launch order is one list of all tiles, pair by pair (tails_last 0), or all full tiles and
// then all tails (1).
struct TilePlan {
  int n_full, n_tail, tail_q, tails_last;
  int split;  // all workgroups are narrow ones of eight wavefronts that share their keys
};

// Launch plan: which workgroups a pair's queries are cut into.
//
// A workgroup's whole key loop is one piece of work, so a launch of a few rounds loses up to a
// round to its last, partly filled one, and a short sequence pays for up to 255 queries that do
// not exist.  Narrow workgroups (192 or 128 queries) lose less there; they are not free, because
// every K/V fragment then feeds fewer products.  Measured over 122 compacted key tiles with 16 pairs, in
// units of what two full-width workgroups on one CU take (201 us): a pair of 192 0.79, of 128 0.58;
// one alone on its CU 0.55 (256 queries), 0.44 (192), 0.34 (128); over 73 tiles, and with 12 pairs, the same within
// 0.01.  Rows in place 0.80, 0.60; 0.58, 0.48, 0.37; through the index list 0.84, 0.63; 0.55, 0.47, 0.37.  The costs
// below are those of a prologue that has since become shorter; the compacted figures in their place would
// change one plan in ninety, by less than 3 % as the model sees it.  The plan takes the narrow
// tail that the cost model below puts at least 1.5 % ahead of full-width workgroups alone.
// Measured with it, attention alone: 10 frames of 37x37 patches, 16 heads, 345 us instead of 373; 24 frames of
// 28x37, 12 heads, ordinary attention, 1452 instead of 1503.  The model knows
// neither the key source nor the number of keys: over 120 random launches for which it takes narrow
// workgroups (all three sources, 1 to 408 key tiles, 4 to 32 heads, 1 to 70 frames) they took 0.70 to
// 1.03 of full-width ones alone, half of them under 0.91; the worst are 10 frames of 37x37 with 20 heads, 484 / 471 us,
// and 53 frames of 16x16 through the index list with 20 heads, 259 / 252.
struct TileCost {
  int queries;
  double paired, alone;  // on a CU that holds two workgroups / this one only
};
static const TileCost kFullCost = {kQTile, 1.0, 0.535};
static const TileCost kTailCosts[] = {{192, 0.79, 0.45}, {128, 0.565, 0.355}};

// Time of a CU that runs `full` full-width and then `tail` narrow workgroups, two at a time.
static inline double cu_time(int64_t full, int64_t tail, const TileCost& c) {
  double t = 0.5 * (full * kFullCost.paired + tail * c.paired);
  if ((full + tail) & 1) t += tail ? c.alone - 0.5 * c.paired : kFullCost.alone - 0.5 * kFullCost.paired;
  return t;
}
// Time of a launch: the full-width workgroups are dealt out evenly, each narrow one goes to the
// CU that is free first.
static inline double launch_time(int64_t full, int64_t tail, const TileCost& c) {
  const int64_t extra = full % kCus;
  const int64_t cus[2] = {kCus - extra, extra};
  const int64_t f[2] = {full / kCus, full / kCus + 1};
  int64_t t[2] = {0, 0};
  double end = cu_time(f[extra ? 1 : 0], 0, c);
  while (tail > 0) {
    const int k = (cus[1] > 0 && cu_time(f[1], t[1], c) < cu_time(f[0], t[0], c)) ? 1 : 0;
    ++t[k];
    tail -= cus[k];
    const double now = cu_time(f[k], t[k], c);
    end = now > end ? now : end;
  }
  return end;
}

static inline TilePlan plan_tiles(int64_t NQ, int npairs, int64_t key_tiles) {
  const int64_t most = NQ / kQTile;
  TilePlan best = {(int)((NQ + kQTile - 1) / kQTile), 0, 0, 0, 0};
  // At most one narrow workgroup per CU: eight wavefronts that share the keys give each SIMD two to
  // alternate between.  The call, us, four / eight wavefronts: 2 frames of 37x37 with 8 heads, every
  // token a key (43 key tiles), 28.2 / 24.5; through the index list 31.7 / 28.0; one frame of 37x37
  // with 16 heads (22 tiles) 16.6 / 15.1.  With few tiles the eight can be behind: 2 frames of 16x16, 6 compacted
  // tiles, 8.9 / 9.4.  One key tile cannot be shared.
  if (key_tiles >= 2 && npairs <= kCus && npairs * ((NQ + 127) / 128) <= kCus)
    return {0, (int)((NQ + 127) / 128), 128, 1, 1};
  if (npairs * NQ > INT32_MAX) return best;  // far past the sizes at which a tail matters
  // With at least a pair per CU the rounds are many, and what is left to gain are the queries
  // that do not exist; the tails then follow their pair's other tiles, whose keys they share.
  // Per-frame attention, 90 frames of 37x37 patches: 662 us instead of 682.  Under eight key tiles they
  // are left out: while such launches had a second one behind them, 50 frames of 16x16 took 51.0 us
  // with them and 50.2 without.  (Now that they redo rows in place it is 39.9 and 40.4; 300 frames of
  // 5x10 37.6 and 50.0.)
  const bool by_pair = npairs >= kCus;
  if (by_pair && key_tiles < 8) return best;
  double least = by_pair ? (double)best.n_full : launch_time(npairs * (int64_t)best.n_full, 0, kFullCost);
  least *= 0.985;
  // full-width workgroups per pair: all that fit, one fewer, and what fills whole rounds
  const int64_t round = 2 * kCus, rounds = npairs * most / round;
  const int64_t tries[] = {most, most - 1, rounds * round / npairs, (rounds - 1) * round / npairs};
  for (int i = 0; i < (by_pair ? 2 : 4); ++i) {
    const int64_t n = tries[i], left = NQ - n * kQTile;
    if (n < 0 || left == 0) continue;
    for (const TileCost& c : kTailCosts) {
      const int64_t m = (left + c.queries - 1) / c.queries;
      const double t = by_pair ? n + m * c.paired : launch_time(npairs * n, npairs * m, c);
      if (t < least) {
        least = t;
        best = {(int)n, (int)m, c.queries, by_pair ? 0 : 1, 0};
      }
    }
  }
  return best;
}

// Whether a launch that is not split redoes rows itself, without a second launch.
//
// An idle second launch is 1 to 17 % of a call with few key tiles, and where one query needs the
// general path the others no longer wait for it; with long key loops the idle launch is lost in
// them, and there redoing everything 128 queries at a time, which reads the keys twice, costs more.
// Attention alone, us, second launch / redo in place, by the width of the last workgroups:
//   full  rows, per-frame, 300 frames of 5x10, 1 tile 58.2 / 49.7;  50 frames of 16x16, 5 tiles 43.6 / 40.0;
//         5 frames of 37x37, 22 tiles 43.0 / 41.1;  ordinary, 5 frames, 108 tiles 168.5 / 166.5
//         compacted, 30 frames of 16x16, 3 tiles 22.5 / 20.6;  12 frames, 16 tiles 24.0 / 22.2;  3 frames of
//         37x37, 12 heads, 44 tiles 45.0 / 43.1;  30 frames, 12 heads, 101 tiles 639 / 633
//         indexed, 12 frames of 16x16, 16 tiles 24.7 / 23.0;  5 frames of 37x37, 45 tiles 81.3 / 79.3
//   192   compacted, 20 frames of 16x16, 3 tiles 18.8 / 16.5;  2 frames of 37x37, 33 tiles 30.7 / 28.7;
//         10 frames, 122 tiles 348 / 344;  indexed, 10 frames 372 / 369;  rows, 2 frames, 43 tiles 36.9 / 35.0
//         (beyond the line: compacted, 12 frames, 133 tiles 460 / 456;  20 frames, 222 tiles 1185 / 1183)
//   128   compacted, 9 frames, 1 tile 29.0 / 26.1;  3 frames, 44 tiles 54.3 / 52.2;
//         rows, per-frame, 90 frames, 22 tiles 669 / 662;  300 frames of 24x24, 10 tiles 558 / 540
// One token out of range (a workgroup of every head) / every workgroup: compacted, 10 frames of 37x37 584 / 399 and
// 535 / 639, the largest loss; indexed, 8 frames of 16x16, 20 heads 40.4 / 44.0 and 41.7 / 48.4; rows, ordinary, 5 frames
// 340 / 230 and 281 / 290; per-frame, 90 frames 704 / 666 and 1533 / 1543; 50 frames of 16x16 56.4 / 41.0
// and 101.9 / 94.1.
static inline bool redo_in_place(int64_t key_tiles) { return key_tiles < 128; }

}  // namespace agg
