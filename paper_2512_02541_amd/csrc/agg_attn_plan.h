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
// every K/V fragment then feeds fewer products.  Measured over 121 key tiles with 16 pairs, in
// units of what two full-width workgroups on one CU take (201 us): a pair of 192 0.79, of 128 0.56;
// one alone on its CU 0.53 (256 queries), 0.45 (192), 0.36 (128).  The plan takes the narrow
// tail that the cost model below puts at least 1.5 % ahead of full-width workgroups alone.
// Measured with it: 10 frames of 37x37 patches, 16 heads, 367 us instead of 401 (attention
// alone); two frames of 16x16 patches 27.6 instead of 33.3 (the whole layer).  The model knows
// neither the key source nor the number of keys: over 120 random launches for which it takes narrow
// workgroups (all three sources, 10 to 670 key tiles, 4 to 32 heads, 1 to 73 frames) they took 0.69 to
// 1.03 of full-width ones alone, half of them under 0.91; the worst are 53 frames of 16x16 through
// the index list with 20 heads, 474 / 462 us, and per-frame attention, 16 frames of 28x37, 79 / 77.
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
  // token a key (43 key tiles), 30.2 / 25.0; through the index list 42.3 / 35.2; one frame of 37x37
  // with 16 heads (22 tiles) 18.7 / 17.6.  One key tile cannot be shared.
  if (key_tiles >= 2 && npairs <= kCus && npairs * ((NQ + 127) / 128) <= kCus)
    return {0, (int)((NQ + 127) / 128), 128, 1, 1};
  if (npairs * NQ > INT32_MAX) return best;  // far past the sizes at which a tail matters
  // With at least a pair per CU the rounds are many, and what is left to gain are the queries
  // that do not exist; the tails then follow their pair's other tiles, whose keys they share.
  // Per-frame attention, 90 frames of 37x37 patches: 710 us instead of 728.  Under eight key tiles they
  // are left out: while such launches had a second one behind them, 50 frames of 16x16 took 51.0 us
  // with them and 50.2 without.  (Now that they redo rows in place it is 42.6 and 43.5; 300 frames of
  // 5x10 37.2 and 49.1.)
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
// An idle second launch is 1 to 18 % of a call with few key tiles, and where one query needs the
// general path the others no longer wait for it; with long key loops the idle launch is lost in
// them, and there redoing everything 128 queries at a time, which reads the keys twice, costs more.
// Attention alone, us, second launch / redo in place, by the width of the last workgroups:
//   full  rows, per-frame, 300 frames of 5x10, 1 tile 57.4 / 48.7;  50 frames of 16x16, 5 tiles 47.7 / 43.4;
//         5 frames of 37x37, 22 tiles 43.1 / 41.0;  ordinary, 5 frames, 108 tiles 170.0 / 167.9
//         compacted, 30 frames of 16x16, 3 tiles 28.3 / 26.3;  12 frames, 16 tiles 26.7 / 24.9;  3 frames of
//         37x37, 12 heads, 44 tiles 51.0 / 49.0;  30 frames, 12 heads, 101 tiles 670 / 656
//         indexed, 12 frames of 16x16, 16 tiles 27.5 / 26.0;  5 frames of 37x37, 45 tiles 88.1 / 86.2
//   192   compacted, 20 frames of 16x16, 3 tiles 21.9 / 19.8;  2 frames of 37x37, 33 tiles 34.1 / 32.5;
//         10 frames, 122 tiles 353 / 350;  indexed, 10 frames 379 / 376;  rows, 2 frames, 43 tiles 37.8 / 35.7
//         (beyond the line: compacted, 12 frames, 133 tiles 488.5 / 485.0;  20 frames, 222 tiles 1254 / 1252)
//   128   compacted, 9 frames, 1 tile 43.5 / 40.9;  3 frames, 44 tiles 55.6 / 53.7;
//         rows, per-frame, 90 frames, 22 tiles 667 / 665;  300 frames of 24x24, 10 tiles 564 / 541
// One query out of range / every workgroup: compacted, 10 frames of 37x37 573 / 351 and 512 / 596, the
// largest loss; indexed, 8 frames of 16x16, 20 heads 33.2 / 36.1 and 32.7 / 36.5; rows, ordinary, 5 frames
// 373 / 231 and 284 / 288; per-frame, 90 frames 737 / 654 and 1629 / 1515; 50 frames of 16x16 64.6 / 43.5
// and 118.8 / 102.5.
static inline bool redo_in_place(int64_t key_tiles) { return key_tiles < 128; }

}  // namespace agg
