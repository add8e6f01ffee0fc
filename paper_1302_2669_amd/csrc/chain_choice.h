// Choice between the chain mappings: one chain per lane (chain_body.h), split
// over L lanes (chain_split.h), one chain per wave (chain_lone.hip), or the
// first two side by side.
//
// The unit is SIMD cycles, per update of 64 chains or per run, from canonical
// starts, p = 0.1, L = 2 to 25, 16 to 600000 chains, 1 to 256 sweeps, both noise
// models (5100 batches: the choice takes 0.2% longer than the best measured mapping
// on average, and more than a tenth longer in 25, at most 1.3 times, where two of
// them cross).
#pragma once

#include <math.h>

#include "internal.h"

namespace mcmc {

// One chain per lane, w waves on the SIMD: a lone wave waits about as long as it
// issues; from two waves on each adds its issue time.  Short rows leave less to
// amortise a row's fixed work over.  Measured and estimated, L = 13: 1 wave 142 /
// 147, 2 184 / 187, 3 242 / 248, 5 366 / 371; L = 3: 283 / 275, 353 / 346, 466 /
// 458, 710 / 682; L = 25: 154 / 141, 196 / 187, 259 / 253, 386 / 385.
__host__ __device__ inline double one_lane_issue(int L) {
  return (58.5 + 480.0 / (L * L)) * (L > 16 ? 1.11 : 1.0);
}
__host__ __device__ inline double one_lane_cycles(int L, double w) {
  return w <= 1.0 ? one_lane_issue(L) + 63.0 + 300.0 / L
                  : one_lane_issue(L) * w + 46.0 + 230.0 / L;
}

// Split over L lanes, a wave's sweep: its lanes' Philox blocks with their
// counts (220 cycles a block) and four phases of one or two row words; and for W
// waves' worth of chains on the SIMD.  Measured and estimated at W = 1: L = 3 294 /
// 267, 9 107 / 103, 13 109 / 105, 17 112 / 115, 25 99 / 103; at 2: 479 / 457, 202 /
// 192, 190 / 199, 208 / 222, 203 / 199.
__host__ __device__ inline double split_cycles(int L) {
  const int blocks = L / 2, words = (L + 15) / 16;
  const double sweep = 220.0 * blocks + 4.0 * (108.0 * words + 23.5);
  return sweep * 64.0 / (split_tile(L) * 2.0 * L * (L - 1));
}
__host__ __device__ inline double split_cycles(int L, double W) {
  return split_cycles(L) * W + 6.0 + 630.0 / (L * L);
}

// A run of `cycles` split, with what its tiles cost beyond a one-lane launch's: each
// spills at its start (0.7 to 2.2 KB a lane: 0.7 GB for 64016 chains at L = 13), comes
// from one counter, and waits for its rows and its stores.  Short runs last as long
// as that takes, some 13 ns a tile, long ones hide most of it (64000 chains at L = 13:
// 363 us for 3 sweeps as for 6, 411 for 14; one lane per chain 161, 217, 360; with
// tiles by wave number instead of the counter 288 for 3, but 10% more for long runs of
// a ragged batch).
__host__ __device__ inline double split_run(int L, double tiles, double cycles, bool beside) {
  const double start = fmin(25600.0, 6000.0 + 88.0 * tiles);
  return fmax(start + (beside ? 24.0 : 68.0) * tiles + 165.0 * L * L,
              start + (beside ? 12.0 : 16.0) * tiles + 195.0 * L * L + cycles);
}

// Both mappings side by side: whole one-lane waves per SIMD, the chains beyond
// them split, running in what the waves leave of the SIMD.  Bound by the
// one-lane waves' own time or by the issue of both.  W = 2.44, L = 25, 50 sweeps:
// 6794 us one-lane, 5466 with two waves; W = 3.3, L = 9, 500 sweeps: 10703, 8342 (two
// waves), 8545 (three); W = 6.2, L = 13, 150 sweeps: 9820, 8680.
__host__ __device__ inline double both_cycles(int L, int h, double rest) {
  return fmax(one_lane_cycles(L, h),
              one_lane_issue(L) * h + 0.82 * split_cycles(L, rest) + 22.5);
}

// The mapping of a batch of `chains` equal chains of `sweeps` sweeps, in waves' worth
// of chains per SIMD.  One chain per lane is left only for a gain of 5%.
enum ChainMapping { CHAINS_ONE_LANE, CHAINS_SPLIT, CHAINS_LONE, CHAINS_BOTH };
struct ChainChoice {
  ChainMapping mapping;
  int waves;     // CHAINS_BOTH: one-lane waves per SIMD
  double gain;   // cycles less than one chain per lane, by the estimate
};
__host__ __device__ inline ChainChoice lanes_choice(int L, int64_t chains, int64_t sweeps,
                                                    int simds, bool beside) {
  const double W = (double)chains / ((double)TILE * simds);
  const double updates = (double)sweeps * 2.0 * L * (L - 1);
  ChainChoice c{CHAINS_ONE_LANE, 0, 0.0};
  const double lanes = 0.947 * one_lane_cycles(L, ceil(W)) * updates;
  double best = lanes;
  const double all = split_run(L, (double)chains / split_tile(L), split_cycles(L, W) * updates, false);
  if (all < best) {
    best = all;
    c.mapping = CHAINS_SPLIT;
  }
  const int top = (int)fmin(floor(W), 1e6);
  for (int h = top; beside && h >= 1 && h >= top - 1; --h) {
    if (W <= h) continue;
    const double rest = (W - h) * TILE * simds / split_tile(L);
    const double t = split_run(L, rest, both_cycles(L, h, W - h) * updates, true);
    if (t < best) {
      best = t;
      c.mapping = CHAINS_BOTH;
      c.waves = h;
    }
  }
  c.gain = lanes - best;
  return c;
}

// Whether a batch of which any part may run `sweeps` sweeps (the rest fewer, in the
// one-lane launch) gets a launch for split chains, forked from and joined to the
// caller's stream: if that saves some part of it more than its 20 us (2000
// syndromes x 16 chains at L = 5 with 5 sweeps: 222 us beside an empty launch, 164
// alone; one at L = 3 133 and 105).
inline bool batch_splits(int L, int64_t n, int64_t per_item, int64_t sweeps, int simds) {
  for (int64_t part = n; part > 0; part /= 2)
    if (lanes_choice(L, part * per_item, sweeps, simds, true).gain > 48000.0) return true;
  return false;
}

// One chain per wave (codes whose draws fill the lanes, LONE_L_MIN) beats L lanes
// while every SIMD has one wave at most (0.5 to 0.9 of the time; 256 sweeps at L = 13
// 0.57), with two from L = 10 on (0.75 to 1.0; L = 8 and 9 0.9 to 0.96 for 300
// sweeps, 1.0 for 64, 1.1 for 8; L = 6 and 7 1.1 to 1.3).
inline bool lone_fits(int L, int64_t chains, int64_t sweeps, int simds) {
  const int two_waves = sweeps >= 64 ? 8 : 10;
  return L >= LONE_L_MIN && chains <= (int64_t)simds * (L >= two_waves ? 2 : 1);
}
// And one chain per lane, from some sweeps on (its waves have no counter to wait for:
// 16 chains at L = 13 75 us for one sweep, 95 one-lane; 1600 112 and 106).
inline bool lone_pays(int L, int64_t chains, int64_t sweeps) {
  return 0.947 * one_lane_cycles(L, 1.0) * (double)sweeps * 2.0 * L * (L - 1) >
         12900.0 + 20.0 * (double)chains;
}

// The mapping of a uniform batch; beside: its split rest may run on another stream.
inline ChainChoice chain_choice(int L, int64_t chains, int64_t sweeps, int simds, bool beside) {
  if (lone_fits(L, chains, sweeps, simds))
    return {lone_pays(L, chains, sweeps) ? CHAINS_LONE : CHAINS_ONE_LANE, 0, 0.0};
  return lanes_choice(L, chains, sweeps, simds, beside);
}

}  // namespace mcmc
