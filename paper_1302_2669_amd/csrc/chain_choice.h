// Choice between the chain mappings: one chain per lane (chain_body.h), split
// over L lanes (chain_split.h), one chain per wave (chain_lone.hip), or the
// first two side by side.
//
// The unit is SIMD cycles per update of 64 chains, measured on full and partly
// filled chips (canonical starts, p = 0.1, L from 3 to 25).
#pragma once

#include <math.h>

#include "internal.h"

namespace mcmc {

// One chain per lane, w waves on the SIMD: a lone wave waits 2.7 times as long
// as it issues; from two waves on each adds its issue time.  Short rows leave
// less to amortise a row's fixed work over.  L = 13, measured and estimated: 1
// wave 186 / 181, 2 217 / 208, 3 272 / 275, 5 406 / 408; L = 5: 187 / 227, 249 /
// 260, 337 / 344, 521 / 512.
__host__ __device__ inline double one_lane_issue(int L) {
  return (64.0 + 500.0 / (L * L)) * (L > 16 ? 1.07 : 1.0);
}
__host__ __device__ inline double one_lane_cycles(int L, double w) {
  return one_lane_issue(L) * (w <= 1.0 ? 2.7 : w + 1.1);
}

// Split over L lanes, a wave's sweep: its lanes' Philox blocks with their
// counts (250 cycles a block) and four phases of one or two row words.
// Measured and estimated: L = 3 203 / 204, 5 139 / 140, 9 97 / 99, 13 106 / 106,
// 16 86 / 86, 17 116 / 118, 21 93 / 89, 25 112 / 107.
__host__ __device__ inline double split_cycles(int L) {
  const int blocks = L / 2, words = (L + 15) / 16;
  const double sweep = 250.0 * blocks + 4.0 * (110.0 * words + 26.0);
  return sweep * 64.0 / (split_tile(L) * 2.0 * L * (L - 1));
}

// Whether a batch of `chains` equal chains of `sweeps` sweeps runs faster
// split: one-lane waves come whole to a SIMD, the split work spreads evenly,
// but its waves take some 40000 cycles longer to set up (3000 syndromes at L = 6
// without a sweep: 171 us one-lane, 193 split).
__host__ __device__ inline bool split_pays(int L, int64_t chains, int64_t sweeps, int simds) {
  const double W = (double)chains / ((double)TILE * simds);
  const double gain = one_lane_cycles(L, ceil(W)) - (split_cycles(L) * W + 20.0);
  return gain * (double)sweeps * 2.0 * L * (L - 1) > 40000.0;
}

// Both mappings side by side: whole one-lane waves per SIMD, the chains beyond
// them split, running in what the waves leave of the SIMD.  Bound by the
// one-lane waves' own time or by the issue of both.  W = 2.44, L = 25: 7133 us
// one-lane, 5728 with two waves; W = 3.3, L = 9: 8374, 6908 (two waves), 7202
// (three); W = 6.2, L = 13: 8587, 7641.
__host__ __device__ inline double both_cycles(int L, int h, double rest) {
  return fmax(one_lane_cycles(L, h), one_lane_issue(L) * h + split_cycles(L) * rest + 20.0);
}

// The one-lane waves per SIMD of a batch that runs side by side, 0 if one
// mapping alone is as good: the estimate has to win 7%, its own error (W = 3.9:
// L = 17 loses 1% at an estimate of 0.94; W = 12.7 and above gain 0 to 4%).
__host__ __device__ inline int both_waves(int L, int64_t chains, int64_t sweeps, int simds) {
  const double W = (double)chains / ((double)TILE * simds);
  const double alone =
      fmin(one_lane_cycles(L, ceil(W)),
           split_pays(L, chains, sweeps, simds) ? split_cycles(L) * W + 20.0 : INFINITY);
  const int top = (int)fmin(floor(W), 1e6);
  int best = 0;
  double cycles = 0.93 * alone;
  for (int h = top; h >= 1 && h >= top - 1; --h) {
    const double c = both_cycles(L, h, W - h);
    if (W > h && c < cycles) {
      cycles = c;
      best = h;
    }
  }
  const double gain = (alone - cycles) * (double)sweeps * 2.0 * L * (L - 1);
  return gain > 40000.0 ? best : 0;
}

// One chain per wave (codes whose draws fill the lanes, LONE_L_MIN) pays up to
// two waves per SIMD: 1966 chains at L = 13 234 us against 255 split, 2560 288
// against 262.
inline bool lone_pays(int L, int64_t chains, int64_t sweeps, int simds) {
  return L >= LONE_L_MIN && chains <= 2 * (int64_t)simds &&
         split_pays(L, chains, sweeps, simds);
}

// The mapping of a uniform batch; beside: its split rest may run on another stream.
enum ChainMapping { CHAINS_ONE_LANE, CHAINS_SPLIT, CHAINS_LONE, CHAINS_BOTH };
struct ChainChoice {
  ChainMapping mapping;
  int waves;   // CHAINS_BOTH: one-lane waves per SIMD
};
inline ChainChoice chain_choice(int L, int64_t chains, int64_t sweeps, int simds, bool beside) {
  const int both = beside ? both_waves(L, chains, sweeps, simds) : 0;
  if (both > 0) return {CHAINS_BOTH, both};
  if (lone_pays(L, chains, sweeps, simds)) return {CHAINS_LONE, 0};
  if (split_pays(L, chains, sweeps, simds)) return {CHAINS_SPLIT, 0};
  return {CHAINS_ONE_LANE, 0};
}

}  // namespace mcmc
