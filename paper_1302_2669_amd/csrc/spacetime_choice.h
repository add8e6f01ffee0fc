// Choice between the space-time kernels of the smaller codes: one lane per
// interval (spacetime_lanes.h) or one lane per chain (spacetime.hip).
//
// The unit is SIMD cycles per run.  One lane per interval splits a chain's moves
// over T lanes, but its time half takes n_q + 2 (T - 2) steps for n_q qubits and
// 64 mod T lanes idle: batches too small to fill the chip with one chain per lane
// gain up to ten times, full batches of small codes lose with T (65536 histories x
// 4 chains: L = 3, 16 rounds 9.9 ms against 5.2, 4 rounds 5.2 against 4.8; L = 7, 8
// rounds 3.9 against 4.2).
#pragma once

#include <math.h>
#include <stdint.h>

namespace mcmc {

// One lane per chain: a move of a wave takes 360 cycles alone on its SIMD (up to
// 520 with every SIMD taken at L = 12) and 148 to 190 among 16; longer rows cost
// more words a move.  Measured and estimated us per sweep, L = 5, 12 rounds, 4
// chains: 1024 histories 212 / 219, 16384 429 / 407, 65536 1479 / 1404.
inline double spacetime_chain_cycles(int L, int T, double chains, double sweeps, int simds) {
  const double moves = T * 2.0 * L * (L - 1) + (T - 1) * 2.0 * (2 * L * L - 2 * L + 1);
  const double w = chains / (64.0 * simds);
  const double among = (138.0 + 0.25 * L * L) * (w < 8.0 ? ceil(w) : w) + 130.0;
  return moves * fmax(360.0 + 0.8 * L * L, among) * (sweeps + 0.1);
}

// One lane per interval: a Philox block 160 cycles, a time step (two moves) 140,
// a spatial move 66 of a wave among others, which come whole to a SIMD; a lone
// wave waits about as long again.  The same three: 34 / 34, 388 / 387, 1655 / 1533.
inline double spacetime_lanes_cycles(int L, int T, double chains, double sweeps, int simds) {
  const double stab = 2.0 * L * (L - 1), steps = T > 1 ? 2 * L * L - 2 * L + 1 + 2.0 * (T - 2) : 0;
  const double sweep = 160.0 * (stab / 4 + steps / 2) + 140.0 * steps + 66.0 * stab + 250.0;
  const double w = chains / ((double)(64 / T) * simds);
  return sweep * fmax(1.85, (w < 8.0 ? ceil(w) : w) + 0.6) * (sweeps + 0.35);
}

// Whether one lane per interval is taken; the other has to win a tenth, the
// estimates' error (332 batches of L = 2 to 12, 1 to 16 rounds, 1 to 64 waves per
// SIMD: it then loses 5% at one, the rule forgoes up to 10% of runs of 5 sweeps
// and more).
inline bool spacetime_lanes_pay(int L, int T, int64_t chains, int64_t sweeps, int simds) {
  return spacetime_chain_cycles(L, T, (double)chains, (double)sweeps, simds) >=
         0.9 * spacetime_lanes_cycles(L, T, (double)chains, (double)sweeps, simds);
}

}  // namespace mcmc
