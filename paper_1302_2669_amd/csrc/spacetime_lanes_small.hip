// Space-time chains with one lane per interval, L = 2 .. 9 (spacetime_lanes.h).
#include "host_common.h"
#include "spacetime_choice.h"
#include "spacetime_lanes.h"

namespace mcmc {

hipError_t launch_spacetime_lanes_small(const SpaceTimeArgs& a, hipStream_t s) {
  return dispatch_lanes<2, ST_LANES_SMALL_L_MAX>(a, s);
}

bool spacetime_lanes_take(const SpaceTimeArgs& a) {
  if (a.L > ST_LANES_L_MAX || a.T > ST_LANES_T_MAX) return false;
  if (a.sp_thr[0] == 0xFFFFFFFFu) return false;
  for (int e = 0; e < 25; ++e)
    if (!((a.t_always >> e) & 1u) && a.t_thr[e] == 0xFFFFFFFFu) return false;
  // above, the other kernel streams the hypothesis through memory: never faster
  return a.L > SPACETIME_FAST_L_MAX ||
         spacetime_lanes_pay(a.L, a.T, a.n_tasks, a.sweep_end, 4 * device_cus());
}

}  // namespace mcmc

// The choice for `chains` chains on `simds` SIMDs (thresholds aside): 1 one lane per
// interval, 0 one lane per chain.
extern "C" int mcmc_spacetime_mapping(int32_t L, int32_t T, int64_t chains, int64_t sweeps,
                                      int32_t simds) {
  if (L > mcmc::ST_LANES_L_MAX || T > mcmc::ST_LANES_T_MAX) return 0;
  return L > mcmc::SPACETIME_FAST_L_MAX || mcmc::spacetime_lanes_pay(L, T, chains, sweeps, simds);
}
