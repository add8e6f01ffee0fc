// Space-time chains with one lane per interval, L = 2 .. 9 (spacetime_lanes.h).
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
  return true;
}

}  // namespace mcmc
