// Space-time chains with one lane per interval, L = 13 .. 15 (spacetime_lanes.h).
#include "spacetime_lanes.h"

namespace mcmc {

hipError_t launch_spacetime_lanes_largest(const SpaceTimeArgs& a, hipStream_t s) {
  return dispatch_lanes<ST_LANES_LARGE_L_MAX + 1, ST_LANES_L_MAX>(a, s);
}

}  // namespace mcmc
