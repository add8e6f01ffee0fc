// Space-time chains with one lane per interval, L = 10 .. 12 (spacetime_lanes.h).
#include "spacetime_lanes.h"

namespace mcmc {

hipError_t launch_spacetime_lanes_large(const SpaceTimeArgs& a, hipStream_t s) {
  return dispatch_lanes<ST_LANES_SMALL_L_MAX + 1, ST_LANES_LARGE_L_MAX>(a, s);
}

}  // namespace mcmc
