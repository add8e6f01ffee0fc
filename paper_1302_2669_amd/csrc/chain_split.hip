// Chains split over lanes (chain_split.h), depolarizing noise.
#include "chain_split.h"

namespace mcmc {

__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(SPLIT_WAVES)))
chains_split_kernel(const RunArgs a) {
  split_persistent<2, 16, 0>(a);
}

__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(SPLIT_WAVES)))
chains_split_wide_kernel(const RunArgs a) {
  split_persistent<17, 25, 0>(a);
}

hipError_t launch_chains_split(const RunArgs& a, bool wide, int waves, hipStream_t s) {
  if (a.n_tiles == 0) return hipSuccess;
  if (a.trace || waves < 1) return hipErrorInvalidValue;
  if (a.noise == MCMC_NOISE_BITPHASE) return launch_chains_split_flip(a, wide, waves, s);
  if (a.noise != MCMC_NOISE_DEPOLARIZING) return hipErrorInvalidValue;
  if (wide)
    hipLaunchKernelGGL(chains_split_wide_kernel, dim3((unsigned)waves), dim3(64), 0, s, a);
  else
    hipLaunchKernelGGL(chains_split_kernel, dim3((unsigned)waves), dim3(64), 0, s, a);
  return hipGetLastError();
}

}  // namespace mcmc
