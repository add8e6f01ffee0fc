// Chains split over lanes (chain_split.h), independent bit/phase flips.
#include "chain_split.h"

namespace mcmc {

__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(SPLIT_WAVES)))
chains_split_flip_kernel(const RunArgs a) {
  split_persistent<2, 16, 1>(a);
}

__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(SPLIT_WAVES)))
chains_split_flip_wide_kernel(const RunArgs a) {
  split_persistent<17, 25, 1>(a);
}

hipError_t launch_chains_split_flip(const RunArgs& a, bool wide, int waves, hipStream_t s) {
  if (wide)
    hipLaunchKernelGGL(chains_split_flip_wide_kernel, dim3((unsigned)waves), dim3(64), 0, s, a);
  else
    hipLaunchKernelGGL(chains_split_flip_kernel, dim3((unsigned)waves), dim3(64), 0, s, a);
  return hipGetLastError();
}

}  // namespace mcmc
