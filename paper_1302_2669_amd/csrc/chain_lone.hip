// Chains of a few syndromes: one chain per wave (chain_split.h with all 64
// lanes drawing for it).
//
// A batch of at most about one wave per SIMD is bound by the length of a
// sweep's instruction sequence, most of it draws; with 64 lanes drawing, each
// takes 2 blocks a sweep at L = 13 instead of 6.
#include "chain_split.h"

namespace mcmc {

namespace {

template <int LMIN, int LMAX, int NOISE>
__device__ __forceinline__ void dispatch_lone(const RunArgs& a, int64_t t, uint32_t* lds) {
  if constexpr (LMIN <= LMAX) {
    if (a.g0.L == LMIN) run_split<LMIN, NOISE, 64>(a, a.g0, t, lds);
    else dispatch_lone<LMIN + 1, LMAX, NOISE>(a, t, lds);
  }
}

template <int LMIN, int LMAX, int NOISE>
__global__ void __launch_bounds__(64) chains_lone_kernel(const RunArgs a) {
  __shared__ __align__(16) uint32_t lds[split_words<LMIN, LMAX, 64>()];
  dispatch_lone<LMIN, LMAX, NOISE>(a, blockIdx.x, lds);
}

}  // namespace

hipError_t launch_chains_lone(const RunArgs& a, hipStream_t s) {
  const int L = a.g0.L;
  if (a.g0.n_tasks == 0) return hipSuccess;
  if (a.trace || a.tiles || a.tile_cum || L < LONE_L_MIN || L > MCMC_L_MAX ||
      a.g0.n_tasks > 0x7FFFFFFF)
    return hipErrorInvalidValue;
  const dim3 grid((unsigned)a.g0.n_tasks), block(64);
  if (a.noise == MCMC_NOISE_BITPHASE)
    hipLaunchKernelGGL((chains_lone_kernel<LONE_L_MIN, MCMC_L_MAX, 1>), grid, block, 0, s, a);
  else if (a.noise == MCMC_NOISE_DEPOLARIZING)
    hipLaunchKernelGGL((chains_lone_kernel<LONE_L_MIN, MCMC_L_MAX, 0>), grid, block, 0, s, a);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace mcmc
