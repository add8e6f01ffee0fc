// Colour-phased Metropolis chains, two chains per lane, for codes up to L = 8
// (Sec. IV, Sec. IV.A, Sec. V of arXiv:1302.2669): the second chain mapping
// a plan can choose for its small codes (mcmc_tuning.pair_small).
//
// A row of a code with L <= 8 fills at most half a 32-bit word, so one lane
// keeps two chains in the same registers: chain A in fields 0..7 and chain B
// in fields 8..15 of every row word.  The SWAR arithmetic of the one-chain
// kernel (chain_body.h) then evaluates a grid row of same-coloured sites of
// both chains at once: their sites land in nibbles 0..3 (A) and 4..7 (B) of
// the neighbour sums.  The only place where the halves would meet is the
// west neighbour of a star in field 0 or 8, which reads the padding value
// instead; every flip mask stays inside its half because rows end at field
// L - 1 <= 7.  Each chain keeps its own draws (Philox counter of its own
// syndrome, class, temperature and replica, the blocks of both chains
// computed together), its own acceptance thresholds (two LDS columns per
// lane) and its own weight, sums and accept count, so every output is the
// one-chain kernel's bit for bit.
//
// Tasks: a pair tile of a group covers tasks first .. first + 127; lane l
// runs tasks first + l (A) and first + 64 + l (B).  A lane whose B task is
// past the group's end runs B as a copy of A and writes nothing for it.
// Plans only: no trace, no resume, no exported state.
#include "chain_body.h"

namespace mcmc {

namespace {

constexpr uint32_t HALF_LO = 0x0000FFFFu;

// fields 0..n-1 of both halves
__host__ __device__ constexpr uint32_t pair_fields(int n) {
  return field_mask(n, 0) | (field_mask(n, 0) << 16);
}
// nibble-top mask of the sites of one row in both halves
__host__ __device__ constexpr uint32_t pair_sites(int par, int limit) {
  return site_tops(par, limit, 0) | (site_tops(par, limit, 0) << 16);
}

// Blocks BLK of two chains' streams together (both keyed by the same seed).
template <int BLK>
__device__ __forceinline__ void block_two(const ChainRng& A, const ChainRng& B, uint4& a,
                                          uint4& b) {
  a = A.template after_two<BLK>();
  b = B.template after_two<BLK>();
  philox_rounds2(a, b, A.k0, A.k1, 2);
}

struct PairChain {
  ItemDesc it;
  int64_t out;
  int cls, kt, chain;
};

__device__ __forceinline__ PairChain pair_chain(const RunArgs& a, const GroupDesc& g, int64_t t) {
  PairChain c;
  const int64_t per_item = 4 * (int64_t)g.K * g.C;
  const int64_t item_local = t / per_item;
  const int rem = (int)(t - item_local * per_item);
  c.chain = rem % g.C;
  c.kt = (rem / g.C) % g.K;
  c.cls = rem / (g.C * g.K);
  c.it = a.items[g.first_item + item_local];
  c.out = c.it.chain_off + rem;
  return c;
}

template <int L, int NOISE>
__device__ __forceinline__ void run_pair(const RunArgs& a, const GroupDesc& g, int64_t tA,
                                         bool has_b, uint32_t (*lds_tbl)[512], const int col) {
  using G = Geo<L>;
  constexpr int R = G::R, S = G::S;
  static_assert(L <= PAIR_L_MAX && PAIR_L_MAX <= 8, "two chains per word need rows of at most 8 fields");
  const PairChain A = pair_chain(a, g, tA);
  const PairChain B = has_b ? pair_chain(a, g, tA + 64) : A;

#pragma unroll
  for (int e = 0; e < 9; ++e) {
    uint32_t va = 0xFFFFFFFFu, vb = 0xFFFFFFFFu;
    if (e > 4) {
      va = a.tables[A.it.table_off + A.kt * 4 + (e - 5)];
      vb = a.tables[B.it.table_off + B.kt * 4 + (e - 5)];
    }
    lds_tbl[e][col] = va;
    lds_tbl[e][256 + col] = vb;
  }

  uint32_t st[R];
#pragma unroll
  for (int r = 0; r < R; ++r)
    st[r] = reg_code((a.init_rows[A.it.rows_off + r * 4 + A.cls] & HALF_LO) |
                     (a.init_rows[B.it.rows_off + r * 4 + B.cls] << 16));
  int32_t nA = a.init_n[A.it.orig * 4 + A.cls];
  int32_t nB = a.init_n[B.it.orig * 4 + B.cls];
  int64_t SA = 0, SB = 0, AA = 0, AB = 0;

  ChainRng rA, rB;
  rA.init(a.k0, a.k1, A.it.sid, ((uint32_t)A.cls << 28) | ((uint32_t)(A.kt + 1) << 20) |
                                    (uint32_t)A.chain);
  rB.init(a.k0, a.k1, B.it.sid, ((uint32_t)B.cls << 28) | ((uint32_t)(B.kt + 1) << 20) |
                                    (uint32_t)B.chain);

  // the top bit of every nibble, as in the one-chain kernel
  uint32_t site_bit[8];
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    site_bit[m] = 8u << (4 * m);
    asm volatile("" : "+v"(site_bit[m]));
  }

  for (int sweep = g.sweep_begin; sweep < g.sweep_end; ++sweep) {
    rA.begin_sweep((uint32_t)sweep);
    rB.begin_sweep((uint32_t)sweep);
    uint4 bA = make_uint4(0, 0, 0, 0), bB = make_uint4(0, 0, 0, 0);
    uint32_t dA = 0, dB = 0;  // 8 x the sum of Delta n + 4 over the phase's accepted moves
    int32_t cA = 0, cB = 0;   // accepted moves of the sweep
    int32_t pA = 0, pB = 0;   // of them, before the current phase

    // as in the one-chain kernel: no computation of a later row is hoisted
    // above the end of the current one
    auto fence = [&]() {
#pragma unroll
      for (int r = 0; r < R; ++r) asm volatile("" : "+v"(st[r]));
      asm volatile("" : "+v"(dA), "+v"(dB), "+v"(cA), "+v"(cB));
    };
    auto end_phase = [&]() {
      nA += (int32_t)(dA >> 3) - 4 * (cA - pA);
      nB += (int32_t)(dB >> 3) - 4 * (cB - pB);
      dA = dB = 0;
      pA = cA;
      pB = cB;
      if (sweep >= g.burn) {
        SA += nA;
        SB += nB;
      }
    };

    // Accept decisions of one row of both chains (nibble m of `sum`: site m
    // of A, nibble 4 + m: site m of B); returns the accepted sites as the top
    // bits of their nibbles.
    auto decide_row = [&](auto PAR, auto NSITE, auto D0, auto LIMIT, uint32_t sum) -> uint32_t {
      constexpr int par = decltype(PAR)::value, nsite = decltype(NSITE)::value;
      constexpr int d0 = decltype(D0)::value, limit = decltype(LIMIT)::value;
      uint32_t rej = 0;
      static_for<nsite>([&](auto MM) {
        constexpr int m = decltype(MM)::value;
        constexpr int d = d0 + m;
        if constexpr ((d & 3) == 0) block_two<d / 4>(rA, rB, bA, bB);
        const uint32_t ta = lds_tbl[(sum >> (4 * m)) & 15u][col];
        const uint32_t tb = lds_tbl[(sum >> (16 + 4 * m)) & 15u][256 + col];
        const uint32_t ra = reject_bit(word_of(bA, d & 3), ta, site_bit[m]);
        const uint32_t rb = reject_bit(word_of(bB, d & 3), tb, site_bit[4 + m]);
        if constexpr (m == 0) rej = ra | rb;
        else rej = rej | ra | rb;
      });
      constexpr uint32_t sites = pair_sites(par, limit);
      const uint32_t acc = bitop3<0x2A>(sum + 0x33333333u, rej, sites);   // ~(a & b) & c
      const uint32_t aA = acc & HALF_LO, aB = acc & ~HALF_LO;
      dA = __builtin_amdgcn_udot8(sum, aA, dA, false);
      dB = __builtin_amdgcn_udot8(sum, aB, dB, false);
      cA += (int32_t)__builtin_popcount(aA);
      cB += (int32_t)__builtin_popcount(aB);
      return acc;
    };

    // ---------------- stars: colours 0 and 1 ----------------
    static_for<2>([&](auto PH) {
      constexpr int phi = decltype(PH)::value;
      uint32_t cN = c_star_of<NOISE>(st[0]);   // carried from row to row, as in the one-chain kernel
      static_for<L - 1>([&](auto I) {
        constexpr int i = decltype(I)::value;
        constexpr int par = (i + phi) & 1;
        constexpr int nsite = (L - par + 1) / 2;
        constexpr int rank0 = star_row_rank<L>(i, phi);
        uint32_t cO = c_star_of<NOISE>(st[2 * i + 1]);
        if constexpr (NOISE == 1) cO |= 0x55555555u & ~pair_fields(L - 1);   // pad: c = 1
        const uint32_t cS = c_star_of<NOISE>(st[2 * i + 2]);
        // west neighbours; fields 0 and 8 read the padding value 1
        const uint32_t cWest = ((cO << 2) & ~0x00030003u) | 0x00010001u;
        constexpr uint32_t M = 0x33333333u;
        const uint32_t sum = ((cN >> (2 * par)) & M) + ((cS >> (2 * par)) & M) +
                             ((cO >> (2 * par)) & M) + ((cWest >> (2 * par)) & M);
        cN = cS;
        const uint32_t acc = decide_row(std::integral_constant<int, par>{},
                                        std::integral_constant<int, nsite>{},
                                        std::integral_constant<int, phi * S + rank0>{},
                                        std::integral_constant<int, L>{}, sum);
        const uint32_t ax = shift_by<2 * par - 2>(acc);
        st[2 * i] ^= ax;
        st[2 * i + 2] ^= ax;
        st[2 * i + 1] ^= (ax | (ax >> 2)) & pair_fields(L - 1) & 0xAAAAAAAAu;
        fence();
      });
      end_phase();
    });

    // ---------------- plaquettes: colours 2 and 3 ----------------
    static_for<2>([&](auto PH) {
      constexpr int phi = 2 + decltype(PH)::value;
      uint32_t cN = 0x55555555u;
      static_for<L>([&](auto I) {
        constexpr int i = decltype(I)::value;
        constexpr int par = (i + phi - 2) & 1;
        constexpr int nsite = (L - par) / 2;
        constexpr int rank0 = plaq_row_rank<L>(i, phi - 2);
        if constexpr (nsite > 0) {
          const uint32_t cE = c_plaq_of<NOISE>(st[2 * i]);
          uint32_t cS = 0x55555555u;
          if constexpr (i < L - 1) cS = c_plaq_of<NOISE>(st[2 * i + 1]);
          const uint32_t cEast = cE >> 2;   // a site's east field stays in its half
          constexpr uint32_t M = 0x33333333u;
          const uint32_t sum = ((cN >> (2 * par)) & M) + ((cS >> (2 * par)) & M) +
                               ((cE >> (2 * par)) & M) + ((cEast >> (2 * par)) & M);
          cN = cS;
          const uint32_t acc = decide_row(std::integral_constant<int, par>{},
                                          std::integral_constant<int, nsite>{},
                                          std::integral_constant<int, phi * S + rank0>{},
                                          std::integral_constant<int, L - 1>{}, sum);
          const uint32_t az = shift_by<2 * par - 3>(acc);
          if constexpr (i > 0) st[2 * i - 1] ^= az;
          if constexpr (i < L - 1) st[2 * i + 1] ^= az;
          st[2 * i] ^= az | (az << 2);
          fence();
        } else if constexpr (i < L - 1) {   // L = 2: a row without sites of this colour
          cN = c_plaq_of<NOISE>(st[2 * i + 1]);
        }
      });
      end_phase();
    });
    AA += cA;
    AB += cB;
  }

  a.S_out[A.out] = SA;
  a.A_out[A.out] = AA;
  a.n_out[A.out] = nA;
  if (has_b) {
    a.S_out[B.out] = SB;
    a.A_out[B.out] = AB;
    a.n_out[B.out] = nB;
  }
  // final rows: fields past each row's end hold Y in the stored layout
  if (a.final_rows && A.chain == 0 && A.kt == g.K - 1) {
#pragma unroll
    for (int r = 0; r < R; ++r)
      a.final_rows[A.it.rows_off + r * 4 + A.cls] = (row_code(st[r]) & HALF_LO) | ~HALF_LO;
  }
  if (a.final_rows && has_b && B.chain == 0 && B.kt == g.K - 1) {
#pragma unroll
    for (int r = 0; r < R; ++r)
      a.final_rows[B.it.rows_off + r * 4 + B.cls] = (row_code(st[r]) >> 16) | ~HALF_LO;
  }
}

template <int LMIN, int NOISE>
__device__ __forceinline__ void dispatch_pair(const RunArgs& a, const GroupDesc& g, int L,
                                              int64_t t, bool has_b, uint32_t (*lds)[512],
                                              int col) {
  if constexpr (LMIN <= PAIR_L_MAX) {
    if (L == LMIN) {
      run_pair<LMIN, NOISE>(a, g, t, has_b, lds, col);
      return;
    }
    dispatch_pair<LMIN + 1, NOISE>(a, g, L, t, has_b, lds, col);
  }
}

template <int NOISE>
__device__ __forceinline__ void pair_persistent(const RunArgs& a) {
  __shared__ uint32_t lds_tbl[9][512];
  const int col = threadIdx.x;
  const int lane = threadIdx.x & 63;
  while (true) {
    uint32_t tile = 0;
    if (lane == 0) tile = atomicAdd(a.queue, 1u);
    tile = __builtin_amdgcn_readfirstlane(tile);  // lane 0 is active: the loop is wave-uniform
    if ((int64_t)tile >= a.n_tiles) break;
    const TileDesc td = a.tiles[tile];
    const GroupDesc g = a.groups[td.group];
    if (td.L < 2 || td.L > PAIR_L_MAX) continue;
    const int64_t t = td.first_task + lane;
    if (t < g.n_tasks) dispatch_pair<2, NOISE>(a, g, td.L, t, t + 64 < g.n_tasks, lds_tbl, col);
  }
}

__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(PAIR_WAVES)))
chains_pair_kernel(const RunArgs a) {
  pair_persistent<0>(a);
}

__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(PAIR_WAVES)))
chains_pair_flip_kernel(const RunArgs a) {
  pair_persistent<1>(a);
}

}  // namespace

hipError_t launch_chains_pair(const RunArgs& a, int waves, int wg, hipStream_t s) {
  if (a.n_tiles == 0) return hipSuccess;
  if (wg != 64 && wg != 128 && wg != 256) return hipErrorInvalidValue;
  if (!a.items || !a.tiles || !a.tables || a.trace || a.resume_rows || a.state_rows)
    return hipErrorInvalidValue;
  const int per_wg = wg / 64;
  const int blocks = (waves + per_wg - 1) / per_wg;
  if (a.noise == MCMC_NOISE_BITPHASE)
    hipLaunchKernelGGL(chains_pair_flip_kernel, dim3((unsigned)blocks), dim3((unsigned)wg), 0, s,
                       a);
  else if (a.noise == MCMC_NOISE_DEPOLARIZING)
    hipLaunchKernelGGL(chains_pair_kernel, dim3((unsigned)blocks), dim3((unsigned)wg), 0, s, a);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace mcmc
