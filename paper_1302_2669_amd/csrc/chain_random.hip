// Random-scan chains (Sec. IV as written): every Metropolis step picks one
// stabilizer uniformly at random among all n_stab, computes its change of
// energy and applies it with the Metropolis probability; n is summed after
// every step.  A sweep is n_stab steps.  This is the paper's own chain, kept
// beside the colour-phased kernels as a statistical cross-check of their scan
// order; it is not the throughput path.
//
// Mapping.  One lane per chain as in the colour-phased kernels, but a random
// site needs its rows by a runtime index, so each lane's configuration lives
// in LDS, one word (L <= 15) or one 64-bit word per grid row, row-major with
// the lanes side by side (no bank conflicts).  A site touches one
// qubit of the row above, two neighbouring ones of its own row and one of the
// row below: three reads at one address with fixed offsets.  To make that hold
// at the boundaries there is a padding row above and below, and odd rows are
// stored one field up, so that field j and j + 1 of its own row are the site's
// neighbours for stars and plaquettes alike.  Padding is Y: a star's move does
// not change its weight whatever the x part, nor a plaquette's whatever the z
// part, and no other move reaches that padding, so it may be flipped along.
//
// What bounds it.  A step is a serial chain (read, weight change, write), and
// everything before it, the draws, the site's table entry and the number of
// acceptance thresholds the draw reaches, depends on no state.  So a lane
// takes its steps in batches of four: while the reads of a step are in
// flight it works on the draws of the next batch, half a Philox block and the
// entry of the slot freed by the step before.
// A lone wave issues an instruction in about 4.7 cycles whatever it waits for,
// so the count of them is the time: 90 a step with the batch copied and 77 now.
// 4096 syndromes x 16 chains x 169 sweeps at L = 13, one wave per SIMD: 25.8 ->
// 8.0 ms, 1175 -> 362 cycles per step.
//
// Randomness: step t of a sweep uses block t >> 1 of Philox4x32-10 at counter
// (t >> 1, sweep, syndrome_id, 2<<30 | cls<<28 | temp<<20 | chain): word
// 2(t&1) picks the site, floor(u n_stab / 2^32), word 2(t&1)+1 decides.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "device_common.h"
#include "host_common.h"
#include "internal.h"

namespace mcmc {
namespace {

// Four waves share a site table, their lanes side by side in the rows: a wave on
// every SIMD of a compute unit.  Smaller workgroups are not spread evenly over the
// SIMDs: with one wave each the first launch above took 11.6 ms and the others
// 8.06, with two each all of them 11.6; 40000 x 16 chains x 10 sweeps 4.08 ms with
// one, 2.93 with four.  Where four waves' rows leave a compute unit fewer waves
// than single ones do (L = 19 to 22), full batches take those, and so do batches
// of at most one wave per compute unit, whose LDS each then has to itself (16000
// chains at L = 17: 1.99 ms, 2.05 with four).
constexpr int RS_WAVES = 4;
// steps per batch: two Philox blocks; n_stab = 2 L (L - 1) is a multiple of 4
constexpr int RS_BATCH = 4;
// codes with one 32-bit word per row, the field past an odd row's end included
constexpr int RS_NARROW_L_MAX = 15;

template <bool WIDE>
struct RowWord {
  using type = uint32_t;
};
template <>
struct RowWord<true> {
  using type = uint64_t;
};

// Table entry of a site (center row r, first field j of the row's pair):
//   x: bits 0-5 shift of the pair (2 j), then the row's offset in LDS (the row
//      above: r times the workgroup's lanes and 4 or 8 bytes, up to bit 15 narrow
//      or 16 wide), from bit 16 or 17 on the shift of the fields above and below;
//   y: bits 0-5 and 8-13 the same shifts plus the flipped part's bit t (0:
//      x, star; 1: z, plaquette), 16-20 2 - 2t, 24-31 the flipped part's bits
//      of the four gathered codes (missing neighbours left out under
//      bit/phase flips, where their padding would count).
template <int NOISE, bool WIDE, int LANES>
__device__ uint2 site_entry(int L, int s) {
  const int nstar = L * (L - 1);
  const bool star = s < nstar;
  const int k = star ? s : s - nstar, w = star ? L : L - 1;
  const int i = k / w, j = k % w, t = star ? 0 : 1;
  const int r = star ? 2 * i + 1 : 2 * i;
  // odd rows are stored one field up: a plaquette's neighbours above and below
  const int pair = 2 * j, single = star ? 2 * j : 2 * j + 2;
  uint32_t own = star ? 0x55u : 0xAAu;
  if (NOISE == 1) {   // gathered: above, below, first and second of the pair
    if (star && j == 0) own &= ~0x30u;
    if (star && j == L - 1) own &= ~0xC0u;
    if (!star && i == 0) own &= ~0x03u;
    if (!star && i == L - 1) own &= ~0x0Cu;
  }
  uint2 e;
  e.x = (uint32_t)pair | ((uint32_t)(r * LANES * (WIDE ? 8 : 4))) |
        ((uint32_t)single << (WIDE ? 17 : 16));
  e.y = (uint32_t)(pair + t) | ((uint32_t)(single + t) << 8) | ((uint32_t)(2 - 2 * t) << 16) |
        (own << 24);
  return e;
}

// philox_round with the compiler's own three-input operation: behind one in
// inline asm it leaves a wait state, which a lone wave feels (8.70 and 8.60 ms
// on the launch above).
__device__ __forceinline__ uint4 keyed_round(uint4 c, uint32_t k0, uint32_t k1) {
  uint32_t h0, l0, h1, l1;
  mulhilo(PHILOX_M0, c.x, h0, l0);
  mulhilo(PHILOX_M1, c.z, h1, l1);
  return make_uint4(bitop3<0x96>(h1, c.y, k0), l1, bitop3<0x96>(h0, c.w, k1), l0);
}

// How many of the four thresholds u stays below.  A mask (VCC or an SGPR pair) is
// read from the third instruction after the one that writes it, at the earliest:
// the other compares and adds fill that gap (the decode with the launch above 8.23
// ms; with wait states 9.18, as the compiler orders it 8.91).
__device__ __forceinline__ int32_t count_below(uint32_t u, const uint32_t thr[4]) {
  int32_t q;
  uint64_t m0, m1;
  asm("v_cmp_lt_u32 vcc, %3, %4\n\tv_cmp_lt_u32 %1, %3, %5\n\t"
      "v_cmp_lt_u32 %2, %3, %6\n\tv_cndmask_b32 %0, 0, 1, vcc\n\t"
      "v_cmp_lt_u32 vcc, %3, %7\n\tv_addc_co_u32 %0, %1, 0, %0, %1\n\t"
      "v_addc_co_u32 %0, %2, 0, %0, %2\n\tv_addc_co_u32 %0, vcc, 0, %0, vcc"
      : "=&v"(q), "=&s"(m0), "=&s"(m1)
      : "v"(u), "v"(thr[0]), "v"(thr[1]), "v"(thr[2]), "v"(thr[3])
      : "vcc");
  return q;
}

// One step ahead of its turn: its site's entry and how many of the four
// thresholds its draw stays below (Delta n is accepted iff it is at most that).
struct Step {
  uint2 site;
  int32_t q;
};

template <int NOISE, bool WIDE, int WAVES>
__global__ void __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(4)))
chains_random_kernel(const RunArgs a) {
  using Row = typename RowWord<WIDE>::type;
  constexpr int RS_LANES = 64 * WAVES;
  constexpr uint32_t kSingle = WIDE ? 17 : 16;
  constexpr uint32_t kRowMask =
      ((1u << kSingle) - 1u) & ~(uint32_t)(RS_LANES * sizeof(Row) - 1);
  extern __shared__ __align__(16) uint32_t rs_lds[];
  const GroupDesc g = a.g0;
  const int L = g.L;
  const int W = words_per_row(L);
  const int R = 2 * L - 1;
  const int RW = R * W;
  const int nstab = 2 * L * (L - 1);
  const int lane = threadIdx.x;
  Row* rows = reinterpret_cast<Row*>(rs_lds);   // [R + 2][RS_LANES], aligned as a row offset
  uint2* sites = reinterpret_cast<uint2*>(rows + (R + 2) * RS_LANES);
  for (int s = lane; s < nstab; s += RS_LANES) sites[s] = site_entry<NOISE, WIDE, RS_LANES>(L, s);
  __syncthreads();

  const int64_t t = (int64_t)blockIdx.x * RS_LANES + lane;
  if (t >= g.n_tasks) return;
  const int K = g.K, C = g.C;
  const int64_t per_item = 4 * (int64_t)K * C;
  const int64_t item = t / per_item;
  const int rem = (int)(t - item * per_item);
  const int chain = rem % C;
  const int kt = (rem / C) % K;
  const int cls = rem / (C * K);
  const int64_t out = item * per_item + rem;
  const int64_t rows_off = item * RW * 4;
  const uint32_t sid = a.syndrome_ids ? a.syndrome_ids[item] : (uint32_t)item;
  uint32_t thr[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) thr[k] = a.table0[kt][k];

  rows[lane] = ~(Row)0;
  rows[(R + 1) * RS_LANES + lane] = ~(Row)0;
  for (int r = 0; r < R; ++r) {
    Row v = ~(Row)0;
    for (int w = W - 1; w >= 0; --w) {
      const int k = r * W + w;
      const uint32_t word = a.resume_rows ? a.resume_rows[(int64_t)k * a.total_chains + out]
                                          : a.init_rows[rows_off + k * 4 + cls];
      if constexpr (WIDE) v = w == 1 ? ((Row)word << 32) | 0xFFFFFFFFu : (v & ~(Row)0xFFFFFFFFu) | word;
      else v = word;
    }
    rows[(r + 1) * RS_LANES + lane] = (r & 1) ? (v << 2) | 3u : v;
  }
  int32_t n = a.resume_rows ? a.resume_n[out] : a.init_n[item * 4 + cls];
  int64_t Ssum = a.resume_rows ? a.resume_S[out] : 0;
  int64_t Acnt = a.resume_rows ? a.resume_A[out] : 0;

  ChainRng rng;
  rng.init(a.k0, a.k1, sid, (2u << 30) | ((uint32_t)cls << 28) | ((uint32_t)(kt + 1) << 20) |
                                (uint32_t)chain);
  // the first five rounds of block b of the sweep begun last (b the same in
  // every lane), and the others
  auto block = [&](uint32_t b) -> uint4 {
    uint32_t hi0, lo0, qh, ql;
    mulhilo(PHILOX_M0, b, hi0, lo0);
    mulhilo(PHILOX_M1, hi0 ^ rng.ctr3, qh, ql);
    uint4 v = make_uint4(qh ^ rng.sid_x, ql, rng.sw_x ^ lo0, rng.sw_lo);
#pragma unroll
    for (uint32_t r = 2; r < 5; ++r) v = keyed_round(v, a.k0 + r * PHILOX_W0, a.k1 + r * PHILOX_W1);
    return v;
  };
  auto finish = [&](uint4 v) -> uint4 {
#pragma unroll
    for (uint32_t r = 5; r < 10; ++r) v = keyed_round(v, a.k0 + r * PHILOX_W0, a.k1 + r * PHILOX_W1);
    return v;
  };
  auto step_of = [&](uint32_t u_site, uint32_t u_acc) -> Step {
    Step s;
    s.site = sites[__umulhi(u_site, (uint32_t)nstab)];
    s.q = count_below(u_acc, thr);
    return s;
  };

  // this lane's column; the kernel's only shared memory begins at LDS address 0
  typedef Row __attribute__((address_space(3))) * LdsRow;
  const uint32_t column = (uint32_t)(uintptr_t)(LdsRow)(rows + lane);
  constexpr uint32_t kShift = WIDE ? 63u : 31u;
  // the steps to come: slot k holds the next step at position k of a batch; va
  // and vb are the blocks of slots 0, 1 and 2, 3
  Step slot[RS_BATCH];
  uint4 va = make_uint4(0, 0, 0, 0), vb = va;
  if (g.sweep_begin < g.sweep_end) {
    rng.begin_sweep((uint32_t)g.sweep_begin);
    va = finish(block(0u));
    vb = finish(block(1u));
    slot[0] = step_of(va.x, va.y);
    slot[1] = step_of(va.z, va.w);
    slot[2] = step_of(vb.x, vb.y);
  }
  for (int sweep = g.sweep_begin; sweep < g.sweep_end; ++sweep) {
    int32_t moves = 0;
    int64_t sum = 0;
    for (int first = 0; first < nstab; first += RS_BATCH) {
      // the batch after this one: of this sweep or the first of the next
      uint32_t b = (uint32_t)(first + RS_BATCH) >> 1;
      if (first + RS_BATCH == nstab) {
        rng.begin_sweep((uint32_t)sweep + 1);
        b = 0;
      }
      int32_t batch_sum = 0;
#pragma unroll
      for (int k = 0; k < RS_BATCH; ++k) {
        const uint2 e = slot[k].site;
        const LdsRow p = (LdsRow)(uintptr_t)((e.x & kRowMask) | column);
        const Row up = p[0], mid = p[RS_LANES], down = p[2 * RS_LANES];
        __builtin_amdgcn_sched_barrier(0);
        // while they arrive: half a block, and the slot that is free again
        if (k == 0) {
          slot[3] = step_of(vb.z, vb.w);
          va = block(b);
        } else if (k == 1) {
          va = finish(va);
          slot[0] = step_of(va.x, va.y);
        } else if (k == 2) {
          slot[1] = step_of(va.z, va.w);
          vb = block(b + 1);
        } else {
          vb = finish(vb);
          slot[2] = step_of(vb.x, vb.y);
        }
        __builtin_amdgcn_sched_barrier(0);
        // the four codes: above, below, the pair
        uint32_t code;
        if constexpr (WIDE) {
          const uint32_t single = e.x >> kSingle;
          code = (((uint32_t)(mid >> (e.x & kShift)) & 15u) << 2) |
                 ((uint32_t)(down >> (single & kShift)) & 3u);
          code = (code << 2) | ((uint32_t)(up >> (single & kShift)) & 3u);
        } else {
          const uint32_t single = e.x >> kSingle;
          code = (__builtin_amdgcn_ubfe(mid, e.x, 4) << 2) | __builtin_amdgcn_ubfe(down, single, 2);
          code = (code << 2) | __builtin_amdgcn_ubfe(up, single, 2);
        }
        // Delta n = the qubits that the move makes wrong minus those that it
        // mends: the valid ones without and with the flipped part set, under
        // depolarizing noise only those without the other part
        const uint32_t own = e.y >> 24;
        uint32_t other = 0;
        if constexpr (NOISE == 0) other = (code << 1) >> ((e.y >> 16) & 31u);
        const int32_t delta = (int32_t)__builtin_popcount(bitop3<0x10>(own, code, other)) -
                              (int32_t)__builtin_popcount(bitop3<0x40>(own, code, other));
        if (delta <= slot[k].q) {
          const Row ms = (Row)1 << ((e.y >> 8) & 0xFFu), mp = (Row)5 << (e.y & kShift);
          p[0] = up ^ ms;
          p[RS_LANES] = mid ^ mp;
          p[2 * RS_LANES] = down ^ ms;
          n += delta;
          ++moves;
        }
        batch_sum += n;
      }
      sum += batch_sum;
    }
    if (sweep >= g.burn) Ssum += sum;
    Acnt += moves;
  }

  a.S_out[out] = Ssum;
  a.A_out[out] = Acnt;
  a.n_out[out] = n;
  for (int r = 0; r < R; ++r) {
    Row v = rows[(r + 1) * RS_LANES + lane];
    if (r & 1) v >>= 2;
    for (int w = 0; w < W; ++w) {
      const uint32_t word = (uint32_t)(v >> (32 * w)) | ~field_mask((r & 1) ? L - 1 : L, w);
      if (a.state_rows) a.state_rows[(int64_t)(r * W + w) * a.total_chains + out] = word;
      if (a.final_rows && chain == 0 && kt == K - 1)
        a.final_rows[rows_off + (r * W + w) * 4 + cls] = word;
    }
  }
}

size_t random_scan_lds_bytes(int L, int waves) {
  const size_t row = L <= RS_NARROW_L_MAX ? 4 : 8;
  return (size_t)(2 * L * (L - 1)) * sizeof(uint2) + (size_t)(2 * L + 1) * 64 * waves * row;
}

template <int NOISE, bool WIDE, int WAVES>
hipError_t launch_random(const RunArgs& a, hipStream_t s) {
  auto* fn = chains_random_kernel<NOISE, WIDE, WAVES>;
  const int64_t blocks = (a.g0.n_tasks + 64 * WAVES - 1) / (64 * WAVES);
  if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
  const size_t lds = random_scan_lds_bytes(a.g0.L, WAVES);
  if (lds > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(fn, dim3((unsigned)blocks), dim3(64 * WAVES), lds, s, a);
  return hipGetLastError();
}

template <int WAVES>
hipError_t launch_random_waves(const RunArgs& a, hipStream_t s) {
  const bool wide = a.g0.L > RS_NARROW_L_MAX;
  if (a.noise == MCMC_NOISE_BITPHASE)
    return wide ? launch_random<1, true, WAVES>(a, s) : launch_random<1, false, WAVES>(a, s);
  return wide ? launch_random<0, true, WAVES>(a, s) : launch_random<0, false, WAVES>(a, s);
}

}  // namespace

hipError_t launch_chains_random(const RunArgs& a, hipStream_t s) {
  if (a.g0.n_tasks == 0) return hipSuccess;
  // waves that a compute unit's LDS holds at once in workgroups of four or one
  const size_t lds = 160 * 1024;
  const int64_t fours = RS_WAVES * (int64_t)(lds / random_scan_lds_bytes(a.g0.L, RS_WAVES));
  const int64_t ones = (int64_t)(lds / random_scan_lds_bytes(a.g0.L, 1));
  const int64_t waves = (a.g0.n_tasks + 63) / 64, cus = device_cus();
  if (waves > cus && (fours >= std::min<int64_t>(ones, 16) || waves <= fours * cus))
    return launch_random_waves<RS_WAVES>(a, s);
  return launch_random_waves<1>(a, s);
}

}  // namespace mcmc
