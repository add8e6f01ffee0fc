// Space-time chains with one lane per interval (Sec. VI), codes up to
// ST_LANES_L_MAX and at most ST_LANES_T_MAX rounds.  Same moves, order
// and draws as the register-interval kernel of spacetime.hip, so the chains
// are bit-identical.
//
// Mapping.  A chain takes T neighbouring lanes, 64 / T chains a wave; lane t
// keeps interval t's data error and round t's wrong outcomes in registers for
// the whole run (the one-lane kernel moves the hypothesis through memory once
// per interval and half, and at 32768 chains leaves half of the SIMDs idle).
//
// Spatial half.  Intervals do not interact, so the T lanes take move k of
// their own interval together: n_stab steps instead of T n_stab.
//
// Time half.  Move (t, q, P) touches qubit q in intervals t and t + 1 and the
// outcomes of round t, so it must follow (t - 1, q, P) but may run beside moves
// (t - 1, q + 2, ...): lane t runs two qubits behind lane t - 1, at step s on
// qubit q = s - 2t, and the half takes n_q + 2 (T - 2) steps.  To keep every
// bit index a compile-time constant lane t stores its words shifted up by 2t
// positions (skewed) during the half: its own qubit is always at position s,
// qubit q of interval t + 1 at position s + 2 of lane t + 1, from where it is
// read before the half (no earlier move of the half changes it) and where an
// accepted flip goes by a one-lane DPP shift.  Two, not one, so that all lanes
// start a Philox block together.
//
// Outcomes are stored in grid-cell order (bit h is the stabilizer on cell
// 2h + 1 of the (2L-1)^2 grid; qubit q is cell 2q), which puts the neighbours
// of every qubit at h = q - 1, q (west, east), q - L and q + L - 1 (north,
// south); which of them are plaquettes, and which exist, comes from a small
// table by q.  A move's threshold is one table read by its gathered codes and
// set outcomes, "always" being 2^32 - 1 against min(u, 2^32 - 2).  n and m are
// popcounts of the words after each half.
//
// What bounds it: vector issue, once the code fits the instruction cache.  The
// spatial half is unrolled over its n_stab moves; the time half is unrolled up
// to L = 7 and else a loop over groups of 32 steps, the words turning by 32
// positions between groups so that the bit indices stay constants.  L = 7, 2048
// histories of 7 rounds, 4 chains, 784 sweeps: 204 ms one lane per chain, 43.4
// ms here (63 of 64 lanes, 3.56 waves per SIMD).  Unrolled, 300 histories of 12
// rounds at L = 12 take 6.7 ms, rolled 4.7; 1000 of 9 rounds at L = 9 5.7, 5.5.  At L = 13
// to 15 the spatial half alone outgrows the cache (100 KB of code and more) and
// some registers spill, yet it beats the streaming window of spacetime_win.h at
// every batch: 60 histories of 13 rounds at L = 13, 145 sweeps, 260 ms there, 13
// here; 3000 of 14 at L = 14 8.2, 2.9; 16000 of 9 at L = 15 11.3, 7.6; 30000 of 3
// at L = 13 7.0, 5.4 (with 3 waves per SIMD and fewer spills 13, 2.9, 8.0, 5.5).
#pragma once

#include "spacetime_common.h"

namespace mcmc {

constexpr int ST_LANES_T_MAX = 16;

// The chains of an L in this family's range; false where thresholds that are
// not "always" reach 2^32 - 1 (see above), T is larger, or one lane per chain is
// faster (spacetime_choice.h).
bool spacetime_lanes_take(const SpaceTimeArgs& a);
hipError_t launch_spacetime_lanes_small(const SpaceTimeArgs& a, hipStream_t s);   // L <= 9
hipError_t launch_spacetime_lanes_large(const SpaceTimeArgs& a, hipStream_t s);   // L <= 12
hipError_t launch_spacetime_lanes_largest(const SpaceTimeArgs& a, hipStream_t s);
constexpr int ST_LANES_SMALL_L_MAX = 9, ST_LANES_LARGE_L_MAX = 12, ST_LANES_L_MAX = 15;

namespace {

__device__ __forceinline__ uint32_t st_next_lane(uint32_t v) {   // 0 past the wave
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x130, 0xf, 0xf, false);
}
__device__ __forceinline__ uint32_t st_prev_lane(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x138, 0xf, 0xf, false);
}
// v shifted by the constant k, left if positive
template <int K>
__device__ __forceinline__ uint32_t st_shift(uint32_t v) {
  if constexpr (K >= 0) return v << K;
  else return v >> -K;
}

constexpr int ST_WAVES = 4;   // per workgroup: they share the tables

template <int L>
struct StLanes {
  using G = StGeo<L>;
  static constexpr int NQ = G::NQ, SIDE = G::SIDE;
  static constexpr int SKEW = 2 * (ST_LANES_T_MAX - 1);          // positions, last lane
  static constexpr int STEPS = NQ + 2 * (ST_LANES_T_MAX - 2);    // of the time half, at most
  // The time half rolled into groups of 32 steps, from the size on at which its
  // code does not fit the instruction cache beside the spatial half's (8192
  // histories of 3 rounds at L = 3: 27.1 ms unrolled, 28.1 rolled; L = 7: 8.49,
  // 8.57; 1000 of 8 rounds at L = 8: 4.47, 4.40).  Outcome bits then lie one word
  // up, and both kinds of words are rings.
  static constexpr bool ROLLED = L >= 8;
  static constexpr int OFF = ROLLED ? 32 : 0;
  static constexpr int WO = (G::NSTAB + SKEW + OFF + 31) / 32;              // skewed outcome words
  static constexpr int WE = ROLLED ? 2 * WO : (NQ + SKEW + 15) / 16;        // skewed data words
  static_assert(!ROLLED || (16 * WE >= NQ + SKEW + 2 && 32 * WO >= STEPS), "room for every step");
  static constexpr int PAD = SKEW + 2;                           // table entries below qubit 0
  static constexpr int NTAB = PAD + STEPS + 2;
  // stabilizer on cell (r, c)
  static constexpr int stab_at(int r, int c) {
    return (r & 1) ? ((r - 1) / 2) * L + c / 2 : G::NSTAR + (r / 2) * (L - 1) + (c - 1) / 2;
  }
  static constexpr int stab_of_bit(int h) { return stab_at((2 * h + 1) / SIDE, (2 * h + 1) % SIDE); }
};

// Table entry of qubit q: bits 0-3 which of its west, east, north and south
// outcomes an X move toggles, 4-7 the same for Z, 8-11 and 12-15 three times
// their numbers; 0 (nothing, never accepted) outside the code.
template <int L>
__device__ __forceinline__ uint32_t st_qubit_entry(int q) {
  using S = StLanes<L>;
  if (q < 0 || q >= S::NQ) return 0u;
  const int r = (2 * q) / S::SIDE, c = 2 * q - r * S::SIDE;
  uint32_t we = 0, ns = 0;
  if (c > 0) we |= 1u;
  if (c < S::SIDE - 1) we |= 2u;
  if (r > 0) ns |= 4u;
  if (r < S::SIDE - 1) ns |= 8u;
  // X toggles plaquettes: beside a qubit of an even row, above and below one
  // of an odd row
  const uint32_t mx = (r & 1) ? ns : we, mz = (r & 1) ? we : ns;
  return mx | (mz << 4) | ((uint32_t)(3 * __builtin_popcount(mx)) << 8) |
         ((uint32_t)(3 * __builtin_popcount(mz)) << 12);
}

// weight change of code (x + 2z) under X (kind 0) or Z (kind 1)
__device__ __forceinline__ int st_term(uint32_t code, int kind) {
  const int own = (int)((code >> kind) & 1u), other = (int)((code >> (1 - kind)) & 1u);
  return (1 - other) * (1 - 2 * own);
}

template <int L>
__global__ void __launch_bounds__(64 * ST_WAVES) __attribute__((amdgpu_waves_per_eu(4)))
st_chain_lanes_kernel(const SpaceTimeArgs a) {
  using G = StGeo<L>;
  using S = StLanes<L>;
  constexpr int NQ = G::NQ, NSTAB = G::NSTAB, NSTAR = G::NSTAR, WQ = G::WQ;
  constexpr int WE = S::WE, WO = S::WO, SIDE = S::SIDE;
  __shared__ uint32_t space[2][256];        // spatial thresholds by the four codes
  __shared__ uint32_t timed[2][9][16];      // time thresholds by 3 x neighbours + set, two codes
  __shared__ uint32_t qubit[2 * S::NTAB];   // entries; the second half is all 0
  for (int k = threadIdx.x; k < 512; k += blockDim.x) {
    int delta = 0;
    for (int f = 0; f < 4; ++f) delta += st_term((uint32_t)(k >> (2 * f)) & 3u, k >> 8);
    space[k >> 8][k & 255] = delta <= 0 ? 0xFFFFFFFFu : a.sp_thr[delta - 1];
  }
  for (int k = threadIdx.x; k < 288; k += blockDim.x) {
    const int kind = k / 144, row = (k / 16) % 9, code = k & 15;
    const int many = row / 3, set = row % 3;
    uint32_t thr = 0;
    if (many > 0 && set <= many) {
      const int dn = st_term((uint32_t)code & 3u, kind) + st_term((uint32_t)code >> 2, kind);
      const int e = (dn + 2) * 5 + many - 2 * set + 2;
      thr = ((a.t_always >> e) & 1u) ? 0xFFFFFFFFu : a.t_thr[e];
    }
    timed[kind][row][code] = thr;
  }
  for (int k = threadIdx.x; k < 2 * S::NTAB; k += blockDim.x)
    qubit[k] = k < S::NTAB ? st_qubit_entry<L>(k - S::PAD) : 0u;
  __syncthreads();

  const int T = a.T, lane = threadIdx.x & 63;
  const int per_wave = 64 / T;
  const int c = lane / T, t = lane - c * T;
  const int64_t first = ((int64_t)blockIdx.x * ST_WAVES + (threadIdx.x >> 6)) * per_wave;
  if (first >= a.n_tasks) return;
  // idle lanes and chains past the end repeat the last chain and store nothing
  const bool mine = c < per_wave && first + c < a.n_tasks;
  const StTask tk = st_task(a, mine ? first + c : a.n_tasks - 1);

  // interval t's data error: none before the last interval, there the class
  // start; round t's outcomes: every flipped one blamed on the measurement
  uint32_t e[WQ], out[WO];
  static_for<WQ>([&](auto WW) { e[decltype(WW)::value] = 0u; });
  static_for<WO>([&](auto WW) { out[decltype(WW)::value] = 0u; });
  if (c < per_wave && t == T - 1) {
    const uint8_t* rep = a.reps + (tk.item * 4 + tk.cls) * NQ;
    static_for<NQ>([&](auto QQ) {
      constexpr int q = decltype(QQ)::value;
      e[q >> 4] |= (uint32_t)(rep[q] & 3u) << (2 * (q & 15));
    });
  } else if (c < per_wave) {
    const uint8_t* o = a.obs + (tk.item * T + t) * NSTAB;
    uint32_t raw[WO + 1];   // a word up, for the shift; two if rolled
    static_for<WO + 1>([&](auto WW) { raw[decltype(WW)::value] = 0u; });
    static_for<NSTAB>([&](auto HH) {
      constexpr int h = decltype(HH)::value;
      if (o[S::stab_of_bit(h)] != 0) raw[(h >> 5) + 1 + S::OFF / 32] |= 1u << (h & 31);
    });
    // skewed for good: the spatial half does not use them
    static_for<WO>([&](auto WW) {
      constexpr int w = decltype(WW)::value;
      out[w] = (uint32_t)(((((uint64_t)raw[w + 1] << 32) | raw[w]) << (2 * t)) >> 32);
    });
  }

  ChainRng rng;
  rng.init(a.k0, a.k1, tk.sid, (3u << 30) | ((uint32_t)tk.cls << 28) | (1u << 20) |
                                   (uint32_t)tk.chain);
  auto block = [&](uint32_t b) -> uint4 {
    uint32_t hi0, lo0, qh, ql;
    mulhilo(PHILOX_M0, b, hi0, lo0);
    mulhilo(PHILOX_M1, hi0 ^ rng.ctr3, qh, ql);
    uint4 v = make_uint4(qh ^ rng.sid_x, ql, rng.sw_x ^ lo0, rng.sw_lo);
#pragma unroll
    for (uint32_t r = 2; r < 10; ++r) v = philox_round(v, a.k0 + r * PHILOX_W0, a.k1 + r * PHILOX_W1);
    return make_uint4(min(v.x, 0xFFFFFFFEu), min(v.y, 0xFFFFFFFEu), min(v.z, 0xFFFFFFFEu),
                      min(v.w, 0xFFFFFFFEu));
  };
  auto weight = [&]() -> int32_t {
    int32_t n = 0;
    static_for<WQ>([&](auto WW) {
      const uint32_t v = e[decltype(WW)::value];
      n += (int32_t)__builtin_popcount((v | (v >> 1)) & 0x55555555u);
    });
    return n;
  };
  auto outcomes = [&]() -> int32_t {
    int32_t m = 0;
    static_for<WO>([&](auto WW) { m += (int32_t)__builtin_popcount(out[decltype(WW)::value]); });
    return m;
  };

  // the skew is 4t bits of the data words: t / 8 words and 4 (t mod 8) bits
  const bool word_skew = (t & 8) != 0;
  const uint32_t bit_skew = 4u * (uint32_t)(t & 7);
  // this lane's entry at step s; the last interval and idle lanes never move
  const uint32_t* entry = qubit + (t < T - 1 && c < per_wave ? S::PAD - 2 * t : S::NTAB);
  const uint32_t space_block = (uint32_t)t * (NSTAB / 4);
  const uint32_t time_block = (uint32_t)T * (NSTAB / 4) + (uint32_t)t * ((NQ + 1) / 2) - (uint32_t)t;
  const int steps = NQ + 2 * (T - 2);
  const char* thr_space = reinterpret_cast<const char*>(&space[0][0]);
  const char* thr_time = reinterpret_cast<const char*>(&timed[0][0][0]);
  auto threshold = [&](const char* table, uint32_t at) {
    return *reinterpret_cast<const uint32_t*>(table + at);
  };

  int32_t n = weight(), m = outcomes();
  int64_t Sn = 0, Sm = 0, Acnt = 0;
  for (int sweep = 0; sweep < a.sweep_end; ++sweep) {
    const bool counted = sweep >= a.burn;
    rng.begin_sweep((uint32_t)sweep);
    uint32_t moves = 0;
    // ---------------- spatial half: move k of every interval ----------------
    uint4 next = block(space_block);
    static_for<NSTAB / 4>([&](auto BB) {
      constexpr int b = decltype(BB)::value;
      const uint4 blk = next;
      if constexpr (b + 1 < NSTAB / 4) next = block(st_opaque(space_block + (uint32_t)(b + 1)));
      static_for<4>([&](auto DD) {
        constexpr int s = 4 * b + decltype(DD)::value;
        constexpr int kind = s < NSTAR ? 0 : 1;
        constexpr int k = kind ? s - NSTAR : s, wd = kind ? L - 1 : L;
        constexpr int r = kind ? 2 * (k / wd) : 2 * (k / wd) + 1;
        constexpr int col = kind ? 2 * (k % wd) + 1 : 2 * (k % wd);
        constexpr int up = r > 0 ? ((r - 1) * SIDE + col) / 2 : -1;
        constexpr int down = r < SIDE - 1 ? ((r + 1) * SIDE + col) / 2 : -1;
        constexpr int left = col > 0 ? (r * SIDE + col - 1) / 2 : -1;
        constexpr int right = col < SIDE - 1 ? (r * SIDE + col + 1) / 2 : -1;
        // codes of the four qubits; a missing one reads Y, which no move of
        // either kind changes the weight of
        auto code_at = [&](auto QQ) -> uint32_t {
          constexpr int q = decltype(QQ)::value;
          if constexpr (q < 0) return 3u;
          else return (e[q >> 4] >> (2 * (q & 15))) & 3u;
        };
        uint32_t code;
        if constexpr (left >= 0 && right >= 0 && (left >> 4) == (right >> 4))
          code = (e[left >> 4] >> (2 * (left & 15))) & 15u;
        else
          code = code_at(std::integral_constant<int, left>{}) |
                 (code_at(std::integral_constant<int, right>{}) << 2);
        code = (code << 2) | code_at(std::integral_constant<int, down>{});
        code = (code << 2) | code_at(std::integral_constant<int, up>{});
        const uint32_t thr = threshold(thr_space + 1024 * kind, code << 2);
        const uint32_t am = word_of(blk, s & 3) < thr ? 0xFFFFFFFFu : 0u;
        moves -= am;
        constexpr int qs[4] = {up, down, left, right};
        static_for<WQ>([&](auto WW) {
          constexpr int w = decltype(WW)::value;
          constexpr uint32_t flip = [&] {
            uint32_t f = 0;
            for (int x : qs)
              if (x >= 0 && (x >> 4) == w) f |= (1u << kind) << (2 * (x & 15));
            return f;
          }();
          if constexpr (flip != 0) e[w] = bitop3<0x78>(e[w], am, flip);   // a ^ (b & c)
        });
        st_fence(e);
        st_fence1(moves);
      });
    });
    n = weight();
    if (counted) { Sn += n; Sm += m; }

    // ---------------- time half ----------------
    if (T > 1) {
      // skew the data words, and take interval t + 1's, one lane up and two
      // positions on
      uint32_t es[WE], nb[WE];
      static_for<WE>([&](auto WW) {
        constexpr int w = decltype(WW)::value;
        auto at = [&](auto KK) -> uint32_t {
          constexpr int k = decltype(KK)::value;
          if constexpr (k < 0 || k >= WQ) return 0u;
          else return e[k];
        };
        const uint32_t hi = word_skew ? at(std::integral_constant<int, w - 1>{})
                                      : at(std::integral_constant<int, w>{});
        const uint32_t lo = word_skew ? at(std::integral_constant<int, w - 2>{})
                                      : at(std::integral_constant<int, w - 1>{});
        es[w] = (uint32_t)(((((uint64_t)hi << 32) | lo) << bit_skew) >> 32);
      });
      static_for<WE>([&](auto WW) {
        constexpr int w = decltype(WW)::value;
        const uint32_t lo = st_next_lane(es[w]);
        uint32_t hi = 0;
        if constexpr (w + 1 < WE) hi = st_next_lane(es[w + 1]);
        nb[w] = __builtin_amdgcn_alignbit(hi, lo, 4u);
      });
      uint4 tnext = block(time_block);
#pragma unroll 1
      for (int group = 0; group < (S::ROLLED ? WO : 1); ++group) {
        const int left = steps - 32 * group;
        const uint32_t* group_entry = entry + 32 * group;
        const uint32_t group_block = time_block + 16u * (uint32_t)group;
        static_for<S::ROLLED ? 16 : (S::STEPS + 1) / 2>([&](auto PP) {
          constexpr int i0 = 2 * decltype(PP)::value;
          // uniform; always for the first n_q steps
          if ((!S::ROLLED && i0 < NQ) || i0 < left) {
            const uint4 blk = tnext;
            tnext = block(st_opaque(group_block + (uint32_t)(i0 / 2 + 1)));
            static_for<2>([&](auto HH) {
              constexpr int i = i0 + decltype(HH)::value;   // step 32 group + i
              const uint32_t en = group_entry[i];
              // outcomes west, east, north, south of the qubit at bits 0..3
              constexpr int pe = i + S::OFF, pw = pe - 1, pn = pe - L, ps = pe + L - 1;
              constexpr bool pair = pw >= 0 && (pw >> 5) == (pe >> 5) && (pe >> 5) < WO;
              auto bit_at = [&](auto KK) -> uint32_t {
                constexpr int p = decltype(KK)::value;
                if constexpr (p < 0 || (p >> 5) >= WO) return 0u;
                else return (out[p >> 5] >> (p & 31)) & 1u;
              };
              uint32_t around;
              if constexpr (pair)
                around = (out[pe >> 5] >> (pw & 31)) & 3u;
              else
                around = bit_at(std::integral_constant<int, pw>{}) |
                         (bit_at(std::integral_constant<int, pe>{}) << 1);
              around |= bit_at(std::integral_constant<int, pn>{}) << 2;
              around |= bit_at(std::integral_constant<int, ps>{}) << 3;
              // the qubit's codes in intervals t and t + 1, times 4
              constexpr int w = i >> 4, sh = 2 * (i & 15);
              uint32_t codes = 0;
              if constexpr (w < WE)
                codes = (((es[w] >> sh) & 3u) << 2) | (((nb[w] >> sh) & 3u) << 4);
              // X: row 3 x neighbours + set ones of its table
              const uint32_t row_x =
                  (uint32_t)__builtin_popcount(around & en & 15u) + ((en >> 8) & 15u);
              const uint32_t thr_x = threshold(thr_time, (row_x << 6) + codes);
              const uint32_t ax = word_of(blk, (2 * i) & 3) < thr_x ? 0xFFFFFFFFu : 0u;
              codes = bitop3<0x78>(codes, ax, 0x14u);
              const uint32_t en_z = en >> 4;
              const uint32_t row_z = (uint32_t)__builtin_popcount(around & en_z & 15u) + (en >> 12);
              const uint32_t thr_z = threshold(thr_time + 576, (row_z << 6) + codes);
              const uint32_t az = word_of(blk, (2 * i + 1) & 3) < thr_z ? 0xFFFFFFFFu : 0u;
              moves -= ax;
              moves -= az;
              // flips: the qubit here and, two positions on, one lane up ...
              const uint32_t flip = (ax & 1u) | (az & 2u);
              if constexpr (w < WE) es[w] ^= flip << sh;
              constexpr int wu = (i + 2) >> 4, shu = 2 * ((i + 2) & 15);
              if constexpr (wu < WE) es[wu] ^= st_prev_lane(flip << shu);
              // ... and the outcomes around it
              const uint32_t turn = (ax & en & 15u) ^ (az & en_z & 15u);
              if constexpr (pair) {
                out[pe >> 5] =
                    bitop3<0x78>(out[pe >> 5], turn << (pw & 31), 3u << (pw & 31));
              } else {
                if constexpr (pw >= 0 && (pw >> 5) < WO)
                  out[pw >> 5] = bitop3<0x78>(out[pw >> 5], turn << (pw & 31), 1u << (pw & 31));
                if constexpr ((pe >> 5) < WO)
                  out[pe >> 5] =
                      bitop3<0x78>(out[pe >> 5], st_shift<(pe & 31) - 1>(turn), 1u << (pe & 31));
              }
              if constexpr (pn >= 0 && (pn >> 5) < WO)
                out[pn >> 5] =
                    bitop3<0x78>(out[pn >> 5], st_shift<(pn & 31) - 2>(turn), 1u << (pn & 31));
              if constexpr ((ps >> 5) < WO)
                out[ps >> 5] =
                    bitop3<0x78>(out[ps >> 5], st_shift<(ps & 31) - 3>(turn), 1u << (ps & 31));
              st_fence(es);
              st_fence(out);
              st_fence1(moves);
            });
          }
        });
        if constexpr (S::ROLLED) {
          // turn the rings; interval t + 1's words are used up
          const uint32_t es0 = es[0], es1 = es[1], out0 = out[0];
          static_for<WE - 2>([&](auto WW) {
            constexpr int w = decltype(WW)::value;
            es[w] = es[w + 2];
            nb[w] = nb[w + 2];
          });
          es[WE - 2] = es0;
          es[WE - 1] = es1;
          static_for<WO - 1>([&](auto WW) {
            out[decltype(WW)::value] = out[decltype(WW)::value + 1];
          });
          out[WO - 1] = out0;
        }
      }
      // back to plain positions
      static_for<WQ>([&](auto WW) {
        constexpr int w = decltype(WW)::value;
        auto at = [&](auto KK) -> uint32_t {
          constexpr int k = decltype(KK)::value;
          if constexpr (k >= WE) return 0u;
          else return es[k];
        };
        const uint32_t lo = word_skew ? at(std::integral_constant<int, w + 1>{})
                                      : at(std::integral_constant<int, w>{});
        const uint32_t hi = word_skew ? at(std::integral_constant<int, w + 2>{})
                                      : at(std::integral_constant<int, w + 1>{});
        e[w] = __builtin_amdgcn_alignbit(hi, lo, bit_skew);
      });
      n = weight();
      m = outcomes();
    }
    if (counted) { Sn += n; Sm += m; }
    Acnt += moves;
  }

  // the chain's sums over its lanes, and its accumulated data error, to lane 0
  auto lane_sum = [&](int64_t v) -> int64_t {
    int64_t sum = v;
    for (int k = 1; k < T; ++k) {
      const int from = lane + k;
      const int lo = __shfl((int)(uint32_t)v, from & 63), hi = __shfl((int)(v >> 32), from & 63);
      sum += (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
    }
    return sum;
  };
  const int64_t sum_n = lane_sum(Sn), sum_m = lane_sum(Sm), sum_a = lane_sum(Acnt);
  const int64_t last_n = lane_sum(n), last_m = lane_sum(m);
  if (mine && t == 0) {
    const int64_t at = tk.item * 4 * a.chains + tk.rem;
    a.Sn[at] = sum_n;
    a.Sm[at] = sum_m;
    a.A[at] = sum_a;
    a.n_final[at] = (int32_t)last_n;
    a.m_final[at] = (int32_t)last_m;
  }
  if (a.final_c) {
    uint8_t* o = a.final_c + (tk.item * 4 + tk.cls) * NQ;
    static_for<WQ>([&](auto WW) {
      constexpr int w = decltype(WW)::value;
      uint32_t word = e[w];
      for (int k = 1; k < T; ++k) word ^= (uint32_t)__shfl((int)e[w], (lane + k) & 63);
      if (mine && t == 0 && tk.chain == 0)
        for (int f = 0; f < 16 && 16 * w + f < NQ; ++f)
          o[16 * w + f] = (uint8_t)((word >> (2 * f)) & 3u);
    });
  }
}

template <int L>
hipError_t launch_lanes(const SpaceTimeArgs& a, hipStream_t s) {
  const int64_t per_group = (int64_t)(64 / a.T) * ST_WAVES;
  const int64_t groups = (a.n_tasks + per_group - 1) / per_group;
  if (groups > 0x7FFFFFFF) return hipErrorInvalidValue;
  hipLaunchKernelGGL(st_chain_lanes_kernel<L>, dim3((unsigned)groups), dim3(64 * ST_WAVES), 0, s, a);
  return hipGetLastError();
}

template <int LL, int LMAX>
hipError_t dispatch_lanes(const SpaceTimeArgs& a, hipStream_t s) {
  if constexpr (LL > LMAX) {
    return hipErrorInvalidValue;
  } else {
    if (a.L == LL) return launch_lanes<LL>(a, s);
    return dispatch_lanes<LL + 1, LMAX>(a, s);
  }
}

}  // namespace

}  // namespace mcmc
