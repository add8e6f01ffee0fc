// Colour-phased Metropolis chains, one chain over L lanes (Sec. IV, Sec. IV.A,
// Sec. V of arXiv:1302.2669): the mapping of batches too small to fill the
// chip with one chain per lane.
//
// What bounds it.  A chain of chain_body.h is one lane's serial work: a sweep
// at L = 13 takes a wave 25 us however few waves there are, so a batch below
// one wave per SIMD costs the same 4.3 ms (169 sweeps) as one syndrome.  Rows
// of one colour share no qubit, so lane i of a chain's L lanes owns grid rows
// 2i and 2i + 1 and decides star row i or plaquette row i of the phase; the
// rows it shares with its neighbours move by one-lane DPP shifts (a star row
// reads the even row of lane i + 1 and flips it, a plaquette row the odd row
// of lane i - 1).  A phase is then a few dozen instructions instead of L rows
// of them: 1952 chains at L = 13 take 1.4 us per sweep (19 one per lane), 64016 3.2
// ms instead of 5.3 with flips and 169 sweeps.
//
// Draws.  The 2 L (L - 1) draws of a sweep are the L (L - 1) / 2 Philox
// blocks of the one-lane kernel, block b on lane b mod L, so no block is
// computed twice although rows start anywhere inside one.  A draw u matters
// only through how many of the four thresholds it reaches, and that does not
// depend on the state: qbar = #{k : u >= A[k]} (the thresholds fall with k),
// a move with t = Delta n + 4 is rejected iff t + qbar >= 9.  So a block is
// reduced to four 4-bit counts as it is drawn, the counts go through LDS (2
// bytes per block, one wave, no barrier) one sweep ahead, each lane reads its
// rows' counts as nibble strings at any alignment, and a whole row is decided
// by four word operations: no threshold lookup is left on the serial path.
//
// Against the one-lane kernel it issues 1.5 to 1.7 times the instructions per
// update (idle lanes when L does not divide 64, eight compares per draw), so
// full batches stay there (chain_choice.h).  Counting the far two thresholds
// only when some lane's draw of a block reaches that low saves a seventh of the
// instructions at p = 0.1, but its branches keep a lone wave from overlapping
// draws with phases (0.56 -> 0.71 us per sweep at L = 3) and cost registers
// (1.4 times slower at L = 25), so all four are counted.
#pragma once

#include "chain_body.h"

namespace mcmc {

// Rank of row i's first site in its colour: star_row_rank and plaq_row_rank
// in closed form for a runtime row.
template <int L>
__device__ __forceinline__ int star_rank(int i, int phi) {
  return i * (L / 2) + (L % 2 ? (i + 1 - phi) / 2 : 0);
}
template <int L>
__device__ __forceinline__ int plaq_rank(int i, int phi) {
  return L % 2 ? i * ((L - 1) / 2) : i * (L / 2 - 1) + (i + 1 - phi) / 2;
}

// Value of the next / previous lane (all ones past the wave's ends).
__device__ __forceinline__ uint32_t lane_above(uint32_t v, uint32_t edge) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)edge, (int)v, 0x130, 0xf, 0xf, false);
}
__device__ __forceinline__ uint32_t lane_below(uint32_t v, uint32_t edge) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)edge, (int)v, 0x138, 0xf, 0xf, false);
}

// acc plus how many of the four thresholds u reaches.  A mask (VCC or an SGPR pair)
// is read from the third instruction after the VALU one that writes it, at the
// earliest.  FILLED: other compares and adds fill that gap, four of the eight
// instructions in their 8-byte encoding; else one mask beside VCC and a few wait
// states, which other waves' instructions fill.  Measured against a gap left open:
// 16 x 1000 syndromes at L = 3 0.96 of the time, 4001 x 16 chains at L = 13, 17 and
// 25 with flips 1.03, 1.05, 1.03 filled and 1.01, 1.02, 0.99 with waits, 200 x 16
// at L = 13 0.98 and 1.02 (wait states alone: 1.10 there, 0.98 at 4001).
template <bool FILLED>
__device__ __forceinline__ uint32_t count_reached(uint32_t acc, uint32_t u,
                                                  const uint32_t (&thr)[4]) {
  uint64_t m0;
  if constexpr (FILLED) {
    uint64_t m1;
    asm("v_cmp_ge_u32 vcc, %3, %4\n\tv_cmp_ge_u32 %1, %3, %5\n\t"
        "v_cmp_ge_u32 %2, %3, %6\n\tv_addc_co_u32 %0, vcc, 0, %0, vcc\n\t"
        "v_cmp_ge_u32 vcc, %3, %7\n\tv_addc_co_u32 %0, %1, 0, %0, %1\n\t"
        "v_addc_co_u32 %0, %2, 0, %0, %2\n\tv_addc_co_u32 %0, vcc, 0, %0, vcc"
        : "+&v"(acc), "=&s"(m0), "=&s"(m1)
        : "v"(u), "v"(thr[0]), "v"(thr[1]), "v"(thr[2]), "v"(thr[3])
        : "vcc");
  } else {
    asm("v_cmp_ge_u32 vcc, %2, %3\n\tv_cmp_ge_u32 %1, %2, %4\n\ts_nop 0\n\t"
        "v_addc_co_u32 %0, vcc, 0, %0, vcc\n\tv_cmp_ge_u32 vcc, %2, %5\n\t"
        "v_addc_co_u32 %0, %1, 0, %0, %1\n\ts_nop 0\n\tv_addc_co_u32 %0, vcc, 0, %0, vcc\n\t"
        "v_cmp_ge_u32 vcc, %2, %6\n\ts_nop 1\n\tv_addc_co_u32 %0, vcc, 0, %0, vcc"
        : "+&v"(acc), "=&s"(m0)
        : "v"(u), "v"(thr[0]), "v"(thr[1]), "v"(thr[2]), "v"(thr[3])
        : "vcc");
  }
  return acc;
}
// The filled form where a wave waits for itself: one chain per wave, and the codes
// whose few draws leave waves idle (up to L = 9 it also wins in full batches).
constexpr int FILLED_L_MAX = 9;

// G lanes per chain: its rows on the first L, its draws on all of them.
template <int L, int G>
struct SplitGeo {
  static_assert(G >= L && G <= 64, "a lane per row pair");
  static constexpr int CW = 64 / G;                       // chains per wave
  static constexpr int SLOTS = 63 / G + 1;                // with the idle lanes' slot
  static constexpr int NB = (L * (L - 1) / 2 + G - 1) / G;   // Philox blocks per lane and sweep
  // words of one chain's counts: NB G blocks of 4 nibbles, and the reads of
  // up to two words past a row's first
  static constexpr int WORDS = (NB * G + 1) / 2 + 2;
};

// Tile t0 .. t0 + CW - 1 of group g on this wave.  lds: SLOTS * WORDS words of
// counts, then 64 x (S, A, n) of the lanes at the end.
template <int L, int NOISE, int G>
__device__ __forceinline__ void run_split(const RunArgs& a, const GroupDesc& g, int64_t t0,
                                          uint32_t* lds) {
  using P = SplitGeo<L, G>;
  constexpr int W = Geo<L>::W, S = Geo<L>::S, NB = P::NB;
  const int lane = threadIdx.x & 63;
  const int c = lane / G, i = lane - c * G;      // chain slot and row pair of this lane
  const int K = g.K, C = g.C;

  // task -> (item, class, temperature, replica); idle lanes and the slots
  // past the group's end repeat its last task and store nothing
  const bool mine = c < P::CW && t0 + c < g.n_tasks;
  const int64_t t = mine ? t0 + c : g.n_tasks - 1;
  const int64_t per_item = 4 * (int64_t)K * C;
  const int64_t item_local = t / per_item;
  const int rem = (int)(t - item_local * per_item);
  const int chain = rem % C;
  const int kt = (rem / C) % K;
  const int cls = rem / (C * K);
  const ItemDesc it = item_of(a, g.first_item + item_local, Geo<L>::RW);
  const int64_t out = it.chain_off + rem;

  uint32_t thr[4];
#pragma unroll
  for (int k = 0; k < 4; ++k)
    thr[k] = a.tables ? a.tables[it.table_off + kt * 4 + k] : a.table0[kt][k];

  // rows 2i and 2i + 1; rows past the code are all padding
  const bool has_odd = i < L - 1, has_even = i < L;
  uint32_t ev[W], od[W];
  static_for<W>([&](auto WW) {
    constexpr int w = decltype(WW)::value;
    const int re = 2 * i * W + w, ro = (2 * i + 1) * W + w;
    if (a.resume_rows) {
      ev[w] = has_even ? a.resume_rows[(int64_t)re * a.total_chains + out] : 0xFFFFFFFFu;
      od[w] = has_odd ? a.resume_rows[(int64_t)ro * a.total_chains + out] : 0xFFFFFFFFu;
    } else {
      ev[w] = has_even ? a.init_rows[it.rows_off + re * 4 + cls] : 0xFFFFFFFFu;
      od[w] = has_odd ? a.init_rows[it.rows_off + ro * 4 + cls] : 0xFFFFFFFFu;
    }
    ev[w] = reg_code(ev[w]);
    od[w] = reg_code(od[w]);
  });
  // 8 x this lane's share of the weight (the first lane starts with all of
  // it) and of its sum over the counted phases, and its accepted moves
  int32_t n8 = 0;
  if (i == 0) n8 = 8 * (a.resume_rows ? a.resume_n[out] : a.init_n[it.orig * 4 + cls]);
  int64_t S8 = 0, Acnt = 0;

  // per colour phase: this lane's sites, field shift and place in the counts
  uint32_t sites[4][W];
  int at[4], sh[4];
  const int odd_row = i & 1;
  static_for<4>([&](auto PH) {
    constexpr int ph = decltype(PH)::value;
    const int par = odd_row ^ (ph & 1);
    static_for<W>([&](auto WW) {
      constexpr int w = decltype(WW)::value;
      constexpr int limit = ph < 2 ? L : L - 1;
      sites[ph][w] = par ? site_tops(1, limit, w) : site_tops(0, limit, w);
      if (ph < 2 ? !has_odd : !has_even) sites[ph][w] = 0u;
    });
    const int rank = ph < 2 ? star_rank<L>(has_odd ? i : 0, ph)
                            : plaq_rank<L>(has_even ? i : 0, ph - 2);
    const int d = ph * S + rank;
    at[ph] = d >> 3;
    sh[ph] = 4 * (d & 7);
  });
  const uint32_t own_odd = has_odd ? 0xFFFFFFFFu : 0u;
  // bit/phase flips: the padding reads c = 0, a missing neighbour is c = 1
  const uint32_t no_above = i == 0 ? 0x55555555u : 0u, no_below = has_odd ? 0u : 0x55555555u;

  // block b = i + G k after its second round holds (pa ^ ..., pb, lo ^ ...,
  // ...): the parts that only depend on the chain and the block
  ChainRng rng;
  rng.init(a.k0, a.k1, it.sid, ((uint32_t)cls << 28) | ((uint32_t)(kt + 1) << 20) | (uint32_t)chain);
  uint32_t pa[NB], pb[NB], lo[NB];
  static_for<NB>([&](auto KK) {
    constexpr int k = decltype(KK)::value;
    uint32_t hi0, qh;
    mulhilo(PHILOX_M0, (uint32_t)(i + G * k), hi0, lo[k]);
    mulhilo(PHILOX_M1, hi0 ^ rng.ctr3, qh, pb[k]);
    pa[k] = qh ^ rng.sid_x;
  });

  uint32_t* counts = lds + c * P::WORDS;
  uint16_t* drawn = reinterpret_cast<uint16_t*>(counts) + i;
  auto draw_sweep = [&](uint32_t sweep) {
    rng.begin_sweep(sweep);
    static_for<NB>([&](auto KK) {
      constexpr int k = decltype(KK)::value;
      uint4 v = make_uint4(pa[k], pb[k], rng.sw_x ^ lo[k], rng.sw_lo);
      static_for<8>([&](auto RR) {
        constexpr uint32_t r = 2 + decltype(RR)::value;
        v = philox_round(v, a.k0 + r * PHILOX_W0, a.k1 + r * PHILOX_W1);
      });
      uint32_t q = 0;
      static_for<4>([&](auto DD) {
        constexpr int d = 3 - decltype(DD)::value;
        if constexpr (d < 3) q <<= 4;
        q = count_reached<G == 64 || L <= FILLED_L_MAX>(q, word_of(v, d), thr);
      });
      drawn[G * k] = (uint16_t)q;
    });
  };
  auto order_lds = [&]() {   // one wave's LDS accesses run in order: hold the compiler to it
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };

  if (g.sweep_begin < g.sweep_end) draw_sweep((uint32_t)g.sweep_begin);
  for (int sweep = g.sweep_begin; sweep < g.sweep_end; ++sweep) {
    order_lds();
    uint32_t qbar[4][W];
    static_for<4>([&](auto PH) {
      constexpr int ph = decltype(PH)::value;
      uint32_t word[W + 1];
      static_for<W + 1>([&](auto WW) { word[decltype(WW)::value] = counts[at[ph] + decltype(WW)::value]; });
      static_for<W>([&](auto WW) {
        constexpr int w = decltype(WW)::value;
        qbar[ph][w] = __builtin_amdgcn_alignbit(word[w + 1], word[w], (uint32_t)sh[ph]);
      });
    });
    order_lds();
    draw_sweep((uint32_t)sweep + 1);

    // sum holds t = Delta n + 4 in the nibble of every site of the lane's row
    uint32_t sum[W], acc[W];
    int32_t moves = 0, s8 = 0;   // of this sweep
    auto decide = [&](auto PH) {
      constexpr int ph = decltype(PH)::value;
      int32_t cnt = 0;
      static_for<W>([&](auto WW) {
        constexpr int w = decltype(WW)::value;
        const uint32_t r = sum[w] + qbar[ph][w];              // <= 12; >= 9: rejected
        const uint32_t low = (r & 0x77777777u) + 0x77777777u;  // top bit: r mod 8 != 0
        acc[w] = bitop3<0x2A>(r, low, sites[ph][w]);          // ~(a & b) & c
        n8 = (int32_t)__builtin_amdgcn_udot8(sum[w], acc[w], (uint32_t)n8, false);
        cnt += (int32_t)__builtin_popcount(acc[w]);
      });
      n8 -= 32 * cnt;
      moves += cnt;
      s8 += n8;
    };

    // ---------------- stars: colours 0 and 1 ----------------
    static_for<2>([&](auto PH) {
      constexpr int ph = decltype(PH)::value;
      const uint32_t s0 = 2u * (uint32_t)(odd_row ^ ph);
      constexpr uint32_t M = 0x33333333u;
      uint32_t cO[W];
      static_for<W>([&](auto WW) {
        constexpr int w = decltype(WW)::value;
        cO[w] = c_star_of<NOISE>(od[w]);
        if constexpr (NOISE == 1) cO[w] |= 0x55555555u & ~field_mask(L - 1, w);
      });
      static_for<W>([&](auto WW) {
        constexpr int w = decltype(WW)::value;
        const uint32_t cN = c_star_of<NOISE>(ev[w]);
        const uint32_t cS = lane_above(cN, 0u);
        uint32_t cWest;
        if constexpr (w == 0) cWest = (cO[0] << 2) | 1u;
        else cWest = (cO[w] << 2) | (cO[w - 1] >> 30);
        sum[w] = ((cN >> s0) & M) + ((cS >> s0) & M) + ((cO[w] >> s0) & M) + ((cWest >> s0) & M);
      });
      decide(PH);
      // accepted sites at bit 3 of their nibbles -> the fields' high bits
      uint32_t ax[W];
      static_for<W>([&](auto WW) { ax[decltype(WW)::value] = acc[decltype(WW)::value] >> (2u - s0); });
      static_for<W>([&](auto WW) {
        constexpr int w = decltype(WW)::value;
        ev[w] ^= ax[w] ^ lane_below(ax[w], 0u);
        uint32_t westward = ax[w] >> 2;
        if constexpr (w + 1 < W) westward |= ax[w + 1] << 30;
        od[w] ^= (ax[w] | westward) & field_mask(L - 1, w) & 0xAAAAAAAAu;
      });
    });

    // ---------------- plaquettes: colours 2 and 3 ----------------
    static_for<2>([&](auto PH) {
      constexpr int ph = 2 + decltype(PH)::value;
      const uint32_t s0 = 2u * (uint32_t)(odd_row ^ (ph & 1));
      constexpr uint32_t M = 0x33333333u;
      uint32_t cE[W];
      static_for<W>([&](auto WW) { cE[decltype(WW)::value] = c_plaq_of<NOISE>(ev[decltype(WW)::value]); });
      static_for<W>([&](auto WW) {
        constexpr int w = decltype(WW)::value;
        uint32_t cS = c_plaq_of<NOISE>(od[w]);
        uint32_t cN = lane_below(cS, 0x55555555u);
        if constexpr (NOISE == 1) {
          cN |= no_above;
          cS |= no_below;
        }
        uint32_t cEast = cE[w] >> 2;
        if constexpr (w + 1 < W) cEast |= cE[w + 1] << 30;
        sum[w] = ((cN >> s0) & M) + ((cS >> s0) & M) + ((cE[w] >> s0) & M) + ((cEast >> s0) & M);
      });
      decide(std::integral_constant<int, ph>{});
      // -> the fields' low bits
      uint32_t az[W];
      static_for<W>([&](auto WW) { az[decltype(WW)::value] = acc[decltype(WW)::value] >> (3u - s0); });
      static_for<W>([&](auto WW) {
        constexpr int w = decltype(WW)::value;
        od[w] ^= (az[w] ^ lane_above(az[w], 0u)) & own_odd;
        uint32_t eastward = az[w] << 2;
        if constexpr (w > 0) eastward |= az[w - 1] >> 30;
        ev[w] ^= az[w] | eastward;
      });
    });
    Acnt += moves;
    if (sweep >= g.burn) S8 += s8;
  }

  // the chain's sums: its first lane adds the lanes' shares
  order_lds();
  int64_t* part = reinterpret_cast<int64_t*>(lds + ((P::SLOTS * P::WORDS + 1) & ~1));
  part[lane] = S8;
  part[64 + lane] = Acnt;
  part[128 + lane] = n8;
  order_lds();
  if (mine && i == 0) {
    int64_t sum8 = 0, ac = 0, nn = 0;
    for (int k = 0; k < L; ++k) {
      sum8 += part[lane + k];
      ac += part[64 + lane + k];
      nn += part[128 + lane + k];
    }
    a.S_out[out] = (a.resume_rows ? a.resume_S[out] : 0) + sum8 / 8;
    a.A_out[out] = (a.resume_rows ? a.resume_A[out] : 0) + ac;
    a.n_out[out] = (int32_t)(nn / 8);
  }
  order_lds();
  if (mine && has_even) {
    static_for<W>([&](auto WW) {
      constexpr int w = decltype(WW)::value;
      const int re = 2 * i * W + w, ro = (2 * i + 1) * W + w;
      if (a.state_rows) {
        a.state_rows[(int64_t)re * a.total_chains + out] = row_code(ev[w]);
        if (has_odd) a.state_rows[(int64_t)ro * a.total_chains + out] = row_code(od[w]);
      }
      if (a.final_rows && chain == 0 && kt == K - 1) {
        a.final_rows[it.rows_off + re * 4 + cls] = row_code(ev[w]);
        if (has_odd) a.final_rows[it.rows_off + ro * 4 + cls] = row_code(od[w]);
      }
    });
  }
}

// LDS words of one wave for the largest need among LMIN .. LMAX; LANES 0: L
// lanes per chain.
template <int LMIN, int LMAX, int LANES = 0>
__host__ __device__ constexpr int split_words() {
  int most = 0;
  if constexpr (LMIN <= LMAX) {
    using P = SplitGeo<LMIN, LANES ? LANES : LMIN>;
    most = ((P::SLOTS * P::WORDS + 1) & ~1) + 3 * 128;
    const int rest = split_words<LMIN + 1, LMAX, LANES>();
    if (rest > most) most = rest;
  }
  return most;
}

template <int LMIN, int LMAX, int NOISE>
__device__ __forceinline__ void dispatch_split(const RunArgs& a, const GroupDesc& g, int L,
                                               int64_t t0, uint32_t* lds) {
  if constexpr (LMIN <= LMAX) {
    if (L == LMIN) {
      run_split<LMIN, NOISE, LMIN>(a, g, t0, lds);
      return;
    }
    dispatch_split<LMIN + 1, LMAX, NOISE>(a, g, L, t0, lds);
  }
}

// Persistent tile loop, one wave per workgroup, as in chains_persistent.  A
// plan's entry is a whole group: its first_task field holds the number of tiles
// before it.  A device-built plan has one group to split, its last.
template <int LMIN, int LMAX, int NOISE>
__device__ __forceinline__ void split_persistent(const RunArgs& a) {
  __shared__ __align__(16) uint32_t lds[split_words<LMIN, LMAX>()];
  const int lane = threadIdx.x & 63;
  const int64_t n_tiles = a.tile_cum ? (int64_t)a.tile_cum[3] : a.n_tiles;
  // a device-built plan may have fewer tiles than waves, or none: the waves beyond
  // leave the counter alone (2000 syndromes at L = 5 with 1 sweep, none of them split,
  // 227 us beside 4096 waves asking in vain, now 136)
  if ((int64_t)blockIdx.x >= n_tiles) return;
  while (true) {
    uint32_t tile = 0;
    if (lane == 0) tile = atomicAdd(a.queue, 1u);
    tile = __builtin_amdgcn_readfirstlane(tile);
    if ((int64_t)tile >= n_tiles) break;
    GroupDesc g;
    int L;
    int64_t first;
    if (a.tile_cum) {
      g = a.groups[3];
      L = g.L;
      first = (int64_t)tile * split_tile(L);
    } else if (a.tiles) {
      int lo = 0, hi = a.n_split - 1;   // the last entry that starts at or before the tile
      while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if (a.tiles[mid].first_task <= (int64_t)tile) lo = mid;
        else hi = mid - 1;
      }
      const TileDesc td = a.tiles[lo];
      g = a.groups[td.group];
      L = td.L;
      first = ((int64_t)tile - td.first_task) * split_tile(L);
    } else {
      g = a.g0;
      L = a.g0.L;
      first = a.split_from + (int64_t)tile * split_tile(L);
    }
    if (L < LMIN || L > LMAX || first >= g.n_tasks) continue;
    dispatch_split<LMIN, LMAX, NOISE>(a, g, L, first, lds);
  }
}

}  // namespace mcmc
