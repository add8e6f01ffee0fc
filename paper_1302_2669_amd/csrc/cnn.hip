// Gate network kernels: a small convolutional network over the syndrome
// planes of one code size, trained on the decoder's own class probabilities
// to predict the class and a sweep budget (the learned-gate pattern grown on
// the decoder; not part of the paper's method).
//
// Layout: activations channels-last [pixel][channel] in bfloat16 (pixel =
// sample*L*L + y*L + x); master parameters fp32 in the order W1 [32][9][3],
// b1, W2 [32][9][32], b2, W3 [32][9][32], b3, Wh [7][L*L*32], bh [7].
// Convolutions are implicit GEMMs on v_mfma_f32_16x16x32_bf16 (bf16 operands,
// fp32 accumulation): forward M = pixels, N = 32 output channels,
// K = 9 taps x input channels; backward-data the same with the taps mirrored
// and the weight roles transposed; weight gradients M = 32, N = taps x input
// channels, K = pixels (v_mfma_f32_32x32x16_bf16), split over samples and
// reduced in a fixed order.
// Lane layout of the 16x16x32 MFMA: lane l holds A[l%16][8(l/16)..+7],
// B[8(l/16)..+7][l%16] and D[4(l/16)+i][l%16], i = 0..3.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "host_common.h"
#include "internal.h"

namespace mcmc {
namespace {

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int CH = 32;

__device__ __forceinline__ bf16x8 load8(const bf16* p) {
  const uint4 v = *reinterpret_cast<const uint4*>(p);
  return __builtin_bit_cast(bf16x8, v);
}
__device__ __forceinline__ bf16x8 lds8(const bf16* p) {
  return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(p));
}
__device__ __forceinline__ bf16x8 zero8() { return __builtin_bit_cast(bf16x8, make_uint4(0, 0, 0, 0)); }

__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ int tap_dy(int t) { return t / 3 - 1; }
__device__ __forceinline__ int tap_dx(int t) { return t % 3 - 1; }

// ---- parameter casts -------------------------------------------------------
// wb1 [32][96] (k = tap*8 + ci, ci < 3), wb2/wb3 [32][288] (k = tap*32 + ci),
// wt2/wt3 [32 ci][288 (tap*32 + co)] = W[co][tap][ci], whb [16][L*L*32].
__global__ void cast_kernel(int L, const float* __restrict__ prm, const CnnOffsets off,
                            bf16* __restrict__ wb1, bf16* __restrict__ wb2, bf16* __restrict__ wb3,
                            bf16* __restrict__ wt2, bf16* __restrict__ wt3, bf16* __restrict__ whb) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t kh = (int64_t)L * L * CH;
  if (i < 32 * 96) {
    const int co = (int)(i / 96), k = (int)(i % 96), tap = k / 8, ci = k % 8;
    wb1[i] = (bf16)((tap < 9 && ci < 3) ? prm[off.W1 + (co * 9 + tap) * 3 + ci] : 0.0f);
  }
  if (i < 32 * 288) {
    wb2[i] = (bf16)prm[off.W2 + i];
    wb3[i] = (bf16)prm[off.W3 + i];
    const int ci = (int)(i / 288), k = (int)(i % 288), tap = k / 32, co = k % 32;
    wt2[i] = (bf16)prm[off.W2 + (co * 9 + tap) * 32 + ci];
    wt3[i] = (bf16)prm[off.W3 + (co * 9 + tap) * 32 + ci];
  }
  if (i < 16 * kh) {
    const int o = (int)(i / kh);
    whb[i] = (bf16)(o < 7 ? prm[off.Wh + i] : 0.0f);
  }
}

// ---- forward ---------------------------------------------------------------
// One workgroup (8 waves) runs S samples through the three convolutions and
// the head with every activation in LDS; inference touches global memory only
// for the syndromes, rates, weights and logits, and a training forward
// (STORE) also writes the planes and the three activations out for the
// backward pass.  logits[b][o] = sum_f a3[b][f] * whb[o][f] + bh[o], o < 7:
// the sum over the L*L pixel steps (32 features each) runs as 8 interleaved
// MFMA chains, wave j taking steps j, j+8, ..., added in chain order.
//
// A layer by itself is latency: 86528 pixels of 64 bytes (512 samples of
// L = 13) are a microsecond or two of traffic, but as one launch per layer,
// with the weights read again for every 16 pixels, the planes, the layers and
// the head took 3.7 + 6.6 + 2 x 13.5 + 7.7 us; this kernel takes 18.1.
constexpr int FWD_THREADS = 512;
constexpr int FWD_WAVES = FWD_THREADS / 64;
constexpr int ASTR = 40;      // bf16 per pixel of a 32-channel activation (80 B: 16 lanes
                              // reading 16 B each at this stride hit disjoint banks)
constexpr int W1STR = 104;    // bf16 per row of conv1 weights (96 used)
constexpr int W23STR = 296;   // bf16 per row of conv2/conv3 weights (288 used)
constexpr int FWD_PIXEL_BYTES = 2 * ASTR * 2 + 2;   // two activation buffers, the tap mask
constexpr int HEAD_TRIP = 24;
constexpr int FWD_WEIGHT_BYTES = 32 * W1STR * 2 + 2 * 32 * W23STR * 2;
constexpr int FWD_PART_BYTES = FWD_WAVES * 256 * 4 + 3 * CH * 4 + 16;  // + biases, zero slot

// One convolution over the group's pixels, from LDS.  Forward: relu(sum +
// bias); MIRROR (data gradient): the taps point the other way and the sum is
// kept where the layer's own input, mask, is positive.  Each wave takes two
// 16-pixel tiles per trip (four independent MFMA chains).  Weights are the
// A operand (held in VGPRs for the layer), activations the B operand, so a
// lane ends with four consecutive channels of one pixel and writes them in
// one 8-byte store: to LDS (out, if TO_LDS) and, for the first nglob
// pixels, to global memory (gout).  A tap outside the image (or a pixel past
// the group) is read from a 16-byte slot of zeros: taps[q] holds the validity
// of the nine taps of pixel q, built once per kernel (tap_masks); mirrored,
// tap t is tap 8 - t.  Biases are read from LDS as well: a global load at the
// start of each layer is 0.4 us in which nothing else runs.
template <int CIN, int WSTR, int INSTR, bool MIRROR, bool TO_LDS>
__device__ __forceinline__ void conv_lds(int L, int npix, const bf16* in, const bf16* w,
                                         const float* bias, const uint16_t* taps,
                                         const bf16* __restrict__ mask, bf16* out,
                                         bf16* __restrict__ gout, int nglob, const bf16* zslot) {
  constexpr int KP = (9 * CIN + 31) / 32 * 32;
  constexpr int STEPS = KP / 32;
  constexpr int CHUNKS = CIN / 8;
  constexpr int SGN = MIRROR ? -1 : 1;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, grp = lane >> 4, n = lane & 15;
  bf16x8 w0[STEPS], w1[STEPS];
#pragma unroll
  for (int st = 0; st < STEPS; ++st) {
    w0[st] = lds8(w + n * WSTR + st * 32 + 8 * grp);
    w1[st] = lds8(w + (n + 16) * WSTR + st * 32 + 8 * grp);
  }
  float bias0[4], bias1[4];
  if (!MIRROR) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      bias0[i] = bias[4 * grp + i];
      bias1[i] = bias[16 + 4 * grp + i];
    }
  }
  const int ntiles = (npix + 15) / 16;
  for (int t0 = wave; t0 < ntiles; t0 += 2 * FWD_WAVES) {
    int q[2];
    uint32_t valid[2];
    bf16x4 m0[2], m1[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      q[u] = (t0 + u * FWD_WAVES) * 16 + n;
      valid[u] = q[u] < npix ? taps[q[u]] : 0u;
      if (MIRROR && q[u] < nglob) {
        m0[u] = *reinterpret_cast<const bf16x4*>(mask + (int64_t)q[u] * CH + 4 * grp);
        m1[u] = *reinterpret_cast<const bf16x4*>(mask + (int64_t)q[u] * CH + 16 + 4 * grp);
      } else {
        m0[u] = m1[u] = bf16x4{0, 0, 0, 0};
      }
    }
    f32x4 acc[2][2] = {{{0, 0, 0, 0}, {0, 0, 0, 0}}, {{0, 0, 0, 0}, {0, 0, 0, 0}}};
#pragma unroll
    for (int st = 0; st < STEPS; ++st) {
      const int g = 4 * st + grp;
      const int tap = g / CHUNKS, cc = g % CHUNKS;
      const int toff = SGN * (tap_dy(tap) * L + tap_dx(tap)) * INSTR + cc * 8;
      bf16x8 xa[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const bool in_img = tap < 9 && ((valid[u] >> (MIRROR ? 8 - tap : tap)) & 1u);
        xa[u] = lds8(in_img ? in + q[u] * INSTR + toff : zslot);
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        acc[u][0] = mfma(w0[st], xa[u], acc[u][0]);
        acc[u][1] = mfma(w1[st], xa[u], acc[u][1]);
      }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (q[u] >= npix) continue;
      bf16x8 o;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (MIRROR) {
          o[i] = (bf16)((float)m0[u][i] > 0.0f ? acc[u][0][i] : 0.0f);
          o[4 + i] = (bf16)((float)m1[u][i] > 0.0f ? acc[u][1][i] : 0.0f);
        } else {
          o[i] = (bf16)fmaxf(acc[u][0][i] + bias0[i], 0.0f);
          o[4 + i] = (bf16)fmaxf(acc[u][1][i] + bias1[i], 0.0f);
        }
      }
      const uint4 ov = __builtin_bit_cast(uint4, o);
      if (TO_LDS) {
        *reinterpret_cast<uint2*>(out + q[u] * ASTR + 4 * grp) = make_uint2(ov.x, ov.y);
        *reinterpret_cast<uint2*>(out + q[u] * ASTR + 16 + 4 * grp) = make_uint2(ov.z, ov.w);
      }
      if (q[u] < nglob) {
        bf16* go = gout + (int64_t)q[u] * CH + 4 * grp;
        *reinterpret_cast<uint2*>(go) = make_uint2(ov.x, ov.y);
        *reinterpret_cast<uint2*>(go + 16) = make_uint2(ov.z, ov.w);
      }
    }
  }
}

// q / d for q < 2^16 with inv = 2^32 / d + 1 (d >= 2).
__host__ __device__ inline uint32_t inverse(uint32_t d) { return 0xFFFFFFFFu / d + 1u; }
__device__ __forceinline__ int quotient(int q, uint32_t inv) {
  return (int)__umulhi((uint32_t)q, inv);
}

// taps[q], bit t: pixel q's tap t lies inside the image.
__device__ __forceinline__ void tap_masks(int L, int npix, uint32_t inv_LL, uint32_t inv_L,
                                          uint16_t* taps) {
  for (int q = threadIdx.x; q < npix; q += FWD_THREADS) {
    const int r = q - quotient(q, inv_LL) * L * L;
    const int y = quotient(r, inv_L), x = r - y * L;
    const uint32_t cols = (x > 0 ? 1u : 0u) | 2u | (x < L - 1 ? 4u : 0u);
    taps[q] = (uint16_t)((y > 0 ? cols : 0u) | cols << 3 | (y < L - 1 ? cols << 6 : 0u));
  }
}

// Two [32][288] weight arrays into LDS rows of W23STR.
__device__ __forceinline__ void stage_weights(bf16* d0, const bf16* __restrict__ g0, bf16* d1,
                                              const bf16* __restrict__ g1) {
  for (int i = threadIdx.x; i < 32 * 36; i += FWD_THREADS) {
    const int r = i / 36, c = i % 36;
    *reinterpret_cast<uint4*>(d0 + r * W23STR + c * 8) =
        *reinterpret_cast<const uint4*>(g0 + r * 288 + c * 8);
    *reinterpret_cast<uint4*>(d1 + r * W23STR + c * 8) =
        *reinterpret_cast<const uint4*>(g1 + r * 288 + c * 8);
  }
}

// x0[pixel][8]: 0 lit star (i, j) at (i, j), 1 lit plaquette (i, j) at (i, j),
// 2 the sample's p, 3..7 zero.  acts: x0, a1, a2, a3 of the whole batch
// (STORE only).
struct CnnActs {
  bf16 *x0, *a1, *a2, *a3;
};

template <bool STORE>
__global__ void __launch_bounds__(FWD_THREADS) forward_kernel(
    int L, int S, int64_t B, const uint8_t* __restrict__ syn, const float* __restrict__ p,
    const bf16* __restrict__ wb1, const bf16* __restrict__ wb2, const bf16* __restrict__ wb3,
    const bf16* __restrict__ whb, const float* __restrict__ b1, const float* __restrict__ b2,
    const float* __restrict__ b3, const float* __restrict__ bh, float* __restrict__ logits,
    int64_t n_groups, CnnActs acts) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int LL = L * L, npix = S * LL, nst = 2 * L * (L - 1), ns = L * (L - 1);
  bf16* w1s = reinterpret_cast<bf16*>(smem);
  bf16* w2s = w1s + 32 * W1STR;
  bf16* w3s = w2s + 32 * W23STR;
  float* part = reinterpret_cast<float*>(w3s + 32 * W23STR);     // [waves][16][16]
  float* bias = part + FWD_WAVES * 256;                          // [3][32]
  bf16* zslot = reinterpret_cast<bf16*>(bias + 3 * CH);
  bf16* bufA = zslot + 8;
  bf16* bufB = bufA + npix * ASTR;
  uint16_t* taps = reinterpret_cast<uint16_t*>(bufB + npix * ASTR);
  const uint32_t inv_LL = inverse(LL), inv_L = inverse(L);
  const int tid = threadIdx.x;

  for (int i = tid; i < 32 * 12; i += FWD_THREADS) {
    const int r = i / 12, c = i % 12;
    *reinterpret_cast<uint4*>(w1s + r * W1STR + c * 8) =
        *reinterpret_cast<const uint4*>(wb1 + r * 96 + c * 8);
  }
  stage_weights(w2s, wb2, w3s, wb3);
  if (tid < CH) {
    bias[tid] = b1[tid];
    bias[CH + tid] = b2[tid];
    bias[2 * CH + tid] = b3[tid];
  }
  if (tid < 8) zslot[tid] = (bf16)0.0f;
  tap_masks(L, npix, inv_LL, inv_L, taps);
  // persistent: the weights stay in LDS while the workgroup walks its groups
  // of S samples (the barriers between the stages already order every
  // buffer's reuse from one group to the next)
  for (int64_t grp = blockIdx.x; grp < n_groups; grp += gridDim.x) {
  const int64_t s0 = grp * S;
  const int nsm = (int)min((int64_t)S, B - s0);
  const int64_t pix0 = s0 * LL;
  const int nglob = STORE ? nsm * LL : 0;
  // input planes, 8 channels per pixel
  for (int q = tid; q < npix; q += FWD_THREADS) {
    const int sm = quotient(q, inv_LL), r = q - sm * LL, y = quotient(r, inv_L), x = r - y * L;
    bf16x8 v = zero8();
    if (sm < nsm) {
      const uint8_t* sy = syn + (s0 + sm) * nst;
      v[0] = (bf16)((y < L - 1 && sy[y * L + x]) ? 1.0f : 0.0f);
      v[1] = (bf16)((x < L - 1 && sy[ns + y * (L - 1) + x]) ? 1.0f : 0.0f);
      v[2] = (bf16)p[s0 + sm];
    }
    *reinterpret_cast<uint4*>(bufA + q * 8) = __builtin_bit_cast(uint4, v);
    if (STORE && sm < nsm)
      *reinterpret_cast<uint4*>(acts.x0 + (pix0 + q) * 8) = __builtin_bit_cast(uint4, v);
  }
  __syncthreads();
  conv_lds<8, W1STR, 8, false, true>(L, npix, bufA, w1s, bias, taps, nullptr, bufB,
                               acts.a1 + pix0 * CH, nglob, zslot);
  __syncthreads();
  conv_lds<32, W23STR, ASTR, false, true>(L, npix, bufB, w2s, bias + CH, taps, nullptr, bufA,
                                    acts.a2 + pix0 * CH, nglob, zslot);
  __syncthreads();
  conv_lds<32, W23STR, ASTR, false, true>(L, npix, bufA, w3s, bias + 2 * CH, taps, nullptr, bufB,
                                    acts.a3 + pix0 * CH, nglob, zslot);
  __syncthreads();

  // head: wave j runs chain j over pixel steps j, j+8, ...
  {
    const int lane = tid & 63, wave = tid >> 6, grp = lane >> 4, n = lane & 15;
    const int64_t kh = (int64_t)LL * CH;
    f32x4 acc = {0, 0, 0, 0};
    // 24 of this chain's steps per trip (all of them up to L = 13): their
    // weight loads (from L2) are in flight before the first product; rows 7..15 of the padded head
    // weights are zero and not read
    for (int st0 = wave; st0 < LL; st0 += HEAD_TRIP * FWD_WAVES) {
      bf16x8 bq[HEAD_TRIP];
#pragma unroll
      for (int j = 0; j < HEAD_TRIP; ++j) {
        const int st = st0 + j * FWD_WAVES;
        bq[j] = (st < LL && n < 7) ? load8(whb + (int64_t)n * kh + st * 32 + 8 * grp) : zero8();
      }
#pragma unroll
      for (int j = 0; j < HEAD_TRIP; ++j) {
        const int st = st0 + j * FWD_WAVES;
        if (st < LL) {
          const bf16x8 a = n < nsm ? lds8(bufB + (n * LL + st) * ASTR + 8 * grp) : zero8();
          acc = mfma(a, bq[j], acc);
        }
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) part[wave * 256 + (4 * grp + i) * 16 + n] = acc[i];
  }
  __syncthreads();
  if (tid < 16 * 8) {
    const int row = tid >> 3, o = tid & 7;
    if (row < nsm && o < 7) {
      float t = part[row * 16 + o];
      for (int j = 1; j < FWD_WAVES; ++j) t = t + part[j * 256 + row * 16 + o];
      logits[(s0 + row) * 8 + o] = t + bh[o];
    }
  }
  }
}

// ---- backward --------------------------------------------------------------
// Loss and dL/dlogits of one sample (soft cross-entropy on the 4 class logits,
// weighted cross-entropy on the 3 budget logits), averaged over the batch.
__device__ __forceinline__ float sample_loss(const float* __restrict__ z,
                                             const float* __restrict__ tgt, int budget, float wb,
                                             float B, float dz[8]) {
  float m = fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3]));
  float e[4], se = 0.0f;
  for (int k = 0; k < 4; ++k) { e[k] = expf(z[k] - m); se += e[k]; }
  float lc = 0.0f;
  for (int k = 0; k < 4; ++k) {
    const float pk = e[k] / se;
    lc -= tgt[k] * ((z[k] - m) - logf(se));
    dz[k] = (pk - tgt[k]) / B;
  }
  const float mb = fmaxf(fmaxf(z[4], z[5]), z[6]);
  float eb[3], sb = 0.0f;
  for (int k = 0; k < 3; ++k) { eb[k] = expf(z[4 + k] - mb); sb += eb[k]; }
  const int y = min(max(budget, 0), 2);
  const float zy = y == 0 ? z[4] : (y == 1 ? z[5] : z[6]);
  const float lb = -((zy - mb) - logf(sb));
  for (int k = 0; k < 3; ++k) dz[4 + k] = wb * (eb[k] / sb - (k == y ? 1.0f : 0.0f)) / B;
  dz[7] = 0.0f;
  return lc + wb * lb;
}

// The data gradients of S samples per workgroup: loss and dz, then
//   dp3[b][f] = (sum_o dz[b][o] whb[o][f]) * (a3[b][f] > 0), rounded to bf16,
//   dp2 = conv3's data gradient where a2 > 0, dp1 = conv2's where a1 > 0,
// each kept in LDS for the next and written out for the weight gradients.
// Like the forward kernel it holds a sample's whole chain because a launch
// per stage is all latency: loss, head and the two convolutions took
// 3.5 + 8.8 + 2 x 13 us for 512 samples of L = 13; this kernel takes 16.5.
constexpr int BWD_WEIGHT_BYTES = 2 * 32 * W23STR * 2;
constexpr int BWD_SMALL_BYTES = 16 * 8 * 4 + 16;             // dz and the zero slot

__global__ void __launch_bounds__(FWD_THREADS) backward_kernel(
    int L, int S, int64_t B, const float* __restrict__ logits, const float* __restrict__ tgt,
    const int32_t* __restrict__ budget, float wb, const bf16* __restrict__ wt2,
    const bf16* __restrict__ wt3, const bf16* __restrict__ whb, const bf16* __restrict__ a1,
    const bf16* __restrict__ a2, const bf16* __restrict__ a3, float* __restrict__ dz,
    float* __restrict__ loss, bf16* __restrict__ dp1, bf16* __restrict__ dp2,
    bf16* __restrict__ dp3, int64_t n_groups) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int LL = L * L, npix = S * LL;
  const int64_t kh = (int64_t)LL * CH;
  bf16* w3s = reinterpret_cast<bf16*>(smem);
  bf16* w2s = w3s + 32 * W23STR;
  float* dzs = reinterpret_cast<float*>(w2s + 32 * W23STR);      // [16][8]
  bf16* zslot = reinterpret_cast<bf16*>(dzs + 16 * 8);
  bf16* bufA = zslot + 8;
  bf16* bufB = bufA + npix * ASTR;
  uint16_t* taps = reinterpret_cast<uint16_t*>(bufB + npix * ASTR);
  const uint32_t inv_LL = inverse(LL);
  const int tid = threadIdx.x;
  stage_weights(w3s, wt3, w2s, wt2);
  if (tid < 8) zslot[tid] = (bf16)0.0f;
  tap_masks(L, npix, inv_LL, inverse(L), taps);
  for (int64_t grp = blockIdx.x; grp < n_groups; grp += gridDim.x) {
    const int64_t s0 = grp * S;
    const int nsm = (int)min((int64_t)S, B - s0);
    const int64_t pix0 = s0 * LL;
    const int nglob = nsm * LL;
    if (tid < nsm) {
      const int64_t b = s0 + tid;
      float d[8];
      loss[b] = sample_loss(logits + b * 8, tgt + b * 4, budget[b], wb, (float)B, d);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        dz[b * 8 + k] = d[k];
        dzs[tid * 8 + k] = d[k];
      }
    }
    __syncthreads();
    // three chunks of 8 features per thread at a time, their 24 loads in flight together
    for (int i0 = tid; i0 < nglob * 4; i0 += 3 * FWD_THREADS) {
      bf16x8 av[3], wv[3][7];
#pragma unroll
      for (int u = 0; u < 3; ++u) {
        const int i = min(i0 + u * FWD_THREADS, nglob * 4 - 1);
        const int q = i >> 2, c = (i & 3) * 8, r = q - quotient(q, inv_LL) * LL;
        av[u] = load8(a3 + (pix0 + q) * CH + c);
#pragma unroll
        for (int o = 0; o < 7; ++o) wv[u][o] = load8(whb + o * kh + r * CH + c);
      }
#pragma unroll
      for (int u = 0; u < 3; ++u) {
        const int i = i0 + u * FWD_THREADS;
        if (i < nglob * 4) {
          const int q = i >> 2, c = (i & 3) * 8;
          const float* d = dzs + quotient(q, inv_LL) * 8;
          float s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
          for (int o = 0; o < 7; ++o)
#pragma unroll
            for (int j = 0; j < 8; ++j) s[j] += d[o] * (float)wv[u][o][j];
          bf16x8 v;
#pragma unroll
          for (int j = 0; j < 8; ++j) v[j] = (bf16)((float)av[u][j] > 0.0f ? s[j] : 0.0f);
          const uint4 ov = __builtin_bit_cast(uint4, v);
          *reinterpret_cast<uint4*>(bufA + q * ASTR + c) = ov;
          *reinterpret_cast<uint4*>(dp3 + (pix0 + q) * CH + c) = ov;
        }
      }
    }
    __syncthreads();
    conv_lds<32, W23STR, ASTR, true, true>(L, nglob, bufA, w3s, nullptr, taps, a2 + pix0 * CH,
                                           bufB, dp2 + pix0 * CH, nglob, zslot);
    __syncthreads();
    conv_lds<32, W23STR, ASTR, true, false>(L, nglob, bufB, w2s, nullptr, taps, a1 + pix0 * CH,
                                            nullptr, dp1 + pix0 * CH, nglob, zslot);
  }
}

// ---- weight gradients ------------------------------------------------------
// grad W[co][tap][ci] = sum_p dpre[p][co] * in[p + tap][ci]: the contraction
// runs over pixels, which is the outer index of both arrays.  A sample is
// copied to LDS as it lies (16-byte loads, pixel-major), each image row
// followed by one zero pixel and the image framed by zero rows, so a tap is a
// constant offset of dy (L + 1) + dx positions and needs no bounds test.
// ds_read_b64_tr_b16 turns 4 pixels x 16 channels into MFMA operands on the
// way out, for any offset.  Channel-major staging pays a transposing store per
// element and, for the taps' odd offsets, eight 2-byte reads per operand: 512
// samples of L = 13 took 30 us for each of two layers, 13 for the planes and 20
// for the head's sums; all of them in this launch take 13.2, bound by the
// latency of its samples' loads and of the partial sums' stores.
// v_mfma_f32_32x32x16_bf16, D[co][ci]: lane l holds A[l%32][8(l/32)..+7],
// B[8(l/32)..+7][l%32] and D[8(i/4) + 4(l/32) + i%4][l%32], i = 0..15.
//
// A workgroup of three waves walks G samples: wave w takes the taps of row
// dy = w - 1 (32 input channels) or taps 4w .. 4w + 3 (the planes: 8 channels
// a tap, 4 taps to a tile; the columns of "tap" 9 read ones and give the bias
// gradient).  Its row of partial sums lies in the gradients' order,
//   [W1 864][b1 32][W2 9216][b2 32][W3 9216][b3 32],
// each part written by its layer's workgroup.  Adding the tiles of several
// samples in LDS first (two or four samples at once per workgroup) measured
// 16.6 and 19.2 us.
constexpr int WG_THREADS = 192;
constexpr int N_W1 = CH * 27, N_W23 = CH * 288;
constexpr int ROW_FLOATS = N_W1 + 2 * N_W23 + 3 * CH;

struct WgradGeom {
  int PW, KP, MARGIN, lds_bytes;
};
__host__ __device__ inline WgradGeom wgrad_geom(int L) {
  WgradGeom g;
  g.PW = L + 1;
  g.KP = (L * g.PW + 15) / 16 * 16;                // positions, a multiple of the MFMA k
  g.MARGIN = L + 2;                                // positions before and after: the widest tap
  g.lds_bytes = (g.KP + g.KP + 2 * g.MARGIN) * CH * 2;
  return g;
}

__device__ __forceinline__ bf16x4 tr_read(const bf16* p) {
  typedef bf16x4 __attribute__((address_space(3))) * lds4;
  return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds4)p);
}
// k rows 0..7 of a column: two transposed reads, four positions apart
__device__ __forceinline__ bf16x8 tr_operand(const bf16* p, int four) {
  const bf16x4 lo = tr_read(p), hi = tr_read(p + four);
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

// 16-byte chunks i0, i0 + 192, .. (four per thread) of one sample's two
// arrays: loaded together, and for the next sample while this one is
// multiplied.  inp: the LDS position of pixel (0, 0) of the input.
template <int CIN>
struct SampleChunks {
  uint4 d0, d1, d2, d3, v0, v1, v2, v3;
  __device__ __forceinline__ void load(const bf16* __restrict__ dpre, const bf16* __restrict__ in,
                                       int64_t pix0, int LL, int i0) {
    const uint4* d = reinterpret_cast<const uint4*>(dpre + pix0 * CH);
    const uint4* v = reinterpret_cast<const uint4*>(in + pix0 * CIN);
    const int last = LL * 4 - 1;
    const int a = min(i0, last), b = min(a + WG_THREADS, last), c = min(b + WG_THREADS, last),
              e = min(c + WG_THREADS, last);
    constexpr int SH = CIN == 32 ? 0 : 2;
    d0 = d[a]; d1 = d[b]; d2 = d[c]; d3 = d[e];
    v0 = v[a >> SH]; v1 = v[b >> SH]; v2 = v[c >> SH]; v3 = v[e >> SH];
  }
  __device__ __forceinline__ void put(bf16* dT, bf16* inp, int LL, uint32_t inv_L, int i, uint4 d,
                                      uint4 v) const {
    if (i < LL * 4) {
      const int r = i >> 2, c = (i & 3) * 8;
      const int q = r + quotient(r, inv_L);                  // y (L + 1) + x
      *reinterpret_cast<uint4*>(dT + q * CH + c) = d;
      if (CIN == 32) *reinterpret_cast<uint4*>(inp + q * CH + c) = v;
      else if (c == 0) *reinterpret_cast<uint4*>(inp + q * 8) = v;
    }
  }
  __device__ __forceinline__ void stage(bf16* dT, bf16* inp, int LL, uint32_t inv_L,
                                        int i0) const {
    put(dT, inp, LL, inv_L, i0, d0, v0);
    put(dT, inp, LL, inv_L, i0 + WG_THREADS, d1, v1);
    put(dT, inp, LL, inv_L, i0 + 2 * WG_THREADS, d2, v2);
    put(dT, inp, LL, inv_L, i0 + 3 * WG_THREADS, d3, v3);
  }
};

// The operands of one k step: 16 positions from k on.
template <int CIN>
struct Operands {
  bf16x8 a, b[CIN == 32 ? 3 : 1];
  __device__ __forceinline__ void read(const bf16* arow, const bf16* brow, int bstep, int k) {
    a = tr_operand(arow + k * CH, 4 * CH);
    if (CIN == 32) {
#pragma unroll
      for (int t = 0; t < 3; ++t) b[t] = tr_operand(brow + (k + t - 1) * CH, 4 * CH);
    } else {
      b[0] = tr_operand(brow + k * bstep, 4 * bstep);
    }
  }
};

template <int CIN>
__device__ __forceinline__ void wgrad_body(int L, int64_t B, int G, int64_t row,
                                           const bf16* __restrict__ dpre,
                                           const bf16* __restrict__ in,
                                           float* __restrict__ out, unsigned char* smem,
                                           const bf16* ones) {
  constexpr int TAPS = CIN == 32 ? 3 : 1;          // tiles per wave
  constexpr int NT = CIN == 32 ? 4 : 1;            // and wave 1's bias tile
  const WgradGeom gm = wgrad_geom(L);
  const int st = threadIdx.x, lane = st & 63, w = st >> 6;
  bf16* dT = reinterpret_cast<bf16*>(smem);                 // [KP][32]
  bf16* iT = dT + gm.KP * CH;                               // [KP + 2 MARGIN][CIN]

  const int k0 = 8 * (lane >> 5) + ((lane & 15) >> 2);      // this lane's row of a k step
  const int col = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);  // and its four columns
  const bf16* arow = dT + k0 * CH + col;
  const bf16* brow;
  int bstep = CIN;
  if (CIN == 32) {
    brow = iT + (gm.MARGIN + k0 + (w - 1) * gm.PW) * CIN + col;
  } else {
    const int tap = 4 * w + col / 8;
    if (tap < 9) {
      brow = iT + (gm.MARGIN + k0 + tap_dy(tap) * gm.PW + tap_dx(tap)) * CIN + col % 8;
    } else {
      brow = ones;
      bstep = 0;
    }
  }
  const int LL = L * L;
  const uint32_t inv_L = inverse(L);
  f32x16 acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[t][i] = 0.0f;
  bf16x8 one8;
#pragma unroll
  for (int j = 0; j < 8; ++j) one8[j] = (bf16)1.0f;

  SampleChunks<CIN> ch;
  const int64_t first = row * G;
  ch.load(dpre, in, first * LL, LL, st);
  // the frame and the row ends stay zero for every sample
  for (int i = st; i < gm.lds_bytes / 16; i += WG_THREADS)
    reinterpret_cast<uint4*>(smem)[i] = make_uint4(0, 0, 0, 0);
  const int n = (int)min((int64_t)G, B - first);
  for (int g = 0; g < n; ++g) {
    const int64_t smp = first + g;
    __syncthreads();
    ch.stage(dT, iT + gm.MARGIN * CIN, LL, inv_L, st);
    for (int i0 = st + 4 * WG_THREADS; i0 < LL * 4; i0 += 4 * WG_THREADS) {
      ch.load(dpre, in, smp * LL, LL, i0);
      ch.stage(dT, iT + gm.MARGIN * CIN, LL, inv_L, i0);
    }
    __syncthreads();
    if (g + 1 < n) ch.load(dpre, in, (smp + 1) * LL, LL, st);
    // the operands of a k step are read while the step before is multiplied
    Operands<CIN> cur;
    cur.read(arow, brow, bstep, 0);
    for (int k = 0; k < gm.KP; k += 16) {
      Operands<CIN> nxt;
      nxt.read(arow, brow, bstep, min(k + 16, gm.KP - 16));
#pragma unroll
      for (int t = 0; t < TAPS; ++t) acc[t] = mfma32(cur.a, cur.b[t], acc[t]);
      if (CIN == 32 && w == 1) acc[NT - 1] = mfma32(cur.a, one8, acc[NT - 1]);
      cur = nxt;
    }
  }
  const int c = lane & 31;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int co = 8 * (i / 4) + 4 * (lane >> 5) + i % 4;
    if (CIN == 32) {
#pragma unroll
      for (int t = 0; t < 3; ++t) out[co * 288 + (3 * w + t) * 32 + c] = acc[t][i];
      if (w == 1 && c == 0) out[N_W23 + co] = acc[NT - 1][i];
    } else {
      const int tap = 4 * w + c / 8, ci = c % 8;
      if (tap < 9 && ci < 3) out[co * 27 + tap * 3 + ci] = acc[0][i];
      if (tap == 9 && ci == 0) out[N_W1 + co] = acc[0][i];
    }
  }
}

// grad Wh[o][f] = sum_b dz[b][o] a3[b][f]: the batch is cut into HEAD_SEGS
// contiguous segments, each summed in batch order into hpart[seg][o][f].
constexpr int HEAD_SEGS = 16;

__device__ __forceinline__ void head_grad_body(int64_t kh, int64_t B, int64_t block,
                                               const float* __restrict__ dz,
                                               const bf16* __restrict__ a3,
                                               float* __restrict__ hpart) {
  const int64_t blocks_f = (kh / 2 + blockDim.x - 1) / blockDim.x;
  const int seg = (int)(block / blocks_f);
  const int64_t f = 2 * ((block - seg * blocks_f) * blockDim.x + threadIdx.x);
  if (f >= kh) return;
  const int64_t per = (B + HEAD_SEGS - 1) / HEAD_SEGS;
  const int64_t b0 = min(seg * per, B), b1 = min(b0 + per, B);
  float s0[7] = {0, 0, 0, 0, 0, 0, 0}, s1[7] = {0, 0, 0, 0, 0, 0, 0};
  auto add = [&](int64_t b, uint32_t v) {
    const float lo = __uint_as_float(v << 16), hi = __uint_as_float(v & 0xFFFF0000u);
#pragma unroll
    for (int o = 0; o < 7; ++o) {
      s0[o] += dz[b * 8 + o] * lo;
      s1[o] += dz[b * 8 + o] * hi;
    }
  };
  int64_t b = b0;
  for (; b + 8 <= b1; b += 8) {
    uint32_t v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = *reinterpret_cast<const uint32_t*>(a3 + (b + j) * kh + f);
#pragma unroll
    for (int j = 0; j < 8; ++j) add(b + j, v[j]);
  }
  for (; b < b1; ++b) add(b, *reinterpret_cast<const uint32_t*>(a3 + b * kh + f));
#pragma unroll
  for (int o = 0; o < 7; ++o)
    *reinterpret_cast<float2*>(hpart + ((int64_t)seg * 7 + o) * kh + f) = make_float2(s0[o], s1[o]);
}

// Workgroups [0, rows): conv3, [rows, 2 rows): conv2, [2 rows, 3 rows): conv1,
// the rest the head.
__global__ void __launch_bounds__(WG_THREADS) weight_grad_kernel(
    int L, int64_t B, int G, int64_t rows, const bf16* __restrict__ x0,
    const bf16* __restrict__ a1, const bf16* __restrict__ a2, const bf16* __restrict__ a3,
    const bf16* __restrict__ dp1, const bf16* __restrict__ dp2, const bf16* __restrict__ dp3,
    const float* __restrict__ dz, float* __restrict__ part, float* __restrict__ hpart) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ __align__(16) bf16 ones[8];
  if (threadIdx.x < 8) ones[threadIdx.x] = (bf16)1.0f;     // read after the first barrier
  const int64_t blk = blockIdx.x;
  if (blk >= 3 * rows) {
    head_grad_body((int64_t)L * L * CH, B, blk - 3 * rows, dz, a3, hpart);
    return;
  }
  const int layer = (int)(blk / rows);
  const int64_t row = blk - layer * rows;
  float* out = part + row * ROW_FLOATS;
  if (layer == 0)
    wgrad_body<32>(L, B, G, row, dp3, a2, out + N_W1 + CH + N_W23 + CH, smem, ones);
  else if (layer == 1)
    wgrad_body<32>(L, B, G, row, dp2, a1, out + N_W1 + CH, smem, ones);
  else
    wgrad_body<8>(L, B, G, row, dp1, x0, out, smem, ones);
}

// Samples per weight-gradient workgroup: 128 rows of partial sums at most,
// with three workgroups (one per layer) to each.  At 512 samples of L = 13,
// kernel and reduction: 96 rows 15.3 + 4.6 us, 128 rows 13.2 + 5.0, 192 rows
// 13.3 + 5.3, 256 rows 13.6 + 5.7.
inline int wgrad_group(int64_t B) {
  const int64_t target = 128;
  return (int)(B <= target ? 1 : (B + target - 1) / target);
}
inline int64_t wgrad_rows(int64_t B) {
  const int64_t G = wgrad_group(B);
  return (B + G - 1) / G;
}

// All gradients from the partial sums, in one launch: a workgroup takes 32
// outputs and 8 row segments; segment g adds rows g, g+8, ... in order, and
// the 8 segment sums are added in segment order.  Outputs: the convolutions
// (rows of part), the head's weights (HEAD_SEGS rows of hpart), its 7 biases
// (the B rows of dz).
constexpr int RED_OUT = 32, RED_SEG = 8;

__global__ void __launch_bounds__(RED_OUT * RED_SEG) grad_reduce_kernel(
    int64_t rows, int64_t kh, int64_t B, const float* __restrict__ part,
    const float* __restrict__ hpart, const float* __restrict__ dz, float* __restrict__ grads) {
  __shared__ float seg_sum[RED_SEG][RED_OUT];
  const int o = threadIdx.x % RED_OUT, g = threadIdx.x / RED_OUT;
  const int64_t i = (int64_t)blockIdx.x * RED_OUT + o;
  const int64_t n_head = 7 * kh, total = ROW_FLOATS + n_head + 7;
  const float* src = part + i;
  int64_t n = rows, stride = ROW_FLOATS;
  if (i >= ROW_FLOATS) { src = hpart + (i - ROW_FLOATS); n = HEAD_SEGS; stride = n_head; }
  if (i >= ROW_FLOATS + n_head) { src = dz + (i - ROW_FLOATS - n_head); n = B; stride = 8; }
  if (i >= total) n = 0;
  float acc = 0.0f;
  int64_t k = g;
  for (; k + 7 * RED_SEG < n; k += 8 * RED_SEG) {
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = src[(k + j * RED_SEG) * stride];
#pragma unroll
    for (int j = 0; j < 8; ++j) acc += v[j];
  }
  for (; k < n; k += RED_SEG) acc += src[k * stride];
  seg_sum[g][o] = acc;
  __syncthreads();
  if (g == 0 && i < total) {
    float t = seg_sum[0][o];
    for (int j = 1; j < RED_SEG; ++j) t += seg_sum[j][o];
    grads[i] = t;
  }
}

__global__ void adam_kernel(int64_t n, float* __restrict__ prm, const float* __restrict__ g,
                            float* __restrict__ m, float* __restrict__ v, float lr, float b1,
                            float b2, float eps, float c1, float c2) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float mm = b1 * m[i] + (1.0f - b1) * g[i];
  const float vv = b2 * v[i] + (1.0f - b2) * g[i] * g[i];
  m[i] = mm;
  v[i] = vv;
  prm[i] -= lr * (mm / c1) / (sqrtf(vv / c2) + eps);
}

// Gate: class = argmax of the class logits (ties to the lowest); budget
// probabilities q = softmax of the budget logits; conf = (q0, q0 + q1, c),
// the probabilities that 0 and that at most the short budget reach the
// full-budget decision, and c = the class softmax's largest entry.
// route = 0 if q0 >= thr, else 1 if q0 + q1 >= thr, else 2.  With
// class_route the class head is read relative to the start decision: when
// c >= thr the route is 0 and flip = the argmax class (the class to compose
// with the start decision), else flip = 0.
__global__ void gate_kernel(int64_t B, const float* __restrict__ logits, float thr,
                            int class_route, uint8_t* __restrict__ route,
                            uint8_t* __restrict__ cls, float* __restrict__ conf,
                            uint8_t* __restrict__ flip, const GapRoute gap) {
  const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  const float* z = logits + b * 8;
  int best = 0;
  for (int k = 1; k < 4; ++k)
    if (z[k] > z[best]) best = k;
  float ec = 0.0f;
  for (int k = 0; k < 4; ++k) ec += expf(z[k] - z[best]);
  const float cmax = 1.0f / ec;
  const float m = fmaxf(fmaxf(z[4], z[5]), z[6]);
  const float e0 = expf(z[4] - m), e1 = expf(z[5] - m), e2 = expf(z[6] - m);
  const float sum = (e0 + e1) + e2;
  const float q0 = e0 / sum, q01 = (e0 + e1) / sum;
  uint8_t r = (uint8_t)(q0 >= thr ? 0 : (q01 >= thr ? 1 : 2));
  uint8_t f = 0;
  if (class_route && cmax >= thr) {
    r = 0;
    f = (uint8_t)best;
  }
  if (gap.table && r != 0) {  // the start-weight gap route: the no-sweep decision
    const int t = gap.table[gap_bin(gap.p[b])];
    if (t != (int)MCMC_GAP_NEVER && start_weight_gap(gap.weights + 4 * b) >= t) r = 0;
  }
  route[b] = r;
  cls[b] = (uint8_t)best;
  if (flip) flip[b] = f;
  if (conf) {
    conf[3 * b] = q0;
    conf[3 * b + 1] = q01;
    conf[3 * b + 2] = cmax;
  }
}

// Escalation margin of syndrome i from its short run's per-chain sums
// (block [4][K][C] at i 4KC): replica r's key of class e is the decision key
// restricted to that replica, sum_k w_k S[e][k][r] (w = 4, 2, ..., 4, 1 as in
// the decision; 1 for K = 1).  m_e = mean over the C replicas, v_e = their
// sample variance; with b the decided class (least m, ties to the lowest)
// and s the runner-up, z = (m_s - m_b) / sqrt((v_b + v_s) / C) (+inf when
// the spread is zero and m_s > m_b, 0 when m_s = m_b).
// flag[i] = route[i] == 1 && z < thr.
__global__ void escalate_kernel(int64_t n, const uint8_t* __restrict__ route,
                                const int64_t* __restrict__ sum_n, int K, int C, double thr,
                                uint8_t* __restrict__ flag) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  if (route[i] != 1) {
    flag[i] = 0;
    return;
  }
  const int64_t* blk = sum_n + i * 4 * (int64_t)K * C;
  double mean[4], var[4];
  for (int e = 0; e < 4; ++e) {
    double s1 = 0.0;
    for (int r = 0; r < C; ++r) {
      int64_t key = 0;
      for (int k = 0; k < K; ++k) {
        const int64_t w = k + 1 == K ? 1 : ((k + 1) % 2 == 1 ? 4 : 2);
        key += w * blk[((int64_t)e * K + k) * C + r];
      }
      s1 += (double)key;
    }
    mean[e] = s1 / (double)C;
    double s2 = 0.0;
    for (int r = 0; r < C; ++r) {
      int64_t key = 0;
      for (int k = 0; k < K; ++k) {
        const int64_t w = k + 1 == K ? 1 : ((k + 1) % 2 == 1 ? 4 : 2);
        key += w * blk[((int64_t)e * K + k) * C + r];
      }
      const double d = (double)key - mean[e];
      s2 += d * d;
    }
    var[e] = s2 / (double)(C - 1);
  }
  int b = 0;
  for (int e = 1; e < 4; ++e)
    if (mean[e] < mean[b]) b = e;
  int s = b == 0 ? 1 : 0;
  for (int e = 0; e < 4; ++e)
    if (e != b && mean[e] < mean[s]) s = e;
  const double gap = mean[s] - mean[b];
  const double se = sqrt((var[b] + var[s]) / (double)C);
  bool esc;
  if (se > 0.0) esc = gap / se < thr;
  else esc = !(gap > 0.0);
  flag[i] = (uint8_t)esc;
}

__global__ void gather_kernel(int64_t n, int row, const int32_t* __restrict__ idx,
                              const uint8_t* __restrict__ src, uint8_t* __restrict__ dst) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n * row) return;
  const int64_t k = i / row;
  dst[i] = src[(int64_t)idx[k] * row + (i - k * row)];
}

__global__ void scatter_kernel(int64_t n, const int32_t* __restrict__ idx,
                               const uint8_t* __restrict__ src, uint8_t* __restrict__ dst) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[idx[i]] = src[i];
}

__global__ void pick_kernel(int64_t n, int nq, const int32_t* __restrict__ idx,
                            const uint8_t* __restrict__ cls, const uint8_t* __restrict__ reps,
                            uint8_t* __restrict__ corr) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n * nq) return;
  const int64_t k = i / nq;
  const int q = (int)(i - k * nq);
  const int64_t o = idx[k];
  corr[o * nq + q] = reps[(k * 4 + cls[o]) * nq + q];
}

unsigned blocks_for(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

}  // namespace

CnnOffsets cnn_offsets(int L) {
  CnnOffsets o{};
  const int64_t kh = (int64_t)L * L * CH;
  o.W1 = 0;
  o.b1 = o.W1 + CH * 9 * 3;
  o.W2 = o.b1 + CH;
  o.b2 = o.W2 + CH * 9 * CH;
  o.W3 = o.b2 + CH;
  o.b3 = o.W3 + CH * 9 * CH;
  o.Wh = o.b3 + CH;
  o.bh = o.Wh + 7 * kh;
  o.total = o.bh + 7;
  return o;
}

CnnWorkspace cnn_workspace(int L, int64_t B) {
  CnnWorkspace w{};
  const int64_t P = B * L * L, kh = (int64_t)L * L * CH;
  const int64_t rows = wgrad_rows(B);
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t at = off;
    off = (off + bytes + 255) / 256 * 256;
    return at;
  };
  w.x0 = take((size_t)P * 8 * 2);
  w.a1 = take((size_t)P * CH * 2);
  w.a2 = take((size_t)P * CH * 2);
  w.a3 = take((size_t)P * CH * 2);
  w.wb1 = take(32 * 96 * 2);
  w.wb2 = take(32 * 288 * 2);
  w.wb3 = take(32 * 288 * 2);
  w.wt2 = take(32 * 288 * 2);
  w.wt3 = take(32 * 288 * 2);
  w.whb = take((size_t)16 * kh * 2);
  w.dz = take((size_t)B * 8 * 4);
  w.dp3 = take((size_t)P * CH * 2);
  w.dp2 = take((size_t)P * CH * 2);
  w.dp1 = take((size_t)P * CH * 2);
  w.part = take((size_t)rows * ROW_FLOATS * 4);
  w.hpart = take((size_t)HEAD_SEGS * 7 * kh * 4);
  w.loss = take((size_t)B * 4);
  w.bytes = off;
  return w;
}

CnnWeights cnn_weights(int L) {
  CnnWeights w{};
  const int64_t kh = (int64_t)L * L * CH;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t at = off;
    off = (off + bytes + 255) / 256 * 256;
    return at;
  };
  w.wb1 = take(32 * 96 * 2);
  w.wb2 = take(32 * 288 * 2);
  w.wb3 = take(32 * 288 * 2);
  w.wt2 = take(32 * 288 * 2);
  w.wt3 = take(32 * 288 * 2);
  w.whb = take((size_t)16 * kh * 2);
  w.bytes = off;
  return w;
}

int cnn_infer_group(int L) {
  int dev = 0, maxlds = 0;
  (void)hipGetDevice(&dev);
  if (hipDeviceGetAttribute(&maxlds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) !=
      hipSuccess)
    return 0;
  const int per = L * L * FWD_PIXEL_BYTES;
  const int S = (maxlds - FWD_WEIGHT_BYTES - FWD_PART_BYTES) / per;
  return S < 1 ? 0 : (S > 16 ? 16 : S);
}

namespace {

// Workgroups of a kernel that walks groups of samples: as many as LDS lets
// the chip hold at once, four to a CU at most.
int64_t resident_groups(int64_t groups, size_t lds) {
  const int per_cu = std::max<int>(1, std::min<int>(4, (int)(163840 / lds)));
  return std::min<int64_t>(groups, (int64_t)device_cus() * per_cu);
}

// Samples per workgroup of a training pass: the batch over the CUs (the
// registers of the layers' weights leave room for one workgroup on each),
// up to what LDS holds.
int train_group(int L, int64_t B) {
  const int64_t cus = device_cus(), s = (B + cus - 1) / cus;
  return (int)std::max<int64_t>(1, std::min<int64_t>(s, cnn_infer_group(L)));
}

size_t forward_lds_bytes(int L, int S) {
  return (size_t)FWD_WEIGHT_BYTES + FWD_PART_BYTES + (size_t)S * L * L * FWD_PIXEL_BYTES;
}
size_t backward_lds_bytes(int L, int S) {
  return (size_t)BWD_WEIGHT_BYTES + BWD_SMALL_BYTES + (size_t)S * L * L * FWD_PIXEL_BYTES;
}

template <bool STORE>
hipError_t launch_forward(int L, int S, int64_t B, const float* prm, const uint8_t* syn,
                          const float* p, float* logits, bf16* wb1, bf16* wb2, bf16* wb3,
                          bf16* wt2, bf16* wt3, bf16* whb, const CnnActs& acts, hipStream_t s) {
  const CnnOffsets off = cnn_offsets(L);
  const int64_t kh = (int64_t)L * L * CH;
  // one thread per entry of the largest of the cast arrays
  const int64_t n_cast = 16 * kh > 32 * 288 ? 16 * kh : 32 * 288;
  hipLaunchKernelGGL(cast_kernel, dim3(blocks_for(n_cast, 256)), dim3(256), 0, s, L, prm, off, wb1,
                     wb2, wb3, wt2, wt3, whb);
  const size_t lds = forward_lds_bytes(L, S);
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&forward_kernel<STORE>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  const int64_t groups = (B + S - 1) / S;
  hipLaunchKernelGGL((forward_kernel<STORE>), dim3((unsigned)resident_groups(groups, lds)),
                     dim3(FWD_THREADS), lds, s, L, S, B, syn, p, wb1, wb2, wb3, whb, prm + off.b1,
                     prm + off.b2, prm + off.b3, prm + off.bh, logits, groups, acts);
  return hipGetLastError();
}

}  // namespace

hipError_t cnn_infer(int L, int64_t B, const float* prm, const uint8_t* syn, const float* p,
                     float* logits, char* ws, hipStream_t s) {
  const CnnWeights wl = cnn_weights(L);
  const int S = cnn_infer_group(L);
  if (S < 1) return hipErrorInvalidConfiguration;
  auto at = [&](size_t o) { return reinterpret_cast<bf16*>(ws + o); };
  return launch_forward<false>(L, S, B, prm, syn, p, logits, at(wl.wb1), at(wl.wb2), at(wl.wb3),
                               at(wl.wt2), at(wl.wt3), at(wl.whb), CnnActs{}, s);
}

#define WSP(T, name) reinterpret_cast<T*>(ws + wl.name)

hipError_t cnn_forward(int L, int64_t B, const float* prm, const uint8_t* syn, const float* p,
                       float* logits, char* ws, hipStream_t s) {
  const CnnWorkspace wl = cnn_workspace(L, B);
  if (cnn_infer_group(L) < 1) return hipErrorInvalidConfiguration;
  const CnnActs acts{WSP(bf16, x0), WSP(bf16, a1), WSP(bf16, a2), WSP(bf16, a3)};
  return launch_forward<true>(L, train_group(L, B), B, prm, syn, p, logits, WSP(bf16, wb1),
                              WSP(bf16, wb2), WSP(bf16, wb3), WSP(bf16, wt2), WSP(bf16, wt3),
                              WSP(bf16, whb), acts, s);
}

hipError_t cnn_backward(int L, int64_t B, const float* prm, const float* logits, const float* tgt,
                        const int32_t* budget, float wb, float* grads, float* loss, char* ws,
                        hipStream_t s) {
  (void)prm;
  const CnnWorkspace wl = cnn_workspace(L, B);
  if (cnn_infer_group(L) < 1) return hipErrorInvalidConfiguration;
  const int64_t kh = (int64_t)L * L * CH;
  const int S = train_group(L, B);
  const int64_t groups = (B + S - 1) / S;
  const size_t lds_b = backward_lds_bytes(L, S);
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&backward_kernel),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_b);
  hipLaunchKernelGGL(backward_kernel, dim3((unsigned)resident_groups(groups, lds_b)),
                     dim3(FWD_THREADS), lds_b, s, L, S, B, logits, tgt, budget, wb,
                     WSP(bf16, wt2), WSP(bf16, wt3), WSP(bf16, whb), WSP(bf16, a1), WSP(bf16, a2),
                     WSP(bf16, a3), WSP(float, dz), loss ? loss : WSP(float, loss), WSP(bf16, dp1),
                     WSP(bf16, dp2), WSP(bf16, dp3), groups);

  const int G = wgrad_group(B);
  const int64_t rows = wgrad_rows(B);
  const int64_t head = (int64_t)blocks_for(kh / 2, WG_THREADS) * HEAD_SEGS;
  const int lds_w = wgrad_geom(L).lds_bytes;
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&weight_grad_kernel),
                            hipFuncAttributeMaxDynamicSharedMemorySize, lds_w);
  hipLaunchKernelGGL(weight_grad_kernel, dim3((unsigned)(3 * rows + head)), dim3(WG_THREADS),
                     lds_w, s, L, B, G, rows, WSP(bf16, x0), WSP(bf16, a1), WSP(bf16, a2),
                     WSP(bf16, a3), WSP(bf16, dp1), WSP(bf16, dp2), WSP(bf16, dp3), WSP(float, dz),
                     WSP(float, part), WSP(float, hpart));
  hipLaunchKernelGGL(grad_reduce_kernel, dim3(blocks_for(ROW_FLOATS + 7 * kh + 7, RED_OUT)),
                     dim3(RED_OUT * RED_SEG), 0, s, rows, kh, B, WSP(float, part),
                     WSP(float, hpart), WSP(float, dz), grads);
  return hipGetLastError();
}

hipError_t cnn_adam(int64_t n, float* prm, const float* g, float* m, float* v, float lr, float b1,
                    float b2, float eps, float c1, float c2, hipStream_t s) {
  hipLaunchKernelGGL(adam_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, n, prm, g, m, v, lr,
                     b1, b2, eps, c1, c2);
  return hipGetLastError();
}

hipError_t cnn_gate(int64_t B, const float* logits, float thr, bool class_route, uint8_t* route,
                    uint8_t* cls, float* conf, uint8_t* flip, const GapRoute& gap,
                    hipStream_t s) {
  hipLaunchKernelGGL(gate_kernel, dim3(blocks_for(B, 256)), dim3(256), 0, s, B, logits, thr,
                     class_route ? 1 : 0, route, cls, conf, flip, gap);
  return hipGetLastError();
}

hipError_t cnn_escalate_flags(int64_t n, const uint8_t* route, const int64_t* sum_n, int K, int C,
                              double thr, uint8_t* flag, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(escalate_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, n, route, sum_n,
                     K, C, thr, flag);
  return hipGetLastError();
}

hipError_t cnn_gather(int64_t n, int row, const int32_t* idx, const uint8_t* src, uint8_t* dst,
                      hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(gather_kernel, dim3(blocks_for(n * row, 256)), dim3(256), 0, s, n, row, idx,
                     src, dst);
  return hipGetLastError();
}

hipError_t cnn_scatter(int64_t n, const int32_t* idx, const uint8_t* src, uint8_t* dst,
                       hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(scatter_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, n, idx, src, dst);
  return hipGetLastError();
}

hipError_t cnn_pick(int64_t n, int nq, const int32_t* idx, const uint8_t* cls,
                    const uint8_t* reps, uint8_t* corr, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(pick_kernel, dim3(blocks_for(n * nq, 256)), dim3(256), 0, s, n, nq, idx, cls,
                     reps, corr);
  return hipGetLastError();
}

}  // namespace mcmc
