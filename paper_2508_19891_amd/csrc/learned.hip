// Fitting the learned index (router training and leaf fits), all on the GPU.
//
//   learned_sample   kSamples evenly spaced (key, rank) pairs of the sorted
//                    keys -> inputs x = top 24 key bits / 2^24, targets rank/n.
//   learned_init     quantile initialisation of the ramps.
//   learned_train    one workgroup: Adam steps on the mean squared error over
//                    batches of 128 samples (forward and backward written out
//                    below), with w1, W2, w3 projected onto >= 0 after every
//                    step so that the router stays monotone.
//   learned_errors   every sample's squared error and their mean, before and
//   learned_loss     after the training.
//   learned_radix    tabulation of the trained router: the leaf at every
//   learned_xbounds  2^8-th input, and the first input X of every leaf (a
//                    binary search per leaf, valid because routing is
//                    monotone).
//   learned_keybounds first key index of every leaf.
//   learned_piece_offsets  pieces per leaf (ceil(size / kPiece)) and their
//                    exclusive scan (one workgroup).
//   learned_pieces   one wave per piece: first key, interpolation slope and
//                    the exact window of (lower bound - prediction) over every
//                    query key the piece can receive.
#include <hip/hip_runtime.h>

#include "common.h"
#include "internal.h"
#include "learned.h"

namespace sfc {
namespace {

constexpr int kBatch = 128;
constexpr int kTrainWaves = 8;
constexpr int kTrainThreads = kTrainWaves * kWave;

__device__ __forceinline__ float clip01(float v) { return fminf(fmaxf(v, 0.f), 1.f); }
__device__ __forceinline__ float inside01(float v) { return (v > 0.f && v < 1.f) ? 1.f : 0.f; }

// ---- one training step on the matrix cores -----------------------------------
//
// A step is three products over the batch of 128 samples (the second layer's
// forward, its transpose backward, and the weight gradient) and five column
// sums, 4 * 10^5 multiply-adds in a chain of 256 steps: one workgroup, bound
// by the length of a step's dependent chain.  The products run as
// v_mfma_f32_16x16x4_f32, which adds its four terms one after another, each
// a fused multiply-add rounded once (checked bit for bit against fmaf), so a
// chain of them is the plain loop over k, and the parameters are those that
// loop gives, bit for bit.
//
// Wave w holds samples 16 w .. 16 w + 15, sample l % 16 in lane l, and of each
// sample's 32 units those with index 4 s + l / 16 (s = 0..7).  The rows of a
// product are numbered so that its result (unit 4 (4 t + v) + l / 16 in
// register v of tile t) is the next product's operand as it stands: hidden
// values, output and back-propagated errors never leave the registers.  Only
// the weight gradient, whose sum runs over the samples, goes through LDS:
// waves 0..3 take one 16x16 tile of it each, waves 4..6 the column sums, and
// each lane updates (Adam) the parameters whose gradients it holds.
// 256 steps over 2^16 samples take 0.82 ms (0.94 with the lanes' four updates one
// after another, each behind branches); 26.1 ms with one sample per lane and every
// weight read from LDS for each multiply-add.  A step's 7600 cycles are 3600 of
// matrix instructions and 3300 of vector ones a SIMD, in phases that follow from
// each other.
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kWStride = 36;             // LDS row of 32 weights
constexpr int kQStride = 36;             // samples of equal b % 4, by b / 4
constexpr int kBStride = 4 * kQStride + 4;   // LDS row of 128 samples
constexpr int kOwned = 4;                // parameters a lane owns at most

// Rows of 128 samples in LDS, one per unit.
enum { kRowD2 = 0, kRowH1 = 32, kRowE3 = 64, kRowD1X = 96, kRowD1 = 128, kRowG = 160, kRows = 161 };

struct TrainLds {
  float w2[kHidden * kWStride];    // [i][unit_pos(j)]
  float w2t[kHidden * kWStride];   // [j][unit_pos(i)]
  float w1[kHidden], b1[kHidden], b2[kHidden], w3[kHidden];   // [unit_pos(unit)]
  float b3[4];
  float rows[kRows * kBStride];    // [row][sample_pos(b)]
};

// Units of equal index % 4 are neighbours, so that a lane's eight are two
// 16-byte loads; samples likewise.
__device__ __forceinline__ int unit_pos(int k) { return (k & 3) * 8 + (k >> 2); }
__device__ __forceinline__ int sample_pos(int b) { return (b & 3) * kQStride + (b >> 2); }

// Eight consecutive LDS words (16-byte aligned).
__device__ __forceinline__ void load8(const float* p, float v[8]) {
  const f32x4 a = *(const f32x4*)p, b = *(const f32x4*)(p + 4);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[i] = a[i];
    v[4 + i] = b[i];
  }
}

// Parameter r of the ones this lane owns (r < kOwned; -1: none): waves 0..3
// the second layer's weights (tile (w & 1, w >> 1) of the matrix, rows
// 4 (l / 16) + r, column l % 16), wave 4 its biases and the output weights,
// wave 5 the first layer's weights and biases, wave 6's first lane the output
// bias.
__device__ __forceinline__ int owned_param(int r) {
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  if (w < 4) {
    const int i = 16 * (w & 1) + 4 * (l >> 4) + r, j = 16 * (w >> 1) + (l & 15);
    return kOffW2 + i * kHidden + j;
  }
  if (r > 0) return -1;
  if (w == 4) return l < kHidden ? kOffB2 + l : kOffW3 + l - kHidden;
  if (w == 5) return l < kHidden ? kOffW1 + l : kOffB1 + l - kHidden;
  return w == 6 && l == 0 ? kOffB3 : -1;
}

// Puts parameter `at` into its places in LDS.
__device__ __forceinline__ void store_param(TrainLds& S, int at, float v) {
  if (at >= kOffW2 && at < kOffB2) {
    const int i = (at - kOffW2) / kHidden, j = (at - kOffW2) % kHidden;
    S.w2[i * kWStride + unit_pos(j)] = v;
    S.w2t[j * kWStride + unit_pos(i)] = v;
  } else if (at >= kOffB3) {
    S.b3[0] = v;
  } else if (at >= kOffW3) {
    S.w3[unit_pos(at - kOffW3)] = v;
  } else if (at >= kOffB2) {
    S.b2[unit_pos(at - kOffB2)] = v;
  } else if (at >= kOffB1) {
    S.b1[unit_pos(at - kOffB1)] = v;
  } else if (at >= 0) {
    S.w1[unit_pos(at)] = v;
  }
}

// Gradient of the mean squared error over samples 0..cnt - 1 of a batch for
// the parameters in S: G[r] is that of owned_param(r).  x, t: the sample of
// this lane, 16 w + l % 16 (zeros from cnt on).  Returns the sample's error
// y - t.  One barrier; the caller's next one ends the reads of S.  FULL: cnt is
// kBatch.
template <bool FULL>
__device__ __forceinline__ float batch_gradient(TrainLds& S, float x, float t, int count,
                                                float G[kOwned]) {
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63, c = l & 15, grp = l >> 4;
  const int cnt = FULL ? kBatch : count;
  const bool mine = FULL || 16 * w + c < cnt;
  // Forward.  Row r of tile t stands for unit 16 t + 4 (r % 4) + r / 4.
  const int row0 = 4 * (c & 3) + (c >> 2);
  float w1[8], b1[8], w3[8], a1[8], h1[8], a2[8], h2[8];
  load8(S.w1 + 8 * grp, w1);
  load8(S.b1 + 8 * grp, b1);
  f32x4 acc[2];
  acc[0] = *(const f32x4*)(S.b2 + 8 * grp);
  acc[1] = *(const f32x4*)(S.b2 + 8 * grp + 4);
  float m0[8], m1[8];
  load8(S.w2 + row0 * kWStride + 8 * grp, m0);
  load8(S.w2 + (row0 + 16) * kWStride + 8 * grp, m1);
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    a1[s] = __fmaf_rn(w1[s], x, b1[s]);
    h1[s] = clip01(a1[s]);
    acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(m0[s], h1[s], acc[0], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(m1[s], h1[s], acc[1], 0, 0, 0);
  }
  load8(S.w3 + 8 * grp, w3);
  load8(S.w2t + row0 * kWStride + 8 * grp, m0);
  load8(S.w2t + (row0 + 16) * kWStride + 8 * grp, m1);
  const float b3 = S.b3[0];
  f32x4 yv = {b3, b3, b3, b3};   // every row of this product is the output
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    a2[s] = acc[s >> 2][s & 3];
    h2[s] = clip01(a2[s]);
    yv = __builtin_amdgcn_mfma_f32_16x16x4f32(w3[s], h2[s], yv, 0, 0, 0);
  }
  const float err = yv[0] - t;
  const float g = mine ? 2.f * err / (float)cnt : 0.f;
  // Backward through the second layer.
  float* at = S.rows + grp * kBStride + sample_pos(16 * w + c);   // unit 4 s + grp: row 4 s + grp
  acc[0] = acc[1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const float d2 = mine ? g * w3[s] * inside01(a2[s]) : 0.f;
    acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(m0[s], d2, acc[0], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(m1[s], d2, acc[1], 0, 0, 0);
    at[(kRowD2 + 4 * s) * kBStride] = d2;
    at[(kRowH1 + 4 * s) * kBStride] = h1[s];
    at[(kRowE3 + 4 * s) * kBStride] = mine ? g * h2[s] : 0.f;
  }
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const float d1 = mine ? acc[s >> 2][s & 3] * inside01(a1[s]) : 0.f;
    at[(kRowD1X + 4 * s) * kBStride] = d1 * x;
    at[(kRowD1 + 4 * s) * kBStride] = d1;
  }
  if (grp == 0) at[kRowG * kBStride] = g;
  __syncthreads();

  if (w < 4) {
    // dW2[i][j] = sum over the samples, in order, of d2[i] h1[j].
    const float* pa = S.rows + (kRowD2 + 16 * (w & 1) + c) * kBStride + grp * kQStride;
    const float* pb = S.rows + (kRowH1 + 16 * (w >> 1) + c) * kBStride + grp * kQStride;
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < kBatch / 4; q += 4) {
      const f32x4 va = *(const f32x4*)(pa + q), vb = *(const f32x4*)(pb + q);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        sum = __builtin_amdgcn_mfma_f32_16x16x4f32(va[i], vb[i], sum, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < kOwned; ++r) G[r] = sum[r];
  } else if (w < 7) {
    // The row's sum over the samples, in order.
    const int row = w == 4 ? (l < kHidden ? kRowD2 + l : kRowE3 + l - kHidden)
                    : w == 5 ? (l < kHidden ? kRowD1X + l : kRowD1 + l - kHidden)
                             : kRowG;
    const float* p = S.rows + row * kBStride;
    float sum = 0.f;
#pragma unroll
    for (int q = 0; q < kBatch / 4; q += 4) {
      f32x4 v[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = *(const f32x4*)(p + k * kQStride + q);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int k = 0; k < 4; ++k) sum += v[k][i];
    }
    G[0] = sum;
  }
  return err;
}

__global__ __launch_bounds__(kTrainThreads) void learned_grad_kernel(const float* __restrict__ p_in,
                                                                     const float* __restrict__ xs,
                                                                     const float* __restrict__ ts,
                                                                     int cnt,
                                                                     float* __restrict__ g_out,
                                                                     float* __restrict__ loss_out) {
  __shared__ TrainLds S;
  __shared__ float s_red[kBatch];
  for (int i = threadIdx.x; i < kParams; i += kTrainThreads) store_param(S, i, p_in[i]);
  __syncthreads();
  const int b = 16 * (threadIdx.x >> 6) + (threadIdx.x & 15);
  const float x = b < cnt ? xs[b] : 0.f, t = b < cnt ? ts[b] : 0.f;
  float G[kOwned];
  const float err = batch_gradient<false>(S, x, t, cnt, G);
#pragma unroll
  for (int r = 0; r < kOwned; ++r) {
    const int at = owned_param(r);
    if (at >= 0) g_out[at] = G[r];
  }
  // Batch loss (fixed tree over LDS).
  if ((threadIdx.x & 63) < 16) s_red[b] = b < cnt ? err * err : 0.f;
  __syncthreads();
  for (int o = kBatch / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) s_red[threadIdx.x] += s_red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) loss_out[0] = s_red[0] / (float)(cnt > 0 ? cnt : 1);
}

__global__ __launch_bounds__(256) void learned_sample(const uint64_t* __restrict__ keys, uint64_t n,
                                                      uint32_t S, float* __restrict__ xs,
                                                      float* __restrict__ ts) {
  const uint32_t s = blockIdx.x * 256 + threadIdx.x;
  if (s >= S) return;
  const uint64_t i = (uint64_t)s * n / S;
  xs[s] = router_input(keys[i]);
  ts[s] = (float)((double)i / (double)n);
}

// Quantile initialisation: ramp j rises from quantile j/32 to (j+1)/32 of the
// sample inputs; identity second layer; output = mean of the ramps.
__global__ __launch_bounds__(256) void learned_init(const float* __restrict__ xs, uint32_t S,
                                                    float* __restrict__ P) {
  const int tid = threadIdx.x;
  for (int i = kOffW2 + tid; i < kParams; i += 256) {
    float v = 0.f;
    if (i < kOffB2) {
      const int e = i - kOffW2;
      v = (e / kHidden == e % kHidden) ? 1.f : 0.f;
    } else if (i >= kOffW3 && i < kOffB3) {
      v = 1.f / (float)kHidden;
    }
    P[i] = v;
  }
  if (tid < kHidden) {
    const float q0 = xs[(uint64_t)tid * S / kHidden];
    const uint64_t i1 = (uint64_t)(tid + 1) * S / kHidden;
    const float q1 = xs[i1 < S ? i1 : S - 1];
    const float span = fmaxf(q1 - q0, 0x1p-24f);
    P[kOffW1 + tid] = 1.f / span;
    P[kOffB1 + tid] = -q0 / span;
  }
}

// Squared error of the router at every sample.
__global__ __launch_bounds__(256) void learned_errors(const float* __restrict__ P,
                                                      const float* __restrict__ xs,
                                                      const float* __restrict__ ts, uint32_t S,
                                                      float* __restrict__ sq) {
  const uint32_t s = blockIdx.x * 256 + threadIdx.x;
  if (s >= S) return;
  const float d = router_output(P, xs[s]) - ts[s];
  sq[s] = d * d;
}

// Mean of the S squared errors (one workgroup): 256 strided sums, then a tree.
__global__ __launch_bounds__(256) void learned_loss(const float* __restrict__ sq, uint32_t S,
                                                    float* __restrict__ loss) {
  __shared__ float s_red[256];
  float acc = 0.f;
  // Many loads in flight per thread (a round of them is a round trip to memory),
  // added in order; positions past the end load the last one and add nothing.
  constexpr int kAtOnce = 64;
  for (uint32_t s0 = threadIdx.x; s0 < S; s0 += 256 * kAtOnce) {
    float v[kAtOnce];
#pragma unroll
    for (int k = 0; k < kAtOnce; ++k) v[k] = sq[s0 + 256 * k < S ? s0 + 256 * k : S - 1];
#pragma unroll
    for (int k = 0; k < kAtOnce; ++k)
      if (s0 + 256 * k < S) acc += v[k];
  }
  s_red[threadIdx.x] = acc;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) s_red[threadIdx.x] += s_red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) loss[0] = s_red[0] / (float)S;
}

// Adam over `steps` batches, in place on the parameters (one workgroup).
// Batch st: samples (odd multiplier) * (st * kBatch + b) mod S, a permutation
// of the samples within every pass over them.
__global__ __launch_bounds__(kTrainThreads) void learned_train(const float* __restrict__ xs,
                                                               const float* __restrict__ ts,
                                                               uint32_t S, uint32_t steps, float lr,
                                                               float* __restrict__ params) {
  __shared__ TrainLds L;
  const int b = 16 * (threadIdx.x >> 6) + (threadIdx.x & 15);
  float P[kOwned], Mo[kOwned], Vo[kOwned];
#pragma unroll
  for (int r = 0; r < kOwned; ++r) {
    const int at = owned_param(r);
    P[r] = at >= 0 ? params[at] : 0.f;
    Mo[r] = Vo[r] = 0.f;
    if (at >= 0) store_param(L, at, P[r]);
  }
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  float b1t = 1.f, b2t = 1.f;
  const uint32_t mask = S - 1;   // S is a power of two
  // A step's samples are loaded during the step before it.
  uint32_t s = (uint32_t)((uint64_t)b * 2654435761ull) & mask;
  float x = xs[s], t = ts[s];
  // Where the lane's parameters lie in LDS, and whether they stay nonnegative (the
  // second layer's weights twice, as its transpose holds them too).
  const int w = threadIdx.x >> 6, at0 = owned_param(0);
  // (As numbers of words: pointers would be followed as generic ones.)
  float* const lds = (float*)&L;
  int to[kOwned] = {}, tt[kOwned] = {};
  bool nonneg = false;
  if (w < 4) {
#pragma unroll
    for (int r = 0; r < kOwned; ++r) {
      const int e = owned_param(r) - kOffW2, i = e / kHidden, k = e % kHidden;
      to[r] = (int)(L.w2 - lds) + i * kWStride + unit_pos(k);
      tt[r] = (int)(L.w2t - lds) + k * kWStride + unit_pos(i);
    }
  } else if (at0 >= 0) {
    to[0] = at0 >= kOffB3   ? (int)(L.b3 - lds)
            : at0 >= kOffW3 ? (int)(L.w3 - lds) + unit_pos(at0 - kOffW3)
            : at0 >= kOffB2 ? (int)(L.b2 - lds) + unit_pos(at0 - kOffB2)
            : at0 >= kOffB1 ? (int)(L.b1 - lds) + unit_pos(at0 - kOffB1)
                            : (int)(L.w1 - lds) + unit_pos(at0);
    nonneg = at0 < kOffB1 || (at0 >= kOffW3 && at0 < kOffB3);
  }
  __syncthreads();
  for (uint32_t st = 0; st < steps; ++st) {
    s = (uint32_t)(((uint64_t)(st + 1) * kBatch + b) * 2654435761ull) & mask;
    const float nx = xs[s], nt = ts[s];
    float G[kOwned] = {0.f, 0.f, 0.f, 0.f};
    batch_gradient<true>(L, x, t, kBatch, G);
    b1t *= b1;
    b2t *= b2;
    const float c1 = 1.f - b1t, c2 = 1.f - b2t;
    auto adam = [&](int r) {
      const float gi = G[r];
      Mo[r] = b1 * Mo[r] + (1.f - b1) * gi;
      Vo[r] = b2 * Vo[r] + (1.f - b2) * gi * gi;
      const float mh = Mo[r] / c1, vh = Vo[r] / c2;
      return P[r] - lr * mh / (sqrtf(vh) + eps);
    };
    // (No branch between a lane's four: their chains of divisions run together.)
    if (w < 4) {
#pragma unroll
      for (int r = 0; r < kOwned; ++r) P[r] = fmaxf(adam(r), 0.f);
#pragma unroll
      for (int r = 0; r < kOwned; ++r) {
        lds[to[r]] = P[r];
        lds[tt[r]] = P[r];
      }
    } else if (at0 >= 0) {
      const float v = adam(0);
      P[0] = nonneg ? fmaxf(v, 0.f) : v;
      lds[to[0]] = P[0];
    }
    x = nx;
    t = nt;
    __syncthreads();
  }
#pragma unroll
  for (int r = 0; r < kOwned; ++r) {
    const int at = owned_param(r);
    if (at >= 0) params[at] = P[r];
  }
}

// rt[t] = the leaf of input t << 8 (t < 2^16), and of the last input.
__global__ __launch_bounds__(256) void learned_radix(const float* __restrict__ P,
                                                     uint32_t* __restrict__ rt) {
  const uint32_t t = blockIdx.x * 256 + threadIdx.x;
  if (t > kRouteSlots) return;
  const uint32_t X = t < kRouteSlots ? t << (kXBits - kRouteBits) : (1u << kXBits) - 1;
  rt[t] = router_leaf_x(P, X);
}

// xb[l] = the first X with leaf(X) >= l, 2^24 if none.  The table rt (every
// 2^8-th input's leaf) brackets it: routing is monotone, so the search of the
// table leaves at most eight evaluations of the network, a chain of 10^3
// multiply-adds each (all 24 steps by evaluation took 0.09 ms with the table,
// against 0.04 ms).  One wave per workgroup, so that the 65 waves spread over
// the CUs.
__global__ __launch_bounds__(64) void learned_xbounds(const float* __restrict__ P,
                                                      const uint32_t* __restrict__ rt,
                                                      uint32_t* __restrict__ xb) {
  constexpr int kStep = kXBits - kRouteBits;
  const uint32_t l = blockIdx.x * 64 + threadIdx.x;
  if (l > (uint32_t)kLeaves) return;
  if (l == 0 || l == (uint32_t)kLeaves) {
    xb[l] = l == 0 ? 0u : (1u << kXBits);
    return;
  }
  uint32_t t = 0, tl = kRouteSlots;   // first t with rt[t] >= l, kRouteSlots if none
  while (tl > 0) {
    const uint32_t h = tl >> 1;
    if (rt[t + h] < l) {
      t += h + 1;
      tl -= h + 1;
    } else {
      tl = h;
    }
  }
  // leaf((t - 1) << 8) < l <= leaf(t << 8): the first X lies past the former,
  // at most the latter.
  if (t == 0) {
    xb[l] = 0;
    return;
  }
  uint32_t lo = ((t - 1) << kStep) + 1, len = (1u << kStep) - 1;
  while (len > 0) {
    const uint32_t h = len >> 1;
    if (router_leaf_x(P, lo + h) < l) {
      lo += h + 1;
      len -= h + 1;
    } else {
      len = h;
    }
  }
  xb[l] = lo;
}

// lp[l].x = first index whose key routes to a leaf >= l: keys route by their
// top 24 bits, so that is the lower bound of xb[l] << 40 (lp[kLeaves].x = n).
__global__ __launch_bounds__(256) void learned_keybounds(const uint64_t* __restrict__ keys,
                                                         uint64_t n,
                                                         const uint32_t* __restrict__ xb,
                                                         uint2* __restrict__ lp) {
  const uint32_t l = blockIdx.x * 256 + threadIdx.x;
  if (l > (uint32_t)kLeaves) return;
  const uint32_t X = xb[l];
  lp[l].x = (l == (uint32_t)kLeaves || X >= (1u << kXBits))
                ? (uint32_t)n
                : (uint32_t)lower_bound_in(keys, 0, n, (uint64_t)X << (64 - kXBits));
}

// lp[l].y = first piece of leaf l (lp[kLeaves].y = number of pieces); one block.
__global__ __launch_bounds__(256) void learned_piece_offsets(uint2* __restrict__ lp) {
  constexpr int kPer = kLeaves / 256;
  __shared__ uint32_t s_w[4];
  const uint32_t tid = threadIdx.x;
  uint32_t c[kPer], sum = 0;
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const uint32_t l = tid * kPer + i;
    const uint32_t S = lp[l].x, E = lp[l + 1].x;
    const uint32_t size = E > S ? E - S : 0u;
    c[i] = (size + kPiece - 1) / kPiece;
    sum += c[i];
  }
  uint32_t x = sum;   // inclusive scan over the wave
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, 64);
    if ((tid & 63) >= (uint32_t)o) x += y;
  }
  if ((tid & 63) == 63) s_w[tid >> 6] = x;
  __syncthreads();
  uint32_t run = x - sum;
  for (uint32_t w = 0; w < (tid >> 6); ++w) run += s_w[w];
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    lp[tid * kPer + i].y = run;
    run += c[i];
  }
  if (tid == 255) lp[kLeaves].y = run;
}

// One wave per piece j of leaf l: keys[R..Rn), R = lb[l] + (j - po[l]) * kPiece.
// The pieces of all leaves tile the sorted keys in order, so a query key k
// picks the last piece whose first key is < k: the piece receives k in
// (keys[R], kmax] (kmax: the next piece's first key, keys[Rn], or the
// largest key for the last piece), and the lower bound lies in (R, Rn].
// For i in (R, Rn) the keys in (keys[i-1], keys[i]] have lower bound i (when
// keys[i-1] < keys[i]); the keys in (keys[Rn-1], kmax] have lower bound Rn.
// The prediction is monotone in k, so each interval's extremes of
// (bound - prediction) are at its ends.
__global__ __launch_bounds__(256) void learned_pieces(const uint64_t* __restrict__ keys,
                                                      uint64_t n, const uint2* __restrict__ lp,
                                                      uint32_t max_pieces,
                                                      uint64_t* __restrict__ fk,
                                                      PieceRec* __restrict__ pr,
                                                      uint32_t* __restrict__ ps) {
#pragma clang fp contract(off)
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t j = blockIdx.x * 4 + (threadIdx.x >> 6);
  const uint32_t np = lp[kLeaves].y;
  if (j >= np || j >= max_pieces) return;
  uint32_t lo = 0, hi = kLeaves - 1;   // leaf: largest l with first piece <= j
  while (lo < hi) {
    const uint32_t mid = (lo + hi + 1) >> 1;
    if (lp[mid].y <= j) lo = mid;
    else hi = mid - 1;
  }
  const uint32_t l = lo;
  const uint64_t S = lp[l].x, E = lp[l + 1].x < n ? lp[l + 1].x : n;
  const uint64_t R = S + (uint64_t)(j - lp[l].y) * kPiece;
  if (R >= E) return;   // never: pieces cover exactly their leaf
  const uint64_t Rn = R + kPiece < E ? R + kPiece : E;
  const bool last = j + 1 >= lp[l + 1].y;
  const uint64_t f = keys[R];
  const uint64_t kmax = Rn < n ? keys[Rn] : ~0ull;
  // the slope spans the piece's own keys (to the next piece's first key
  // inside the leaf)
  const double span = !last ? (double)(kmax - f) : (double)(keys[E - 1] - f) + 1.0;
  const double sl = span > 0.0 ? (double)(Rn - R) / span : 0.0;
  int64_t emin = INT64_MAX, emax = INT64_MIN;
  for (uint64_t i = R + 1 + lane; i <= Rn; i += 64) {
    uint64_t klo, khi;   // keys with lower bound i: (klo - 1, khi]
    if (i < Rn) {
      if (keys[i - 1] == keys[i]) continue;
      klo = keys[i - 1] + 1;
      khi = keys[i];
    } else {
      if (keys[Rn - 1] >= kmax) continue;
      klo = keys[Rn - 1] + 1;
      khi = kmax;
    }
    const int64_t ii = (int64_t)i;
    emin = min(emin, ii - piece_predict(sl, f, R, Rn, khi));
    emax = max(emax, ii - piece_predict(sl, f, R, Rn, klo));
  }
  for (int o = 32; o > 0; o >>= 1) {
    emin = min(emin, (int64_t)__shfl_xor(emin, o, 64));
    emax = max(emax, (int64_t)__shfl_xor(emax, o, 64));
  }
  if (lane == 0) {
    PieceRec rec;
    rec.s = sl;
    rec.elo = emin > emax ? 0 : (int32_t)emin;
    rec.ehi = emin > emax ? 0 : (int32_t)emax;
    fk[j] = f;
    pr[j] = rec;
    ps[j] = (uint32_t)R;
  }
}

// dt[t] = the number of pieces whose first key is below t << 44 (t < 2^20),
// dt[2^20] = the number of pieces; ps[pieces] = n.
__global__ __launch_bounds__(256) void learned_direct(const uint64_t* __restrict__ fk,
                                                      const uint2* __restrict__ lp, uint64_t n,
                                                      uint32_t* __restrict__ ps,
                                                      uint32_t* __restrict__ dt) {
  const uint32_t t = blockIdx.x * 256 + threadIdx.x;
  if (t > kDirectSlots) return;
  const uint32_t np = lp[kLeaves].y;
  if (t == kDirectSlots) {
    dt[t] = np;
    ps[np] = (uint32_t)n;
    return;
  }
  dt[t] = (uint32_t)lower_bound_in(fk, 0, np, (uint64_t)t << (64 - kDirectBits));
}

hipError_t fit_pieces(const uint64_t* keys, uint64_t n, const LearnedArrays& a, uint32_t max_pieces,
                      hipStream_t s) {
  hipError_t e;
  {
    ProfScope ps("learned_bounds", s);
    learned_keybounds<<<(kLeaves + 1 + 255) / 256, 256, 0, s>>>(keys, n, a.xb, a.lp);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    learned_piece_offsets<<<1, 256, 0, s>>>(a.lp);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  {
    ProfScope ps("learned_pieces", s);
    learned_pieces<<<(max_pieces + 3) / 4, 256, 0, s>>>(keys, n, a.lp, max_pieces, a.fk, a.pr,
                                                        a.ps);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    learned_direct<<<(kDirectSlots + 1 + 255) / 256, 256, 0, s>>>(a.fk, a.lp, n, a.ps, a.dt);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace

size_t learned_scratch_bytes() { return align256(kSamples * 4) * 3 + 256; }

uint32_t learned_max_pieces(uint64_t n) { return (uint32_t)(n / kPiece + kLeaves + 1); }

size_t learned_model_bytes(uint64_t n) {
  const uint64_t np = learned_max_pieces(n);
  return align256((kLeaves + 1) * 4) + align256((kRouteSlots + 1) * 4) +
         align256((kLeaves + 1) * 8) + align256(np * 8) + align256(np * sizeof(PieceRec)) +
         align256((np + 1) * 4) + align256((kDirectSlots + 1) * 4);
}

LearnedArrays learned_carve(void* base, uint64_t n) {
  const uint64_t np = learned_max_pieces(n);
  char* p = (char*)base;
  LearnedArrays a;
  a.xb = (uint32_t*)p;   p += align256((kLeaves + 1) * 4);
  a.rt = (uint32_t*)p;   p += align256((kRouteSlots + 1) * 4);
  a.lp = (uint2*)p;      p += align256((kLeaves + 1) * 8);
  a.fk = (uint64_t*)p;   p += align256(np * 8);
  a.pr = (PieceRec*)p;   p += align256(np * sizeof(PieceRec));
  a.ps = (uint32_t*)p;   p += align256((np + 1) * 4);
  a.dt = (uint32_t*)p;
  a.max_pieces = (uint32_t)np;
  return a;
}

hipError_t learned_fit(const uint64_t* keys, uint64_t n, uint32_t steps, float lr, float* params,
                       const LearnedArrays& a, void* scratch, float* losses, hipStream_t s) {
  if (n == 0) return hipErrorInvalidValue;
  uint32_t S = kSamples;
  while ((uint64_t)S > n) S >>= 1;
  char* p = (char*)scratch;
  float* xs = (float*)p;          p += align256(kSamples * 4);
  float* ts = (float*)p;          p += align256(kSamples * 4);
  float* sq = (float*)p;
  hipError_t e;
  {
    ProfScope ps("learned_sample", s);
    learned_sample<<<(S + 255) / 256, 256, 0, s>>>(keys, n, S, xs, ts);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    learned_init<<<1, 256, 0, s>>>(xs, S, params);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  auto loss = [&](float* out) {
    ProfScope ps("learned_loss", s);
    learned_errors<<<(S + 255) / 256, 256, 0, s>>>(params, xs, ts, S, sq);
    hipError_t le = hipGetLastError();
    if (le != hipSuccess) return le;
    learned_loss<<<1, 256, 0, s>>>(sq, S, out);
    return hipGetLastError();
  };
  if ((e = loss(losses)) != hipSuccess) return e;
  {
    ProfScope ps("learned_train", s);
    learned_train<<<1, kTrainThreads, 0, s>>>(xs, ts, S, steps, lr, params);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if ((e = loss(losses + 1)) != hipSuccess) return e;
  {
    ProfScope ps("learned_tabulate", s);
    learned_radix<<<(kRouteSlots + 1 + 255) / 256, 256, 0, s>>>(params, a.rt);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    learned_xbounds<<<(kLeaves + 1 + 63) / 64, 64, 0, s>>>(params, a.rt, a.xb);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return fit_pieces(keys, n, a, a.max_pieces, s);
}

hipError_t learned_refit_leaves(const uint64_t* keys, uint64_t n, const LearnedArrays& a,
                                hipStream_t s) {
  if (n == 0) return hipErrorInvalidValue;
  return fit_pieces(keys, n, a, a.max_pieces, s);
}

hipError_t learned_grad(const float* params, const float* xs, const float* ts, int cnt,
                        float* grad, float* loss, hipStream_t s) {
  if (cnt < 1 || cnt > kBatch) return hipErrorInvalidValue;
  learned_grad_kernel<<<1, kTrainThreads, 0, s>>>(params, xs, ts, cnt, grad, loss);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void route_both_kernel(const float* __restrict__ P,
                                                         LearnedView v,
                                                         const uint64_t* __restrict__ keys,
                                                         uint64_t count, uint32_t* __restrict__ direct,
                                                         uint32_t* __restrict__ table) {
  const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= count) return;
  const uint32_t X = (uint32_t)(keys[i] >> (64 - kXBits));
  direct[i] = router_leaf_x(P, X);
  table[i] = route(v, X);
}

hipError_t learned_route_both(const float* params, const LearnedArrays& a, const uint64_t* keys,
                              uint64_t count, uint32_t* direct, uint32_t* table, hipStream_t s) {
  if (count == 0) return hipSuccess;
  route_both_kernel<<<(uint32_t)((count + 255) / 256), 256, 0, s>>>(params, a.view(), keys, count,
                                                                   direct, table);
  return hipGetLastError();
}

}  // namespace sfc
