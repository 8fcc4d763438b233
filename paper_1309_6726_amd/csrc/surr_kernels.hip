// Kernels of the MLP surrogate (5 -> 256 -> 256 -> 256 -> 65, ReLU) that maps
// capillary parameters (width, length, reaction rate, contact angle,
// precipitation threshold) to the front trajectory and the pore-closure time.
//
// Every dense-layer product, forward and backward, has the form
//   C[M x N] = A[M x K] * Bt[N x K]^T
// on the matrix cores with v_mfma_f32_32x32x16_bf16 (BF16 operands, FP32
// accumulation, K in ascending steps of 16).  One wavefront owns one 32 x 32
// tile of C.  Lane l passes the elements k0 + 8 (l / 32) .. +7 of row l mod 32
// of its A tile and of its Bt tile; its 16 accumulators hold
// C[8 (i / 4) + 4 (l / 32) + (i mod 4)][l mod 32], i = 0..15.
//
// The network is small (149,825 parameters, 300 KB in BF16), so what a call
// costs is latency: kernel launches and round trips to memory between them.
// One workgroup therefore takes 32 samples through all layers, activations in
// LDS, and training is two launches per minibatch: k_rows (forward, loss,
// backward) and k_update (weight and bias gradients, Adam, operand copies).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "surr_dev.h"

namespace surrdev {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int ROWS = 32;          // samples per workgroup of k_rows
constexpr int HS = NHID + 8;      // LDS row strides in elements: 16-byte aligned,
constexpr int XS = KIN + 8;       // and the 16-byte reads of 16 consecutive rows
constexpr int YS = NOUTP + 8;     // fall on all 64 banks

__device__ __forceinline__ floatx16 zero16() {
  floatx16 z;
#pragma unroll
  for (int i = 0; i < 16; ++i) z[i] = 0.0f;
  return z;
}

// Row of accumulator i in lane l of a 32 x 32 tile.
__device__ __forceinline__ int acc_row(int i, int half) { return 8 * (i >> 2) + 4 * half + (i & 3); }

template <int KS>
__device__ __forceinline__ void load_frags(bf16x8* w, const __bf16* frags, int tile, int lane) {
  const bf16x8* p = (const bf16x8*)frags + (size_t)tile * KS * 64 + lane;
#pragma unroll
  for (int s = 0; s < KS; ++s) w[s] = p[s * 64];
}

// One 32 x 32 tile: A rows from LDS (row stride `stride` elements).
template <int KS>
__device__ __forceinline__ floatx16 product(const __bf16* a, int stride, const bf16x8* w, int lane) {
  const __bf16* ap = a + (lane & 31) * stride + 8 * (lane >> 5);
  floatx16 acc = zero16();
#pragma unroll
  for (int s = 0; s < KS; ++s)
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8*)(ap + 16 * s), w[s], acc, 0, 0, 0);
  return acc;
}

// Element offset of accumulators 4 q .. 4 q + 3 of lane `lane` in fragments
// that have a tile's columns as rows and its rows as contraction: row tile
// `tile` of `ks` steps, contraction elements 32 block .. +31.
__device__ __forceinline__ size_t transposed_at(int ks, int tile, int block, int q, int lane) {
  return ((size_t)tile * ks + 2 * block + (q >> 1)) * 512 + (q & 1) * 256 + (lane & 31) * 8 + 4 * (lane >> 5);
}

__device__ __forceinline__ void store_transposed(__bf16* frags, int ks, int tile, int block,
                                                 const __bf16* v, int lane) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const bf16x4 o = {v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
    *(bf16x4*)(frags + transposed_at(ks, tile, block, q, lane)) = o;
  }
}

// A minibatch of 256 runs on eight CUs, one per XCD, and each XCD's L2 misses
// on all the weights that the update before has just written elsewhere.  In
// training WARMERS more workgroups per XCD therefore read the weights, in the
// order of their use, and drop them: block b runs on XCD b mod 8, so they fill
// the L2 of the XCDs that hold samples.  14.3 -> 13.8 us per minibatch of 256
// (an epoch of 3584 samples 330.6 -> 319.0 us); a prediction's weights stay in
// the L2 from call to call.
constexpr int WARMERS = 8;
template <int L>
__device__ __forceinline__ void warm(const __bf16* w, int part) {
  constexpr int PIECE = 512 * 8, PIECES = LN[L] * LK[L] / PIECE;  // elements of one load of all threads
#pragma unroll
  for (int p = 0; p < (PIECES + WARMERS - 1) / WARMERS; ++p)
    if (p * WARMERS + part < PIECES) {
      const float4 v = ((const float4*)w)[(p * WARMERS + part) * 512 + threadIdx.x];
      asm volatile("" ::"v"(v.x), "v"(v.y), "v"(v.z), "v"(v.w));
    }
}

// Forward pass of 32 samples by one workgroup of eight wavefronts, wavefront
// w owning units 32 w .. +31 of a hidden layer; with TRAIN also the loss
// gradient and the backward pass.
//
// Inputs x = (W, L, k_r, theta, threshold) are normalised to
// 2 (x - lo) / (hi - lo) - 1, with log10 applied to k_r and its bounds; rows
// beyond the last sample have zero inputs and zero loss gradient.
//
// Loss: sum_rows c_r sum_j w_j (y - t)^2 * scale with per-output weights w and
// per-row weights c, added to *loss.
//
// What bounds it: one workgroup reads every weight once (328 KB forward, as
// much again backward) through one CU's memory port, so the fragments of a
// layer are requested two layers ahead of their use.  32 samples is the
// matrix instruction's tile; fewer workgroups than CUs run for small batches.
// Measured: 5.6 us for 8 prediction rows (33 us as six launches and a copy),
// 13.8 us for a training minibatch of 256 (16.0 when the targets' loads went row
// by row behind the weights, the loss branched for each element and its sum
// was folded before the backward pass), which with k_update's 4.8 us took 21
// launches and 120 us when every layer product, bias sum and update was a launch
// of its own.
template <bool TRAIN>
__global__ void __launch_bounds__(512) k_rows(const NetArgs net, const RowArgs ra,
                                              const TrainArgs ta, float* __restrict__ y) {
  __shared__ __align__(16) __bf16 sx[ROWS * XS];
  __shared__ __align__(16) __bf16 sa[ROWS * HS];
  __shared__ __align__(16) __bf16 sb[ROWS * HS];
  __shared__ __align__(16) __bf16 sy[TRAIN ? ROWS * YS : 8];
  __shared__ float st[TRAIN ? ROWS * NOUT : 1];  // targets
  __shared__ float sc[TRAIN ? ROWS : 1];         // row weights
  if constexpr (TRAIN) {
    const int blocks = (ra.rows + ROWS - 1) / ROWS, first = (blocks + 7) & ~7, b = (int)blockIdx.x;
    if (b >= blocks) {
      if (b < first || (b & 7) >= blocks) return;
      const int part = (b - first) >> 3;
      warm<1>(net.wf[1], part);
      warm<2>(net.wf[2], part);
      warm<3>(net.wf[3], part);
      warm<3>(net.wt[3], part);
      warm<2>(net.wt[2], part);
      warm<1>(net.wt[1], part);
      return;
    }
  }
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int col = lane & 31, half = lane >> 5;
  const int r0 = blockIdx.x * ROWS;
  const int unit = 32 * wave + col;

  auto normalise = [](int j, float x, float lo, float hi) {
    if (j == 2) { x = log10f(x); lo = log10f(lo); hi = log10f(hi); }
    return 2.0f * (x - lo) / (hi - lo) - 1.0f;
  };
  constexpr int YI = (ROWS * NOUT + 511) / 512;
  const int tid = threadIdx.x;
  auto target = [&](int i) { return min(tid + 512 * i, ROWS * NOUT - 1); };
  bf16x8 w0[2], wa[16], wb[16];
  float bias[NL], lw = 0.0f, yv[YI], cv = 1.0f;
  auto load_biases = [&]() {
#pragma unroll
    for (int l = 0; l < 3; ++l) bias[l] = net.bias[l][unit];
    bias[3] = wave < 3 ? net.bias[3][unit] : 0.0f;
  };
  if constexpr (TRAIN) {
    // A wavefront's loads return in the order they were requested: the rows'
    // indices come first, then the inputs and targets that hang on them, then
    // the weights.  Rows beyond the last sample read the last one's, unused.
    constexpr int XI = ROWS * KIN / 512;
    static_assert(KIN == 32 && XI * 512 == ROWS * KIN, "thread t loads input t mod 32 of row t / 32 + 16 i");
    auto source = [&](int r) {
      const int at = min(r0 + r, ra.rows - 1);
      return ra.idx ? ra.idx[at] : at;
    };
    int xsrc[XI], ysrc[YI];
#pragma unroll
    for (int i = 0; i < XI; ++i) xsrc[i] = source((tid >> 5) + 16 * i);
#pragma unroll
    for (int i = 0; i < YI; ++i) ysrc[i] = source(target(i) / NOUT);
    const int csrc = ta.RW ? source(tid & (ROWS - 1)) : 0;
    const int j = tid & 31, jin = min(j, NIN - 1);
    const float lo = net.lo[jin], hi = net.hi[jin];
    load_biases();
    if (unit < NOUT) lw = ta.lw[unit];
    load_frags<2>(w0, net.wf[0], wave, lane);
    float xv[XI];
#pragma unroll
    for (int i = 0; i < XI; ++i) xv[i] = ra.X[(size_t)xsrc[i] * NIN + jin];
#pragma unroll
    for (int i = 0; i < YI; ++i) yv[i] = ta.Y[(size_t)ysrc[i] * NOUT + target(i) % NOUT];
    if (ta.RW) cv = ta.RW[csrc];
    load_frags<16>(wa, net.wf[1], wave, lane);
#pragma unroll
    for (int i = 0; i < XI; ++i) {
      asm volatile("" : "+v"(xv[i]));  // keeps the load where it was requested
      const int r = (tid >> 5) + 16 * i;
      const __bf16 v = (__bf16)(r0 + r < ra.rows && j < NIN ? normalise(j, xv[i], lo, hi) : 0.0f);
      sx[r * XS + j] = v;
      // samples as contraction: unit j, sample r of block blockIdx.x
      ta.at[0][((size_t)2 * blockIdx.x + (r >> 4)) * 512 + (((r >> 3) & 1) * 32 + j) * 8 + (r & 7)] = v;
    }
  } else {
    // a prediction's inputs hang on nothing, and few rows leave whole
    // wavefronts without any: weights first (8 rows: 5.7 us; 5.9 to 6.2 with
    // every wavefront's inputs requested before the second layer's weights)
    load_frags<2>(w0, net.wf[0], wave, lane);
    load_frags<16>(wa, net.wf[1], wave, lane);
    load_biases();
    for (int e = tid; e < ROWS * KIN; e += 512) {
      const int r = e / KIN, j = e % KIN;
      float v = 0.0f;
      if (r0 + r < ra.rows && j < NIN) {
        const int src = ra.idx ? ra.idx[r0 + r] : r0 + r;
        v = normalise(j, ra.X[(size_t)src * NIN + j], net.lo[j], net.hi[j]);
      }
      sx[r * XS + j] = (__bf16)v;
    }
  }
  load_frags<16>(wb, net.wf[2], wave, lane);
  __syncthreads();

  unsigned live[3];  // units with a positive activation, one bit per accumulator
  // h = relu(v + b) of one tile: into LDS and, for training, as the next
  // layer's transposed operand
  auto hidden = [&](const floatx16& acc, int l, __bf16* dst) {
    __bf16 h[16];
    live[l] = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float v = fmaxf(acc[i] + bias[l], 0.0f);
      live[l] |= v > 0.0f ? 1u << i : 0u;
      h[i] = (__bf16)v;
      dst[acc_row(i, half) * HS + unit] = h[i];
    }
    if (TRAIN) store_transposed(ta.at[l + 1], ta.ks, wave, blockIdx.x, h, lane);
  };
  hidden(product<2>(sx, XS, w0, lane), 0, sa);
  if (TRAIN) {
#pragma unroll
    for (int i = 0; i < YI; ++i) st[target(i)] = yv[i];  // the last threads write one target's value twice
    if (tid < ROWS) sc[tid] = cv;
  }
  __syncthreads();
  hidden(product<16>(sa, HS, wa, lane), 1, sb);
  if (wave < 3) load_frags<16>(wa, net.wf[3], wave, lane);
  bf16x8 wc[6];
  if (TRAIN) load_frags<6>(wc, net.wt[3], wave, lane);
  __syncthreads();
  hidden(product<16>(sb, HS, wb, lane), 2, sa);
  if (TRAIN) load_frags<16>(wb, net.wt[2], wave, lane);
  __syncthreads();

  double sum = 0.0;  // this lane's part of the loss
  if (wave < 3) {
    const floatx16 acc = product<16>(sa, HS, wa, lane);
    if (!TRAIN) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int r = r0 + acc_row(i, half);
        if (r < ra.rows && unit < NOUT) y[(size_t)r * NOUT + unit] = acc[i] + bias[3];
      }
    } else {
      __bf16 dy[16];
      const int u = min(unit, NOUT - 1);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int r = acc_row(i, half);
        const bool real = r0 + r < ra.rows && unit < NOUT;
        const float yv = acc[i] + bias[3];
        const float diff = yv - st[r * NOUT + u];
        const float c = lw * sc[r] * ta.scale;
        sum += real ? (double)(c * diff * diff) : 0.0;
        dy[i] = (__bf16)(real ? 2.0f * c * diff : 0.0f);
        sy[r * YS + unit] = dy[i];
      }
      store_transposed(ta.dt[3], ta.ks, wave, blockIdx.x, dy, lane);
    }
  }
  if (!TRAIN) return;

  load_frags<16>(wa, net.wt[1], wave, lane);
  __syncthreads();
  // dh = v where the unit was live: into LDS for the next product and as the
  // transposed operand of the weight gradient
  auto masked = [&](const floatx16& acc, int l, __bf16* dst) {
    __bf16 d[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      d[i] = (__bf16)(live[l] & (1u << i) ? acc[i] : 0.0f);
      if (dst) dst[acc_row(i, half) * HS + unit] = d[i];
    }
    store_transposed(ta.dt[l], ta.ks, wave, blockIdx.x, d, lane);
  };
  masked(product<6>(sy, YS, wc, lane), 2, sb);
  __syncthreads();
  masked(product<16>(sb, HS, wb, lane), 1, sa);
  __syncthreads();
  masked(product<16>(sa, HS, wa, lane), 0, nullptr);
  if (wave < 3) {
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_down(sum, o);
    if (lane == 0) atomicAdd(ta.loss, sum);
  }
}

// ---- parameter update ------------------------------------------------------
// Tiles of 32 x 32 weights of each layer, then groups of eight biases.
constexpr int BIAS_GROUP = 8;
__host__ __device__ constexpr int weight_tiles(int l) { return (LN[l] / 32) * (LK[l] / 32); }
constexpr int WEIGHT_TILES = weight_tiles(0) + weight_tiles(1) + weight_tiles(2) + weight_tiles(3);
constexpr int BIAS_GROUPS = (3 * NHID + NOUTP) / BIAS_GROUP;
static_assert(BIAS_GROUPS % 4 == 0, "four bias groups per workgroup");

// Offset of W_l in the packed parameters; b_l follows it.
__host__ __device__ constexpr int packed_weights(int l) {
  constexpr int first = RN[0] * RK[0] + RN[0], hidden = NHID * NHID + NHID;
  return l == 0 ? 0 : first + (l - 1) * hidden;
}

// Adam on one FP32 parameter, the fused multiply-adds written out so that
// every inlined copy rounds alike.
__device__ __forceinline__ float adam(const UpdateArgs& u, float g, float p, float& m1, float& m2) {
  const float a = fmaf(1.0f - u.b1, g, u.b1 * m1);
  const float v = fmaf(g, (1.0f - u.b2) * g, u.b2 * m2);
  m1 = a;
  m2 = v;
  return p - u.lr * (a / u.c1) / (sqrtf(v / u.c2) + u.eps);
}

// Gradient of 32 x 32 weights of layer L (contraction over the batch), then
// Adam on the FP32 master weights and both BF16 operand copies.  Each of the
// four wavefronts forms the whole product (16 matrix instructions for 256
// samples, operands shared in L1) and updates four of its sixteen rows per
// lane: the divisions and square roots of Adam are what this launch waits on
// otherwise.  What is left is one round trip of loads, the products, Adam and
// the stores.  us a minibatch: 7.8 with one wavefront per tile, 6.4 with eight
// steps of operands in flight and a bias's moments behind its sum, 4.8 now.
template <int L>
__device__ __forceinline__ void update_weights(const UpdateArgs& u, int tile, __bf16* lds) {
  constexpr int N = LN[L], K = LK[L], TK = K / 32;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, col = lane & 31, half = lane >> 5;
  const int tn = tile / TK, tk = tile % TK;
  const bf16x8* a = (const bf16x8*)u.dt[L] + (size_t)tn * u.ks * 64 + lane;
  const bf16x8* b = (const bf16x8*)u.at[L] + (size_t)tk * u.ks * 64 + lane;
  const int k = 32 * tk + col;
  const int n0 = 32 * tn + acc_row(4 * wave, half);  // rows n0 .. n0 + 3 of this lane
  float p[4], m1[4], m2[4];
  if (!u.packed) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = (n0 + i) * K + k;
      p[i] = u.p[L][e];
      m1[i] = u.m1[L][e];
      m2[i] = u.m2[L][e];
    }
  }
  floatx16 acc = zero16();
  // sixteen steps of operands in flight, so 256 samples cost one round trip
  int s = 0;
  auto steps = [&](auto count) {
    constexpr int n = decltype(count)::value;
    bf16x8 av[n], bv[n];
#pragma unroll
    for (int q = 0; q < n; ++q) { av[q] = a[(s + q) * 64]; bv[q] = b[(s + q) * 64]; }
    __builtin_amdgcn_sched_barrier(0);  // all of them requested before the first product
#pragma unroll
    for (int q = 0; q < n; ++q)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[q], bv[q], acc, 0, 0, 0);
    s += n;
  };
  while (s + 16 <= u.steps) steps(std::integral_constant<int, 16>{});
  if (s + 8 <= u.steps) steps(std::integral_constant<int, 8>{});
  for (; s < u.steps; ++s)
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[s * 64], b[s * 64], acc, 0, 0, 0);
  float g[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    g[i] = wave < 2 ? (wave == 0 ? acc[i] : acc[4 + i]) : (wave == 2 ? acc[8 + i] : acc[12 + i]);
  if (u.packed) {
    constexpr int w0 = packed_weights(L);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (n0 + i < RN[L] && k < RK[L]) u.packed[w0 + (n0 + i) * RK[L] + k] = g[i];
    return;
  }
  bf16x4 w;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int e = (n0 + i) * K + k;
    const float v = adam(u, g[i], p[i], m1[i], m2[i]);
    u.p[L][e] = v;
    u.m1[L][e] = m1[i];
    u.m2[L][e] = m2[i];
    w[i] = (__bf16)v;
    lds[(acc_row(4 * wave, half) + i) * XS + col] = w[i];
  }
  if (L > 0) *(bf16x4*)(u.wt[L] + transposed_at(N / 16, tk, tn, wave, lane)) = w;
  __syncthreads();
  if (wave >= 2) return;
  bf16x8* wf = (bf16x8*)u.wf[L] + ((size_t)tn * (K / 16) + 2 * tk) * 64 + lane;
  wf[wave * 64] = *(const bf16x8*)(lds + col * XS + 16 * wave + 8 * half);
}

// Eight biases from n0 on: sum over the batch of the pre-activation gradient
// (lane t adds samples t, t + 64, ..., then a fixed tree), then Adam.
template <int L>
__device__ __forceinline__ void update_biases(const UpdateArgs& u, int n0) {
  const int lane = threadIdx.x & 63;
  const __bf16* d = u.dt[L] + (size_t)(n0 >> 5) * u.ks * 512 + (n0 & 31) * 8;
  const int n = n0 + lane, e = LN[L] * LK[L] + n;
  float p = 0.0f, m1 = 0.0f, m2 = 0.0f;  // requested with the gradients
  if (lane < BIAS_GROUP && !u.packed) {
    p = u.p[L][e];
    m1 = u.m1[L][e];
    m2 = u.m2[L][e];
  }
  float s[BIAS_GROUP];
#pragma unroll
  for (int j = 0; j < BIAS_GROUP; ++j) s[j] = 0.0f;
  for (int m = lane; m < 16 * u.steps; m += 64) {
    const __bf16* dm = d + (m >> 4) * 512 + ((m >> 3) & 1) * 256 + (m & 7);
#pragma unroll
    for (int j = 0; j < BIAS_GROUP; ++j) s[j] += (float)dm[8 * j];
  }
  float g = 0.0f;  // lane j: gradient of bias n0 + j
#pragma unroll
  for (int j = 0; j < BIAS_GROUP; ++j) {
    for (int o = 32; o > 0; o >>= 1) s[j] += __shfl_down(s[j], o);
    const float t = __shfl(s[j], 0);
    if (lane == j) g = t;
  }
  if (lane >= BIAS_GROUP) return;
  if (u.packed) {
    if (n < RN[L]) u.packed[packed_weights(L) + RN[L] * RK[L] + n] = g;
    return;
  }
  u.p[L][e] = adam(u, g, p, m1, m2);
  u.m1[L][e] = m1;
  u.m2[L][e] = m2;
}

// One workgroup per weight tile, one wavefront per bias group: 187
// workgroups, each one chain of loads, products and stores.
__global__ void __launch_bounds__(256) k_update(const UpdateArgs u) {
  __shared__ __align__(16) __bf16 lds[32 * XS];
  int t = blockIdx.x;
  if (t < weight_tiles(0)) return update_weights<0>(u, t, lds);
  t -= weight_tiles(0);
  if (t < weight_tiles(1)) return update_weights<1>(u, t, lds);
  t -= weight_tiles(1);
  if (t < weight_tiles(2)) return update_weights<2>(u, t, lds);
  t -= weight_tiles(2);
  if (t < weight_tiles(3)) return update_weights<3>(u, t, lds);
  if (t == weight_tiles(3) && threadIdx.x == 0 && u.loss_out) {
    *u.loss_out = *u.loss;
    *u.loss = 0.0;
  }
  t = 4 * (t - weight_tiles(3)) + (int)(threadIdx.x >> 6);  // bias group
  constexpr int G = NHID / BIAS_GROUP;
  if (t < G) return update_biases<0>(u, t * BIAS_GROUP);
  if (t < 2 * G) return update_biases<1>(u, (t - G) * BIAS_GROUP);
  if (t < 3 * G) return update_biases<2>(u, (t - 2 * G) * BIAS_GROUP);
  update_biases<3>(u, (t - 3 * G) * BIAS_GROUP);
}

// Padded parameters of layer blockIdx.y from the packed ones (zero in the
// padding), Adam moments cleared, and both BF16 operand copies of the weights.
__global__ void k_unpack(const PackArgs a) {
  const int l = blockIdx.y, N = a.n[l], K = a.k[l];
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N * K + N) return;
  const bool weight = i < N * K;
  const int r = weight ? i / K : i - N * K, c = weight ? i - r * K : 0;
  const float* in = a.packed + a.first[l] + (weight ? r * a.rk[l] + c : a.rn[l] * a.rk[l] + r);
  const float v = r < a.rn[l] && c < a.rk[l] ? *in : 0.0f;
  a.p[l][i] = v;
  a.m1[l][i] = 0.0f;
  a.m2[l][i] = 0.0f;
  if (!weight) return;
  auto at = [](int row, int k, int len) {
    return ((size_t)(row >> 5) * (len >> 4) + (k >> 4)) * 512 + (((k >> 3) & 1) * 32 + (row & 31)) * 8 + (k & 7);
  };
  a.wf[l][at(r, c, K)] = (__bf16)v;
  if (l > 0) a.wt[l][at(c, r, N)] = (__bf16)v;
}

// Real entries of the padded parameters (layer blockIdx.y) into the packed
// layout.
__global__ void k_pack(const PackArgs a) {
  const int l = blockIdx.y;
  const int nw = a.rn[l] * a.rk[l], i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nw + a.rn[l])
    a.packed[a.first[l] + i] = i < nw ? a.p[l][(i / a.rk[l]) * a.k[l] + i % a.rk[l]]
                                      : a.p[l][a.n[l] * a.k[l] + i - nw];
}

// Moves `count` values, which may overlap where they go: every thread holds its
// own until all are read.
constexpr int MOVE = 10;  // values per thread: 1024 queries
__global__ void __launch_bounds__(512) k_move(const float* x, float* to, int count) {
  float v[MOVE];
#pragma unroll
  for (int i = 0; i < MOVE; ++i) {
    const int e = threadIdx.x + 512 * i;
    v[i] = e < count ? x[e] : 0.0f;
  }
#pragma unroll
  for (int i = 0; i < MOVE; ++i) asm volatile("" : "+v"(v[i]));  // arrived
  __syncthreads();
#pragma unroll
  for (int i = 0; i < MOVE; ++i) {
    const int e = threadIdx.x + 512 * i;
    if (e < count) to[e] = v[i];
  }
}

// ---- launchers ------------------------------------------------------------
// Answers over their own queries: the queries are moved to the end of the answers
// and taken 32 at a time, first to last.  Of n rows, the first k answers end at
// value k NOUT and the queries after the first k begin at n (NOUT - NIN) + k NIN, which is
// no less for k <= n: a launch overwrites no query of a later one.
static hipError_t predict_in_place(const NetArgs& net, const RowArgs& r, float* y, hipStream_t st) {
  if (r.idx || r.rows * NIN > MOVE * 512) return hipErrorInvalidValue;
  float* const x = y + (size_t)r.rows * (NOUT - NIN);
  hipLaunchKernelGGL(k_move, dim3(1), dim3(512), 0, st, r.X, x, r.rows * NIN);
  for (int first = 0; first < r.rows; first += ROWS) {
    const RowArgs part{x + (size_t)first * NIN, nullptr, r.rows - first < ROWS ? r.rows - first : ROWS};
    hipLaunchKernelGGL(k_rows<false>, dim3(1), dim3(512), 0, st, net, part, TrainArgs{}, y + (size_t)first * NOUT);
  }
  return hipGetLastError();
}

hipError_t predict(const NetArgs& net, const RowArgs& r, float* y, hipStream_t st) {
  // one workgroup reads all its queries before it answers, several do not wait
  // for each other
  if (r.rows > ROWS && overlap(r.X, y, r.rows)) return predict_in_place(net, r, y, st);
  hipLaunchKernelGGL(k_rows<false>, dim3((r.rows + ROWS - 1) / ROWS), dim3(512), 0, st, net, r, TrainArgs{}, y);
  return hipGetLastError();
}

hipError_t forward_backward(const NetArgs& net, const RowArgs& r, const TrainArgs& t, hipStream_t st) {
  // Warming workgroups up to 1024 rows: beyond, the eight and more workgroups
  // of an XCD fetch for each other.  us per minibatch without and with them: 32
  // rows 17.5, 16.9; 256 rows 19.1, 18.4; 1024 rows 26.4, 26.3; 2048 rows 36.5,
  // 36.7; 4096 rows 52.9, 53.1.
  const int blocks = (r.rows + ROWS - 1) / ROWS;
  const int grid = blocks <= 32 ? (blocks + 7) / 8 * 8 + 8 * WARMERS : blocks;
  hipLaunchKernelGGL(k_rows<true>, dim3(grid), dim3(512), 0, st, net, r, t, nullptr);
  return hipGetLastError();
}

hipError_t update(const UpdateArgs& u, hipStream_t st) {
  hipLaunchKernelGGL(k_update, dim3(WEIGHT_TILES + BIAS_GROUPS / 4), dim3(256), 0, st, u);
  return hipGetLastError();
}

static PackArgs with_shapes(PackArgs a) {
  for (int l = 0; l < NL; ++l) {
    a.first[l] = packed_weights(l);
    a.rn[l] = RN[l];
    a.rk[l] = RK[l];
    a.n[l] = LN[l];
    a.k[l] = LK[l];
  }
  return a;
}

static dim3 pack_grid() { return dim3((NHID * NHID + NHID + 255) / 256, NL); }

hipError_t unpack_params(const PackArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(k_unpack, pack_grid(), dim3(256), 0, st, with_shapes(a));
  return hipGetLastError();
}

hipError_t pack_params(const PackArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(k_pack, pack_grid(), dim3(256), 0, st, with_shapes(a));
  return hipGetLastError();
}

}  // namespace surrdev
