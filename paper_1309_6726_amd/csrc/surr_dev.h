// Private declarations of the surrogate kernels (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace surrdev {

constexpr int NIN = 5;      // width, length, reaction rate, contact angle, threshold
constexpr int KIN = 32;     // padded input width
constexpr int NHID = 256;   // hidden units
constexpr int NOUT = 65;    // 64 front positions + closure time
constexpr int NOUTP = 96;   // padded output width
constexpr int NL = 4;       // layers

// padded layer shapes [N x K] and the real ones
constexpr int LN[NL] = {NHID, NHID, NHID, NOUTP};
constexpr int LK[NL] = {KIN, NHID, NHID, NHID};
constexpr int RN[NL] = {NHID, NHID, NHID, NOUT};
constexpr int RK[NL] = {NIN, NHID, NHID, NHID};
constexpr int NPARAMS = NHID * NIN + NHID + 2 * (NHID * NHID + NHID) + NOUT * NHID + NOUT;

// Matrix operands are kept in the order in which the matrix instruction takes
// them ("fragments"): an operand with R rows and contraction length K is
// stored as [R / 32 tiles][K / 16 steps][64 lanes][8], lane l holding the
// elements 8 (l / 32) .. +7 of its step for row l mod 32, so a wavefront's
// load of one fragment is 1 KB in a row.

// The trained network as the kernels read it.
struct NetArgs {
  const __bf16* wf[NL];    // W_l as forward operand (rows = units of layer l)
  const __bf16* wt[NL];    // W_l^T as backward operand (rows = inputs of layer l); l >= 1
  const float* bias[NL];
  const float *lo, *hi;    // normalisation box
};

// Samples of one call: row r is sample idx[r] (r itself without idx).
struct RowArgs {
  const float* X;
  const int32_t* idx;
  int rows;
};

// What training needs beyond the forward pass.  at / dt hold the activations
// entering layer l and the gradient of its pre-activations as fragments with
// the units as rows and the batch as contraction (ks steps of 16 samples per
// tile).
struct TrainArgs {
  const float* Y;      // targets [n x NOUT]
  const float* RW;     // row weights or null
  const float* lw;     // output weights
  float scale;         // 1 / (rows * sum of output weights)
  __bf16* at[NL];
  __bf16* dt[NL];
  int ks;
  double* loss;
};

// Parameters, Adam moments and operand copies of every layer; padded W [N x K]
// followed by the bias [N].
struct UpdateArgs {
  const __bf16* at[NL];
  const __bf16* dt[NL];
  int ks, steps;           // allocated and used steps of 16 samples
  float* p[NL];
  float* m1[NL];
  float* m2[NL];
  __bf16* wf[NL];
  __bf16* wt[NL];
  float lr, b1, b2, eps, c1, c2;
  float* packed;           // gradients only: packed output, nothing is updated
  double* loss;            // with loss_out: the accumulated loss is handed over
  double* loss_out;        // there and its accumulator cleared
};

// Packed parameters and what is kept of them; the launchers fill in the shapes.
struct PackArgs {
  float* packed;
  float* p[NL];
  float* m1[NL];
  float* m2[NL];
  __bf16* wf[NL];
  __bf16* wt[NL];
  int first[NL], rn[NL], rk[NL], n[NL], k[NL];
};

// Whether n queries at x and their answers at y share memory.
inline bool overlap(const float* x, const float* y, size_t n) {
  return (uintptr_t)x < (uintptr_t)(y + n * NOUT) && (uintptr_t)y < (uintptr_t)(x + n * NIN);
}

// y [rows x NOUT] (host-visible or device memory; with at most 1024 rows it may
// overlap the queries).
hipError_t predict(const NetArgs& net, const RowArgs& r, float* y, hipStream_t st);
hipError_t forward_backward(const NetArgs& net, const RowArgs& r, const TrainArgs& t, hipStream_t st);
hipError_t update(const UpdateArgs& u, hipStream_t st);
hipError_t unpack_params(const PackArgs& a, hipStream_t st);
hipError_t pack_params(const PackArgs& a, hipStream_t st);

}  // namespace surrdev
