// Host side of the surrogate C ABI (include/lbm.h, surr_*): workspace layout,
// parameter packing, training epochs, gradients and prediction.  All
// arithmetic runs in the kernels of surr_kernels.hip.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>
#include <memory>
#include <new>
#include <vector>

#include "lbm.h"
#include "lbm_dev.h"
#include "pinned.h"
#include "surr_dev.h"

using lbmdev::fail;
using namespace surrdev;

namespace {

size_t a256(size_t x) { return (x + 255) & ~size_t(255); }

struct SLayout {
  size_t p[NL], m1[NL], m2[NL], wf[NL], wt[NL], at[NL], dt[NL];
  size_t X, Y, RW, perm, qx, qy, lo, hi, lw, loss, total;
  int Bp, max_data;
};

SLayout slayout(int max_batch, int max_data) {
  SLayout S;
  S.Bp = (max_batch + 31) / 32 * 32;
  S.max_data = max_data;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off = a256(off + bytes); return o; };
  const size_t B = S.Bp;
  for (int l = 0; l < NL; ++l) {
    const size_t cnt = (size_t)LN[l] * LK[l] + LN[l];
    S.p[l] = take(cnt * 4);
    S.m1[l] = take(cnt * 4);
    S.m2[l] = take(cnt * 4);
    S.wf[l] = take((size_t)LN[l] * LK[l] * 2);
    S.wt[l] = take((size_t)LN[l] * LK[l] * 2);
    S.at[l] = take(B * LK[l] * 2);
    S.dt[l] = take(B * LN[l] * 2);
  }
  S.X = take((size_t)max_data * NIN * 4);
  S.Y = take((size_t)max_data * NOUT * 4);
  S.RW = take((size_t)max_data * 4);
  S.perm = take((size_t)max_data * 4);
  S.qx = take(B * NIN * 4);
  S.qy = take(B * NOUT * 4);
  S.lo = take(NIN * 4);
  S.hi = take(NIN * 4);
  S.lw = take(NOUT * 4);
  S.loss = take(8);
  S.total = off;
  return S;
}

constexpr int NOALLOC_ROWS = 1024;  // most query rows of one surr_predict_noalloc

// Pinned host memory that a call takes (0.9 MB).  Queries, answers, gradients, the
// loss and the packed parameters pass through it: the kernels read and write it
// themselves, so a call is its launches and one wait.  Copies to and from pageable
// memory cost 10-20 us each, and the copy of the answers' columns out of their
// padded rows went row by row (1.8 ms for 256 rows).
constexpr int HOST_ROWS = 1024;  // rows per launch that reads its samples here
struct HostBuffer {
  double loss;
  float x[HOST_ROWS * NIN];
  float y[HOST_ROWS * NOUT];
  float packed[NPARAMS];
};

}  // namespace

struct surr_net {
  SLayout S;
  char* ws;
  hipStream_t stream;
  int n_data;
  long long adam_t;
  float wsum;    // sum of the loss weights, added in order in FP32
  bool loss_dirty;     // the loss accumulator may hold a failed call's part
  template <typename T> T* at(size_t off) const { return (T*)(ws + off); }
};

namespace {

#define HC(expr)                                                                            \
  do {                                                                                      \
    hipError_t e_ = (expr);                                                                 \
    if (e_ != hipSuccess) return fail(LBM_EDEVICE, "%s: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

// The pinned buffer of one call, whose kernels may use it until wait() or done():
// where a call fails before, HIP gets the buffer back and waits for them.
class CallBuffer {
 public:
  lbm_status take() {
    if (!(host_ = (HostBuffer*)block_.take(sizeof(HostBuffer), true)))
      return fail(LBM_ENOMEM, "no pinned memory");
    block_.in_use();
    return LBM_OK;
  }
  lbm_status wait(hipStream_t st) {
    HC(hipStreamSynchronize(st));
    done();
    return LBM_OK;
  }
  void done() { block_.done(); }
  HostBuffer* operator->() const { return host_; }

 private:
  lbmdev::Pinned block_;
  HostBuffer* host_ = nullptr;
};

NetArgs net_args(const surr_net* s) {
  NetArgs n{};
  for (int l = 0; l < NL; ++l) {
    n.wf[l] = s->at<__bf16>(s->S.wf[l]);
    n.wt[l] = s->at<__bf16>(s->S.wt[l]);
    n.bias[l] = s->at<float>(s->S.p[l]) + (size_t)LN[l] * LK[l];
  }
  n.lo = s->at<float>(s->S.lo);
  n.hi = s->at<float>(s->S.hi);
  return n;
}

// Forward and backward pass of `rows` samples gathered from (X, Y, RW) by idx
// (or in order); the loss is added to S.loss.
lbm_status sample_pass(surr_net* s, const float* X, const float* Y, const float* RW,
                       const int32_t* idx, int rows) {
  const SLayout& S = s->S;
  TrainArgs t{};
  t.Y = Y;
  t.RW = RW;
  t.lw = s->at<float>(S.lw);
  t.scale = 1.0f / ((float)rows * s->wsum);
  for (int l = 0; l < NL; ++l) {
    t.at[l] = s->at<__bf16>(S.at[l]);
    t.dt[l] = s->at<__bf16>(S.dt[l]);
  }
  t.ks = S.Bp / 16;
  t.loss = s->at<double>(S.loss);
  HC(forward_backward(net_args(s), RowArgs{X, idx, rows}, t, s->stream));
  return LBM_OK;
}

// The loss accumulator is zero between calls: the last update of a call hands
// the sum over and clears it.
lbm_status begin_loss(surr_net* s) {
  if (s->loss_dirty) HC(hipMemsetAsync(s->ws + s->S.loss, 0, 8, s->stream));
  s->loss_dirty = true;
  return LBM_OK;
}

// Waits for a call's last update, after which its buffer holds the loss.
lbm_status end_loss(surr_net* s, CallBuffer& host) {
  const lbm_status st = host.wait(s->stream);
  if (st == LBM_OK) s->loss_dirty = false;
  return st;
}

// Gradients of the last sample_pass: packed, or applied by Adam.
UpdateArgs update_args(surr_net* s, int rows) {
  const SLayout& S = s->S;
  UpdateArgs u{};
  for (int l = 0; l < NL; ++l) {
    u.at[l] = s->at<__bf16>(S.at[l]);
    u.dt[l] = s->at<__bf16>(S.dt[l]);
    u.p[l] = s->at<float>(S.p[l]);
    u.m1[l] = s->at<float>(S.m1[l]);
    u.m2[l] = s->at<float>(S.m2[l]);
    u.wf[l] = s->at<__bf16>(S.wf[l]);
    u.wt[l] = s->at<__bf16>(S.wt[l]);
  }
  u.ks = S.Bp / 16;
  u.steps = (rows + 31) / 32 * 2;
  u.loss = s->at<double>(S.loss);
  return u;
}

// loss_out: where the loss goes with a call's last update, else null.
lbm_status adam_step(surr_net* s, int rows, float lr, double* loss_out) {
  UpdateArgs u = update_args(s, rows);
  u.loss_out = loss_out;
  s->adam_t += 1;
  u.lr = lr;
  u.b1 = 0.9f;
  u.b2 = 0.999f;
  u.eps = 1e-8f;
  u.c1 = (float)(1.0 - std::pow(0.9, (double)s->adam_t));
  u.c2 = (float)(1.0 - std::pow(0.999, (double)s->adam_t));
  HC(update(u, s->stream));
  return LBM_OK;
}

PackArgs pack_args(surr_net* s, float* packed) {
  PackArgs a{};
  a.packed = packed;
  for (int l = 0; l < NL; ++l) {
    a.p[l] = s->at<float>(s->S.p[l]);
    a.m1[l] = s->at<float>(s->S.m1[l]);
    a.m2[l] = s->at<float>(s->S.m2[l]);
    a.wf[l] = s->at<__bf16>(s->S.wf[l]);
    a.wt[l] = s->at<__bf16>(s->S.wt[l]);
  }
  return a;
}

}  // namespace

extern "C" {

lbm_status surr_workspace_bytes(int32_t max_batch, int32_t max_data, size_t* bytes) {
  if (!bytes || max_batch < 1 || max_batch > 65536 || max_data < 0 || max_data > (1 << 24))
    return fail(LBM_EINVAL, "bad surrogate sizes");
  *bytes = slayout(max_batch, max_data).total;
  return LBM_OK;
}

lbm_status surr_init(const double* lo, const double* hi, int32_t max_batch, int32_t max_data,
                     void* stream, void* workspace, size_t ws_bytes, surr_net** out) {
  if (!out || !lo || !hi) return fail(LBM_EINVAL, "NULL argument");
  *out = nullptr;
  size_t need = 0;
  lbm_status st = surr_workspace_bytes(max_batch, max_data, &need);
  if (st != LBM_OK) return st;
  if (!workspace || ((uintptr_t)workspace & 255u)) return fail(LBM_EINVAL, "workspace must be 256-byte aligned");
  if (ws_bytes < need) return fail(LBM_EINVAL, "workspace too small: %zu < %zu", ws_bytes, need);
  for (int j = 0; j < NIN; ++j)
    if (!(hi[j] > lo[j]) || !std::isfinite(lo[j]) || !std::isfinite(hi[j]) || (j == 2 && !(lo[j] > 0)))
      return fail(LBM_EINVAL, "bad normalisation box for input %d", j);
  surr_net* s = new (std::nothrow) surr_net();
  if (!s) return fail(LBM_ENOMEM, "surrogate handle");
  s->S = slayout(max_batch, max_data);
  s->ws = (char*)workspace;
  s->stream = (hipStream_t)stream;
  s->n_data = 0;
  s->adam_t = 0;
  s->wsum = (float)NOUT;
  s->loss_dirty = false;
  float lof[NIN], hif[NIN], lw[NOUT];
  for (int j = 0; j < NIN; ++j) { lof[j] = (float)lo[j]; hif[j] = (float)hi[j]; }
  for (int j = 0; j < NOUT; ++j) lw[j] = 1.0f;
  hipError_t e = hipMemsetAsync(s->ws, 0, s->S.total, s->stream);
  if (e == hipSuccess) e = hipMemcpyAsync(s->ws + s->S.lo, lof, sizeof lof, hipMemcpyHostToDevice, s->stream);
  if (e == hipSuccess) e = hipMemcpyAsync(s->ws + s->S.hi, hif, sizeof hif, hipMemcpyHostToDevice, s->stream);
  if (e == hipSuccess) e = hipMemcpyAsync(s->ws + s->S.lw, lw, sizeof lw, hipMemcpyHostToDevice, s->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(s->stream);
  if (e != hipSuccess) { delete s; return fail(LBM_EDEVICE, "surrogate init: %s", hipGetErrorString(e)); }
  *out = s;
  return LBM_OK;
}

lbm_status surr_set_params(surr_net* s, const float* packed) {
  if (!s || !packed) return fail(LBM_EINVAL, "NULL argument");
  CallBuffer host;
  lbm_status st = host.take();
  if (st != LBM_OK) return st;
  memcpy(host->packed, packed, sizeof host->packed);
  HC(unpack_params(pack_args(s, host->packed), s->stream));
  if ((st = host.wait(s->stream)) != LBM_OK) return st;
  s->adam_t = 0;
  return LBM_OK;
}

lbm_status surr_get_params(surr_net* s, float* packed) {
  if (!s || !packed) return fail(LBM_EINVAL, "NULL argument");
  CallBuffer host;
  lbm_status st = host.take();
  if (st != LBM_OK) return st;
  HC(pack_params(pack_args(s, host->packed), s->stream));
  if ((st = host.wait(s->stream)) != LBM_OK) return st;
  memcpy(packed, host->packed, sizeof host->packed);
  return LBM_OK;
}

lbm_status surr_set_loss_weights(surr_net* s, const float* w) {
  if (!s || !w) return fail(LBM_EINVAL, "NULL argument");
  for (int j = 0; j < NOUT; ++j)
    if (!(w[j] >= 0.0f) || !std::isfinite(w[j])) return fail(LBM_EINVAL, "bad loss weight %d", j);
  HC(hipMemcpyAsync(s->ws + s->S.lw, w, NOUT * 4, hipMemcpyHostToDevice, s->stream));
  HC(hipStreamSynchronize(s->stream));
  s->wsum = 0.0f;
  for (int j = 0; j < NOUT; ++j) s->wsum += w[j];
  return LBM_OK;
}

lbm_status surr_set_data(surr_net* s, const float* x, const float* y, const float* row_w, int32_t n) {
  if (!s || !x || !y || n < 1 || n > s->S.max_data) return fail(LBM_EINVAL, "bad training data");
  std::vector<float> w(n, 1.0f);
  if (row_w)
    for (int i = 0; i < n; ++i) {
      if (!(row_w[i] >= 0.0f) || !std::isfinite(row_w[i])) return fail(LBM_EINVAL, "bad row weight %d", i);
      w[i] = row_w[i];
    }
  HC(hipMemcpyAsync(s->ws + s->S.X, x, (size_t)n * NIN * 4, hipMemcpyHostToDevice, s->stream));
  HC(hipMemcpyAsync(s->ws + s->S.Y, y, (size_t)n * NOUT * 4, hipMemcpyHostToDevice, s->stream));
  HC(hipMemcpyAsync(s->ws + s->S.RW, w.data(), (size_t)n * 4, hipMemcpyHostToDevice, s->stream));
  HC(hipStreamSynchronize(s->stream));
  s->n_data = n;
  return LBM_OK;
}

lbm_status surr_train_epoch(surr_net* s, const int32_t* perm, int32_t batch, float lr,
                            double* mean_loss) {
  if (!s || !perm) return fail(LBM_EINVAL, "NULL argument");
  if (s->n_data < 1) return fail(LBM_EINVAL, "no training data");
  if (batch < 1 || batch > s->S.Bp) return fail(LBM_EINVAL, "batch must be in [1, %d]", s->S.Bp);
  if (!(lr > 0.0f) || !std::isfinite(lr)) return fail(LBM_EINVAL, "bad learning rate");
  for (int i = 0; i < s->n_data; ++i)
    if (perm[i] < 0 || perm[i] >= s->n_data) return fail(LBM_EINVAL, "perm[%d] out of range", i);
  CallBuffer host;
  lbm_status st = host.take();
  if (st != LBM_OK) return st;
  HC(hipMemcpyAsync(s->ws + s->S.perm, perm, (size_t)s->n_data * 4, hipMemcpyHostToDevice, s->stream));
  if ((st = begin_loss(s)) != LBM_OK) return st;
  const float* X = s->at<float>(s->S.X);
  const float* Y = s->at<float>(s->S.Y);
  int nb = 0;
  for (int off = 0; off < s->n_data; off += batch, ++nb) {
    const int rows = std::min(batch, s->n_data - off);
    if ((st = sample_pass(s, X, Y, s->at<float>(s->S.RW), s->at<int32_t>(s->S.perm) + off, rows)) != LBM_OK)
      return st;
    if ((st = adam_step(s, rows, lr, off + rows >= s->n_data ? &host->loss : nullptr)) != LBM_OK) return st;
  }
  if ((st = end_loss(s, host)) != LBM_OK) return st;
  if (mean_loss) *mean_loss = host->loss / nb;
  return LBM_OK;
}

lbm_status surr_gradients(surr_net* s, const float* x, const float* y, int32_t n, float* grad,
                          double* loss_out) {
  if (!s || !x || !y || !grad || n < 1 || n > s->S.Bp) return fail(LBM_EINVAL, "bad arguments");
  CallBuffer host;
  lbm_status st = host.take();
  if (st != LBM_OK) return st;
  const float *X = host->x, *Y = host->y;
  if (n <= HOST_ROWS) {
    memcpy(host->x, x, (size_t)n * NIN * 4);
    memcpy(host->y, y, (size_t)n * NOUT * 4);
  } else {
    X = s->at<float>(s->S.qx);
    Y = s->at<float>(s->S.qy);
    HC(hipMemcpyAsync(s->ws + s->S.qx, x, (size_t)n * NIN * 4, hipMemcpyHostToDevice, s->stream));
    HC(hipMemcpyAsync(s->ws + s->S.qy, y, (size_t)n * NOUT * 4, hipMemcpyHostToDevice, s->stream));
  }
  if ((st = begin_loss(s)) != LBM_OK) return st;
  if ((st = sample_pass(s, X, Y, nullptr, nullptr, n)) != LBM_OK) return st;
  UpdateArgs u = update_args(s, n);
  u.packed = host->packed;
  u.loss_out = &host->loss;
  HC(update(u, s->stream));
  if ((st = end_loss(s, host)) != LBM_OK) return st;
  memcpy(grad, host->packed, sizeof host->packed);
  if (loss_out) *loss_out = host->loss;
  return LBM_OK;
}

lbm_status surr_predict(surr_net* s, const float* x, int32_t n, float* y) {
  if (!s || !x || !y || n < 0) return fail(LBM_EINVAL, "bad arguments");
  if (n == 0) return LBM_OK;
  // a chunk's answers may lie over the queries of later ones
  std::unique_ptr<float[]> own;
  if (n > HOST_ROWS && overlap(x, y, n)) {
    own.reset(new (std::nothrow) float[(size_t)n * NIN]);
    if (!own) return fail(LBM_ENOMEM, "copy of %d queries", n);
    memcpy(own.get(), x, (size_t)n * NIN * 4);
    x = own.get();
  }
  CallBuffer host;
  lbm_status st = host.take();
  if (st != LBM_OK) return st;
  for (int off = 0; off < n; off += HOST_ROWS) {
    const int rows = std::min(HOST_ROWS, n - off);
    memcpy(host->x, x + (size_t)off * NIN, (size_t)rows * NIN * 4);
    HC(predict(net_args(s), RowArgs{host->x, nullptr, rows}, host->y, s->stream));
    HC(hipStreamSynchronize(s->stream));
    memcpy(y + (size_t)off * NOUT, host->y, (size_t)rows * NOUT * 4);
  }
  host.done();
  return LBM_OK;
}

lbm_status surr_predict_noalloc(const surr_net* s, const float* x, int32_t n, float* y,
                                void* stream) {
  if (!s || !x || !y) return fail(LBM_EINVAL, "NULL argument");
  if (n < 1 || n > NOALLOC_ROWS)
    return fail(LBM_EINVAL, "surr_predict_noalloc takes 1..%d rows per call, got %d", NOALLOC_ROWS, n);
  const hipStream_t st = (hipStream_t)stream;
  int cur = 0, dev = 0;
  HC(hipGetDevice(&cur));
  dev = cur;
  if (st) HC(hipStreamGetDevice(st, &dev));
  if (dev != cur) return fail(LBM_EINVAL, "the stream's device %d is not the current device %d", dev, cur);
  HC(predict(net_args(s), RowArgs{x, nullptr, n}, y, st));
  return LBM_OK;
}

void surr_destroy(surr_net* s) { delete s; }

}  // extern "C"
