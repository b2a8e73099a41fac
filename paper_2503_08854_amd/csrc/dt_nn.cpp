// dt_nn.cpp -- the learned cell scorer: a small CNN over 21x21 coarse-stacked
// stamps plus an MLP over per-cell features, trained and evaluated entirely by
// this library's HIP kernels (BF16 MFMA products, FP32 master weights, Adam).
//
// Architecture (activations channels-last, weights [K, N] row-major with
// K = (ky * 3 + kx) * C_in + c_in for 3x3 convolutions, zero padding 1):
//   stamp 21x21x1 -> conv s1 (16) -> ReLU -> conv s2 (32) -> ReLU (11x11)
//                 -> conv s2 (32) -> ReLU (6x6) -> FC 1152->64 -> ReLU = h_img
//   features 16   -> FC 16->64 -> ReLU = h_feat
//   [h_img, h_feat] -> FC 128->64 -> ReLU -> FC 64->1 = logit
// Loss: mean binary cross-entropy of the logit.
#include "dt_internal.hpp"

namespace dtk {
namespace {

struct Layer {
  int64_t w, b;  // offsets in the parameter vector
  int K, N;      // weight shape [K, N]
};
// w1 b1 w2 b2 w3 b3 w4 b4 w5 b5 w6 b6 w7 b7
constexpr int NL = 7;
constexpr int LK[NL] = {9, 144, 288, 1152, 16, 128, 64};
constexpr int LN[NL] = {16, 32, 32, 64, 64, 64, 1};

int64_t layer_table(Layer* L) {
  int64_t off = 0;
  for (int i = 0; i < NL; ++i) {
    L[i].K = LK[i];
    L[i].N = LN[i];
    L[i].w = off;
    off += (int64_t)LK[i] * LN[i];
    L[i].b = off;
    off += LN[i];
  }
  return off;
}

}  // namespace
}  // namespace dtk

using namespace dtk;

struct dt_scorer {
  dt_ctx* ctx = nullptr;
  int max_b = 0;
  Layer L[NL];
  int64_t np = 0;
  int64_t step = 0;
  std::vector<std::pair<void*, size_t>> allocs;
  float *w = nullptr, *m = nullptr, *v = nullptr, *g = nullptr;
  uint16_t* wf = nullptr;  // BF16 weights in the order of the kernels' products
  float* z = nullptr;
  uint16_t *h3 = nullptr, *ft = nullptr, *cat = nullptr, *d4 = nullptr, *d5 = nullptr, *d6 = nullptr;
  float* records = nullptr;
};

namespace {

template <typename T>
dt_status salloc(dt_scorer* s, T** p, size_t count, const char* what) {
  dt_status st = ctx_alloc(s->ctx, (void**)p, sizeof(T) * count, what);
  if (st == DT_OK) s->allocs.push_back({(void*)*p, sizeof(T) * count});
  return st;
}

void sfree(dt_scorer* s) {
  for (auto& a : s->allocs) ctx_free(s->ctx, a.first, a.second);
  s->allocs.clear();
}

TrainArgs train_args(dt_scorer* s, const uint16_t* stamps, const uint16_t* feats, const float* labels, int B,
                     float* z) {
  return TrainArgs{stamps, feats, labels, B,     train_splits(B), s->w,  s->wf,     z,
                   s->h3,  s->ft, s->cat, s->d4, s->d5,           s->d6, s->records};
}

dt_status check_io(dt_scorer* s, const uint16_t* stamps, const uint16_t* feats, int B) {
  if (!s || !s->ctx) return fail(DT_E_ARG, "invalid scorer");
  if (B < 1 || B > s->max_b) return fail(DT_E_ARG, "batch %d outside [1, %d]", B, s->max_b);
  if (!stamps || !feats) return fail(DT_E_ARG, "NULL input");
  return DT_OK;
}

}  // namespace

extern "C" {

int64_t dt_scorer_num_params(void) {
  Layer L[NL];
  return layer_table(L);
}

dt_status dt_scorer_create(dt_ctx* c, int32_t max_batch, uint64_t seed, dt_scorer** out) {
  if (!out) return fail(DT_E_ARG, "out is NULL");
  *out = nullptr;
  if (!c || !c->alive) return fail(DT_E_ARG, "invalid context");
  if (max_batch < 1 || max_batch > 32768) return fail(DT_E_ARG, "max_batch must be in [1, 32768]");
  DeviceGuard guard(c->device);
  dt_scorer* s = new dt_scorer();
  s->ctx = c;
  s->max_b = max_batch;
  s->np = layer_table(s->L);
  const size_t B = (size_t)max_batch;
  dt_status st = DT_OK;
  auto A = [&](auto** p, size_t n, const char* what) {
    if (st == DT_OK) st = salloc(s, p, n, what);
  };
  A(&s->w, s->np, "scorer weights");
  A(&s->m, s->np, "scorer Adam m");
  A(&s->v, s->np, "scorer Adam v");
  A(&s->g, s->np, "scorer gradients");
  A(&s->wf, SCORER_FRAGS, "scorer BF16 weights");
  A(&s->z, B, "scorer logits");
  A(&s->h3, B * 1152, "scorer h3");
  A(&s->ft, B * 16, "scorer ft");
  A(&s->cat, B * 128, "scorer cat");
  A(&s->d4, B * 64, "scorer d4");
  A(&s->d5, B * 64, "scorer d5");
  A(&s->d6, B * 64, "scorer d6");
  A(&s->records, (size_t)train_groups(max_batch) * TRAIN_RECORD, "scorer gradient records");
  if (st != DT_OK) {
    sfree(s);
    delete s;
    return st;
  }
  hipError_t e = hipSuccess;
  for (int i = 0; i < NL && e == hipSuccess; ++i) {
    e = launch_init_params(s->w, s->L[i].w, (int64_t)s->L[i].K * s->L[i].N, s->L[i].K, seed, 0, c->stream);
    if (e == hipSuccess) e = launch_init_params(s->w, s->L[i].b, s->L[i].N, 1, seed, 1, c->stream);
  }
  if (e == hipSuccess) e = hipMemsetAsync(s->m, 0, sizeof(float) * s->np, c->stream);
  if (e == hipSuccess) e = hipMemsetAsync(s->v, 0, sizeof(float) * s->np, c->stream);
  if (e == hipSuccess) e = hipMemsetAsync(s->wf, 0, sizeof(uint16_t) * SCORER_FRAGS, c->stream);
  if (e == hipSuccess) e = launch_scorer_weights(s->w, s->wf, c->stream);
  if (e != hipSuccess) {
    sfree(s);
    delete s;
    return hip_fail(e, "scorer init");
  }
  *out = s;
  return DT_OK;
}

dt_status dt_scorer_destroy(dt_scorer* s) {
  if (!s || !s->ctx) return fail(DT_E_ARG, "invalid scorer");
  DeviceGuard guard(s->ctx->device);
  (void)hipStreamSynchronize(s->ctx->stream);
  sfree(s);
  s->ctx = nullptr;
  delete s;
  return DT_OK;
}

dt_status dt_scorer_get_params(dt_scorer* s, float* d_out) {
  if (!s || !s->ctx || !d_out) return fail(DT_E_ARG, "invalid scorer or NULL output");
  DeviceGuard guard(s->ctx->device);
  hipError_t e = hipMemcpyAsync(d_out, s->w, sizeof(float) * s->np, hipMemcpyDeviceToDevice, s->ctx->stream);
  return e == hipSuccess ? DT_OK : hip_fail(e, "scorer params copy");
}

dt_status dt_scorer_set_params(dt_scorer* s, const float* d_in) {
  if (!s || !s->ctx || !d_in) return fail(DT_E_ARG, "invalid scorer or NULL input");
  DeviceGuard guard(s->ctx->device);
  hipStream_t st = s->ctx->stream;
  hipError_t e = hipMemcpyAsync(s->w, d_in, sizeof(float) * s->np, hipMemcpyDeviceToDevice, st);
  if (e == hipSuccess) e = hipMemsetAsync(s->m, 0, sizeof(float) * s->np, st);
  if (e == hipSuccess) e = hipMemsetAsync(s->v, 0, sizeof(float) * s->np, st);
  if (e == hipSuccess) e = launch_scorer_weights(s->w, s->wf, st);
  s->step = 0;
  return e == hipSuccess ? DT_OK : hip_fail(e, "scorer set params");
}

dt_status dt_scorer_forward(dt_scorer* s, const uint16_t* d_stamps, const uint16_t* d_feats, int32_t B,
                            float* d_logits) {
  dt_status st = check_io(s, d_stamps, d_feats, B);
  if (st != DT_OK) return st;
  if (!d_logits) return fail(DT_E_ARG, "NULL logits");
  DeviceGuard guard(s->ctx->device);
  hipError_t e = launch_train_forward(train_args(s, d_stamps, d_feats, nullptr, B, d_logits), s->ctx->stream);
  return e == hipSuccess ? DT_OK : hip_fail(e, "scorer forward");
}

dt_status dt_scorer_infer(dt_scorer* s, const uint16_t* d_stamps, const uint16_t* d_feats, int32_t B,
                          float* d_logits) {
  return dt_scorer_infer_rows(s, d_stamps, d_feats, nullptr, B, d_logits);
}

dt_status dt_scorer_infer_rows(dt_scorer* s, const uint16_t* d_stamps, const uint16_t* d_feats,
                               const int64_t* d_rows, int32_t B, float* d_logits) {
  if (!s || !s->ctx) return fail(DT_E_ARG, "invalid scorer");
  if (B < 0) return fail(DT_E_ARG, "B < 0");
  if (B == 0) return DT_OK;
  if (!d_stamps || !d_feats || !d_logits) return fail(DT_E_ARG, "NULL input or output");
  DeviceGuard guard(s->ctx->device);
  ScorerFusedArgs a{};
  a.stamps = d_stamps;
  a.feats = d_feats;
  a.B = B;
  a.w = s->w;
  for (int i = 0; i < NL; ++i) a.b_off[i] = s->L[i].b;
  a.wf = s->wf;
  a.z = d_logits;
  a.rows = d_rows;
  hipError_t e = launch_scorer_fused(a, s->ctx->stream);
  return e == hipSuccess ? DT_OK : hip_fail(e, "scorer inference");
}

dt_status dt_scorer_grad(dt_scorer* s, const uint16_t* d_stamps, const uint16_t* d_feats, const float* d_labels,
                         int32_t B, float* d_loss, float* d_grad) {
  dt_status st = check_io(s, d_stamps, d_feats, B);
  if (st != DT_OK) return st;
  if (!d_labels) return fail(DT_E_ARG, "NULL labels");
  DeviceGuard guard(s->ctx->device);
  hipError_t e = launch_train_grad(train_args(s, d_stamps, d_feats, d_labels, B, s->z), d_loss,
                                   d_grad ? d_grad : s->g, nullptr, s->ctx->stream);
  return e == hipSuccess ? DT_OK : hip_fail(e, "scorer gradient");
}

dt_status dt_scorer_train_step(dt_scorer* s, const uint16_t* d_stamps, const uint16_t* d_feats,
                               const float* d_labels, int32_t B, float lr, float* d_loss) {
  dt_status st = check_io(s, d_stamps, d_feats, B);
  if (st != DT_OK) return st;
  if (!d_labels || !(lr > 0.f)) return fail(DT_E_ARG, "NULL labels or non-positive learning rate");
  DeviceGuard guard(s->ctx->device);
  ++s->step;
  const AdamArgs adam{s->w, s->m,   s->v,   s->wf, lr, 0.9f, 0.999f, 1e-8f, (float)(1.0 - pow(0.9, (double)s->step)),
                      (float)(1.0 - pow(0.999, (double)s->step))};
  hipError_t e = launch_train_grad(train_args(s, d_stamps, d_feats, d_labels, B, s->z), d_loss,
                                   nullptr, &adam, s->ctx->stream);
  return e == hipSuccess ? DT_OK : hip_fail(e, "scorer train step");
}

}  // extern "C"
