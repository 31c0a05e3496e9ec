// Host side of the warm-start network entry points (include/nmf.h): parameter
// blob layout, batched forward, loss/gradient of one batch through the
// library's own backward kernels, Adam, and minibatch training.
#include <algorithm>
#include <cstring>
#include <random>
#include <vector>

#include "plan_impl.hpp"

using namespace plnmf;

namespace {

nmf_mlp_layout layout_of(int K, int H) {
  nmf_mlp_layout L{};
  const size_t nm = (size_t)H * K + H + (size_t)K * H + K;
  Carver c(nullptr);
  L.n_master = nm;
  c.take<float>(nm);
  L.master = 0;
  L.adam_m = align_up(c.off);
  c.take<float>(nm);
  L.adam_v = align_up(c.off);
  c.take<float>(nm);
  L.w1_bf16 = align_up(c.off);
  c.take<__bf16>((size_t)H * K);
  L.w2_bf16 = align_up(c.off);
  c.take<__bf16>((size_t)K * H);
  L.step = align_up(c.off);
  c.take<int64_t>(1);
  L.total = align_up(c.off);
  return L;
}

struct Params {
  float *W1, *b1, *W2, *b2;  // masters
  float *m, *v;
  __bf16 *W1b, *W2b;
  int64_t* step;
  size_t n;
};

Params view(void* blob, int K, int H) {
  const nmf_mlp_layout L = layout_of(K, H);
  char* b = (char*)blob;
  Params p;
  p.W1 = (float*)(b + L.master);
  p.b1 = p.W1 + (size_t)H * K;
  p.W2 = p.b1 + H;
  p.b2 = p.W2 + (size_t)K * H;
  p.m = (float*)(b + L.adam_m);
  p.v = (float*)(b + L.adam_v);
  p.W1b = (__bf16*)(b + L.w1_bf16);
  p.W2b = (__bf16*)(b + L.w2_bf16);
  p.step = (int64_t*)(b + L.step);
  p.n = L.n_master;
  return p;
}

struct Ws {
  __bf16* xb;
  float* z1;
  __bf16* gb;
  __bf16* dz2b;
  __bf16* dz1b;
  float* partial;   // split sums of gW2, then of gW1
  int max_splits;
  double* red;      // loss per tile
  double* scal;
  double* col2;     // column sums per tile of rows
  double* col1;
  float* grads;
  float* xbat;
  float* ybat;
  int32_t* idx;
  size_t off;
};

// splits of the weight-gradient products (K x H and H x K) the workspace holds:
// it never shrinks as the batch grows, which batch_of relies on
int splits_for(int64_t B) { return (int)std::max<int64_t>(1, std::min<int64_t>(B / 64, 16)); }

constexpr int64_t kTileRowsMin = 64;  // rows of the smallest GEMM tile

Ws ws_layout(void* base, int K, int H, int64_t B) {
  Carver c(base);
  Ws w;
  w.xb = c.take<__bf16>((size_t)(B * K));
  w.z1 = c.take<float>((size_t)(B * H));
  w.gb = c.take<__bf16>((size_t)(B * H));
  w.dz2b = c.take<__bf16>((size_t)(B * K));
  w.dz1b = c.take<__bf16>((size_t)(B * H));
  w.max_splits = splits_for(B);
  w.partial = c.take<float>((size_t)2 * w.max_splits * K * H);
  const int64_t mt = (B + kTileRowsMin - 1) / kTileRowsMin;
  w.red = c.take<double>((size_t)(mt * ((K + 31) / 32)));
  w.scal = c.take<double>(8);
  w.col2 = c.take<double>((size_t)(mt * K));
  w.col1 = c.take<double>((size_t)(mt * H));
  w.grads = c.take<float>((size_t)H * K + H + (size_t)K * H + K);
  w.xbat = c.take<float>((size_t)(B * K));
  w.ybat = c.take<float>((size_t)(B * K));
  w.idx = c.take<int32_t>((size_t)B);
  c.take<char>(kAlign);
  w.off = c.off;
  return w;
}

// largest batch the workspace holds
int64_t batch_of(int K, int H, size_t bytes) {
  const size_t f0 = ws_layout(nullptr, K, H, 1).off;
  if (bytes < f0) return 0;
  int64_t lo = 1, hi = 1;
  while (ws_layout(nullptr, K, H, hi * 2).off <= bytes && hi < ((int64_t)1 << 40)) hi *= 2;
  hi *= 2;
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) / 2;
    if (ws_layout(nullptr, K, H, mid).off <= bytes) lo = mid; else hi = mid;
  }
  return lo;
}

int check_dims(int K, int H) {
  if (K < 1 || K > NMF_MAX_K || H < 1 || H > 4096)
    return fail(NMF_E_SHAPE, "network dims K=%d hidden=%d out of range", K, H);
  return NMF_OK;
}

#define MLPCHECK(expr)                                                                    \
  do {                                                                                    \
    hipError_t e_ = (expr);                                                               \
    if (e_ != hipSuccess) return fail(NMF_E_HIP, "%s failed: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

hipError_t refresh(const Params& p, int K, int H, hipStream_t s) {
  hipError_t e = cast_bf16(p.W1, p.W1b, (int64_t)H * K, s);
  if (e != hipSuccess) return e;
  return cast_bf16(p.W2, p.W2b, (int64_t)K * H, s);
}

// loss (device scal[0], sum over b*K) and gradients of b rows into `grads`
int loss_grad_rows(const Params& p, int K, int H, const float* X, const float* Y, int64_t b,
                   float* grads, const Ws& w, hipStream_t s) {
  MLPCHECK(cast_bf16(X, w.xb, b * K, s));
  GemmArgs g{};
  g.A = w.xb;
  g.lda = K;
  g.B = p.W1b;  // B(k,j) = W1[j*K + k]
  g.ldb = K;
  g.M = b;
  g.N = H;
  g.Kd = K;
  g.C = w.z1;
  g.ldc = H;
  g.epi = EPI_BIAS_GELU;
  g.bias = p.b1;
  g.C2 = w.gb;
  gemm_use(g, Elem::BF16, 1);
  MLPCHECK(gemm(Elem::BF16, false, true, g, s));
  // the output layer, its loss and dz2 = 2 / (b K) (yhat - y) softplus'(z2)
  GemmArgs g2{};
  g2.A = w.gb;
  g2.lda = H;
  g2.B = p.W2b;  // B(j,k) = W2[k*H + j]
  g2.ldb = H;
  g2.M = b;
  g2.N = K;
  g2.Kd = H;
  g2.ldc = K;
  g2.epi = EPI_OUT_GRAD;
  g2.bias = p.b2;
  g2.D = Y;
  g2.ldd = K;
  g2.C2 = w.dz2b;
  g2.scale = (float)(2.0 / (double)(b * K));
  g2.red_out = w.red;
  g2.col_part = w.col2;
  gemm_use(g2, Elem::BF16, 1);
  MLPCHECK(gemm(Elem::BF16, false, true, g2, s));
  float* gW1 = grads;
  float* gb1 = gW1 + (size_t)H * K;
  float* gW2 = gb1 + H;
  float* gb2 = gW2 + (size_t)K * H;
  // gW2 [K,H] = dz2^T g (split sums added by mlp_finish)
  GemmArgs a{};
  a.A = w.dz2b;  // A(k, r) = dz2[r*K + k]
  a.lda = K;
  a.B = w.gb;    // B(r, j) = g[r*H + j]
  a.ldb = H;
  a.M = K;
  a.N = H;
  a.Kd = b;
  a.ldc = H;
  a.epi = EPI_STORE;
  gemm_use(a, Elem::BF16, w.max_splits);
  a.C = a.splits > 1 ? nullptr : gW2;
  a.partial = w.partial;
  MLPCHECK(gemm(Elem::BF16, true, false, a, s));
  // dz1 [b,H] = (dz2 W2) * GELU'(z1)
  GemmArgs d{};
  d.A = w.dz2b;
  d.lda = K;
  d.B = p.W2b;  // B(k, j) = W2[k*H + j]
  d.ldb = H;
  d.M = b;
  d.N = H;
  d.Kd = K;
  d.ldc = H;
  d.epi = EPI_GELU_GRAD;
  d.D = w.z1;
  d.ldd = H;
  d.C2 = w.dz1b;
  d.col_part = w.col1;
  gemm_use(d, Elem::BF16, 1);
  MLPCHECK(gemm(Elem::BF16, false, false, d, s));
  // gW1 [H,K] = dz1^T x
  GemmArgs c{};
  c.A = w.dz1b;  // A(j, r) = dz1[r*H + j]
  c.lda = H;
  c.B = w.xb;    // B(r, k) = x[r*K + k]
  c.ldb = K;
  c.M = H;
  c.N = K;
  c.Kd = b;
  c.ldc = K;
  c.epi = EPI_STORE;
  gemm_use(c, Elem::BF16, w.max_splits);
  c.C = c.splits > 1 ? nullptr : gW1;
  c.partial = w.partial + (size_t)w.max_splits * K * H;
  MLPCHECK(gemm(Elem::BF16, true, false, c, s));
  MlpFinish f{};
  f.part2 = a.splits > 1 ? a.partial : nullptr;
  f.part1 = c.splits > 1 ? c.partial : nullptr;
  f.splits2 = a.splits;
  f.splits1 = c.splits;
  f.n = (int64_t)K * H;
  f.gW2 = gW2;
  f.gW1 = gW1;
  f.col2 = w.col2;
  f.col1 = w.col1;
  f.tiles2 = (int)((b + gemm_tile_rows(g2.cfg) - 1) / gemm_tile_rows(g2.cfg));
  f.tiles1 = (int)((b + gemm_tile_rows(d.cfg) - 1) / gemm_tile_rows(d.cfg));
  f.K = K;
  f.H = H;
  f.gb2 = gb2;
  f.gb1 = gb1;
  f.red = w.red;
  f.n_red = f.tiles2 * ((K + gemm_tile_cols(g2.cfg) - 1) / gemm_tile_cols(g2.cfg));
  f.loss = w.scal;
  MLPCHECK(mlp_finish(f, s));
  return NMF_OK;
}

}  // namespace

namespace plnmf {
// used by fold-in: forward over N rows in workspace-sized batches
// Inference needs only the BF16 input and hidden activations (no FP32
// pre-activations, no backward buffers): about (K + H) * 2 bytes per row.
struct WsI {
  __bf16* xb;  // [B, K]
  __bf16* gb;  // [B, H]
  size_t off;
};
WsI ws_infer_layout(void* base, int K, int H, int64_t B) {
  Carver c(base);
  WsI w;
  w.xb = c.take<__bf16>((size_t)(B * K));
  w.gb = c.take<__bf16>((size_t)(B * H));
  c.take<char>(kAlign);
  w.off = c.off;
  return w;
}
int64_t batch_infer_of(int K, int H, size_t bytes) {
  const size_t per = ws_infer_layout(nullptr, K, H, 2).off - ws_infer_layout(nullptr, K, H, 1).off;
  const size_t f0 = ws_infer_layout(nullptr, K, H, 1).off;
  if (bytes < f0) return 0;
  int64_t b = 1 + (int64_t)((bytes - f0) / std::max<size_t>(per, 1));
  while (b > 1 && ws_infer_layout(nullptr, K, H, b).off > bytes) b--;
  return b;
}

int mlp_forward_impl(const void* params, int K, int H, const float* X, float* Y, int64_t N,
                     void* ws, size_t bytes, hipStream_t s) {
  const int64_t B = batch_infer_of(K, H, bytes);
  if (B < 1) return fail(NMF_E_WORKSPACE, "network workspace too small");
  const WsI w = ws_infer_layout(ws, K, H, B);
  const Params p = view((void*)params, K, H);
  for (int64_t r = 0; r < N; r += B) {
    const int64_t b = std::min(B, N - r);
    MLPCHECK(cast_bf16(X + r * K, w.xb, b * K, s));
    GemmArgs g{};
    g.A = w.xb;
    g.lda = K;
    g.B = p.W1b;  // B(k,j) = W1[j*K + k]
    g.ldb = K;
    g.M = b;
    g.N = H;
    g.Kd = K;
    g.epi = EPI_BIAS_GELU;  // the pre-activation (C) is not kept
    g.bias = p.b1;
    g.C2 = w.gb;
    g.ldc = H;
    gemm_use(g, Elem::BF16, 1);
    MLPCHECK(gemm(Elem::BF16, false, true, g, s));
    GemmArgs g2{};
    g2.A = w.gb;
    g2.lda = H;
    g2.B = p.W2b;  // B(j,k) = W2[k*H + j]
    g2.ldb = H;
    g2.M = b;
    g2.N = K;
    g2.Kd = H;
    g2.epi = EPI_BIAS_SOFTPLUS;
    g2.bias = p.b2;
    g2.C2 = Y + r * K;
    g2.ldc = K;
    gemm_use(g2, Elem::BF16, 1);
    MLPCHECK(gemm(Elem::BF16, false, true, g2, s));
  }
  return NMF_OK;
}
size_t mlp_ws_bytes(int K, int H, int64_t B) { return ws_infer_layout(nullptr, K, H, B).off; }

// The warm start of fold-in: Ht_new = max(eps, ||r|| mlp(r / ||r||)) per row r of
// R.  One fused kernel where the shape allows it, else normalisation, the two
// GEMMs and the rescaling as separate launches (xn, norms, y: [N, K], [N],
// [N, K] scratch for that route).
int mlp_warm_start(const void* params, int K, int H, const float* R, int64_t N, float eps,
                   float* out, float* xn, float* norms, float* y, void* ws, size_t bytes,
                   hipStream_t s) {
  if (mlp_infer_fused_ok(K, H)) {
    const Params p = view((void*)params, K, H);
    MLPCHECK(mlp_infer_fused(R, N, K, H, p.W1b, p.b1, p.W2b, p.b2, eps, out, s));
    return NMF_OK;
  }
  MLPCHECK(row_normalize(R, N, K, xn, norms, s));
  int rc = mlp_forward_impl(params, K, H, xn, y, N, ws, bytes, s);
  if (rc) return rc;
  MLPCHECK(rescale_clip_rows(y, norms, N, K, eps, out, s));
  return NMF_OK;
}
}  // namespace plnmf

extern "C" {

int nmf_mlp_param_bytes(int K, int hidden, nmf_mlp_layout* layout) {
  if (!layout) return fail(NMF_E_ARG, "layout is NULL");
  int rc = check_dims(K, hidden);
  if (rc) return rc;
  *layout = layout_of(K, hidden);
  return NMF_OK;
}

int nmf_mlp_init(void* params, int K, int hidden, uint64_t seed, void* stream) {
  int rc = check_dims(K, hidden);
  if (rc) return rc;
  if (!params || ((uintptr_t)params % kAlign)) return fail(NMF_E_ARG, "params must be 256-byte aligned");
  hipStream_t s = (hipStream_t)stream;
  const Params p = view(params, K, hidden);
  MLPCHECK(mlp_init_params(p.W1, (int64_t)p.n, K, hidden, seed, s));
  MLPCHECK(hipMemsetAsync(p.m, 0, p.n * sizeof(float), s));
  MLPCHECK(hipMemsetAsync(p.v, 0, p.n * sizeof(float), s));
  MLPCHECK(hipMemsetAsync(p.step, 0, sizeof(int64_t), s));
  MLPCHECK(refresh(p, K, hidden, s));
  return NMF_OK;
}

int nmf_mlp_refresh(void* params, int K, int hidden, void* stream) {
  int rc = check_dims(K, hidden);
  if (rc) return rc;
  if (!params || ((uintptr_t)params % kAlign)) return fail(NMF_E_ARG, "params must be 256-byte aligned");
  hipStream_t s = (hipStream_t)stream;
  const Params p = view(params, K, hidden);
  MLPCHECK(hipMemsetAsync(p.m, 0, p.n * sizeof(float), s));
  MLPCHECK(hipMemsetAsync(p.v, 0, p.n * sizeof(float), s));
  MLPCHECK(hipMemsetAsync(p.step, 0, sizeof(int64_t), s));
  MLPCHECK(refresh(p, K, hidden, s));
  return NMF_OK;
}

int nmf_mlp_workspace_bytes(int K, int hidden, int64_t batch, size_t* bytes) {
  int rc = check_dims(K, hidden);
  if (rc) return rc;
  if (!bytes || batch < 1) return fail(NMF_E_ARG, "bad batch or NULL bytes");
  *bytes = ws_layout(nullptr, K, hidden, batch).off;
  return NMF_OK;
}

int nmf_mlp_predict(const void* params, int K, int hidden, const float* X, float* Yhat, int64_t N,
                    void* workspace, size_t workspace_bytes, void* stream) {
  int rc = check_dims(K, hidden);
  if (rc) return rc;
  if (!params || !X || !Yhat || !workspace) return fail(NMF_E_ARG, "NULL argument");
  if (N < 0) return fail(NMF_E_ARG, "N < 0");
  return mlp_forward_impl(params, K, hidden, X, Yhat, N, workspace, workspace_bytes,
                          (hipStream_t)stream);
}

int nmf_mlp_loss_grad(const void* params, int K, int hidden, const float* X, const float* Y,
                      int64_t N, float* grads, double* loss, void* workspace,
                      size_t workspace_bytes, void* stream) {
  int rc = check_dims(K, hidden);
  if (rc) return rc;
  if (!params || !X || !Y || !grads || !workspace) return fail(NMF_E_ARG, "NULL argument");
  const int64_t B = batch_of(K, hidden, workspace_bytes);
  if (N < 1 || N > B) return fail(NMF_E_WORKSPACE, "batch of %lld rows exceeds the workspace (%lld)",
                                  (long long)N, (long long)B);
  hipStream_t s = (hipStream_t)stream;
  const Ws w = ws_layout(workspace, K, hidden, B);
  const Params p = view((void*)params, K, hidden);
  rc = loss_grad_rows(p, K, hidden, X, Y, N, grads, w, s);
  if (rc) return rc;
  if (loss) {
    double v = 0.0;
    MLPCHECK(hipMemcpyAsync(&v, w.scal, sizeof(double), hipMemcpyDeviceToHost, s));
    MLPCHECK(hipStreamSynchronize(s));
    *loss = v / (double)(N * K);
  }
  return NMF_OK;
}

int nmf_mlp_adam_step(void* params, int K, int hidden, const float* grads, float lr, void* stream) {
  int rc = check_dims(K, hidden);
  if (rc) return rc;
  if (!params || !grads) return fail(NMF_E_ARG, "NULL argument");
  hipStream_t s = (hipStream_t)stream;
  const Params p = view(params, K, hidden);
  MLPCHECK(mlp_adam(p.W1, p.m, p.v, grads, K, hidden, lr, p.W1b, p.W2b, p.step, s));
  return NMF_OK;
}

int nmf_mlp_train(void* params, int K, int hidden, const float* X, const float* Y, int64_t N,
                  int epochs, int batch, float lr, uint64_t seed, void* workspace,
                  size_t workspace_bytes, double* epoch_loss, void* stream) {
  int rc = check_dims(K, hidden);
  if (rc) return rc;
  if (!params || !X || !Y || !workspace) return fail(NMF_E_ARG, "NULL argument");
  if (N < 1 || epochs < 0 || batch < 1) return fail(NMF_E_ARG, "bad N, epochs or batch");
  const int64_t B = batch_of(K, hidden, workspace_bytes);
  if (batch > B) return fail(NMF_E_WORKSPACE, "batch %d exceeds the workspace (%lld)", batch,
                             (long long)B);
  hipStream_t s = (hipStream_t)stream;
  const Ws w = ws_layout(workspace, K, hidden, B);
  const Params p = view(params, K, hidden);
  std::vector<int32_t> perm((size_t)N);
  for (int64_t i = 0; i < N; i++) perm[(size_t)i] = (int32_t)i;
  std::mt19937_64 rng(seed);
  for (int ep = 0; ep < epochs; ep++) {
    for (int64_t i = N - 1; i > 0; i--) {  // Fisher-Yates
      const int64_t j = (int64_t)(rng() % (uint64_t)(i + 1));
      std::swap(perm[(size_t)i], perm[(size_t)j]);
    }
    MLPCHECK(hipMemsetAsync(w.scal + 1, 0, sizeof(double), s));
    int64_t nbatches = 0;
    for (int64_t r = 0; r < N; r += batch) {
      const int64_t b = std::min<int64_t>(batch, N - r);
      MLPCHECK(hipMemcpyAsync(w.idx, perm.data() + r, (size_t)b * sizeof(int32_t),
                              hipMemcpyHostToDevice, s));
      MLPCHECK(gather_rows(X, w.idx, b, K, w.xbat, s));
      MLPCHECK(gather_rows(Y, w.idx, b, K, w.ybat, s));
      rc = loss_grad_rows(p, K, hidden, w.xbat, w.ybat, b, w.grads, w, s);
      if (rc) return rc;
      MLPCHECK(acc_scaled(w.scal + 1, w.scal, 1.0 / (double)(b * K), s));
      MLPCHECK(mlp_adam(p.W1, p.m, p.v, w.grads, K, hidden, lr, p.W1b, p.W2b, p.step, s));
      nbatches++;
    }
    // the index uploads read `perm`, which the next epoch reshuffles
    MLPCHECK(hipStreamSynchronize(s));
    if (epoch_loss) {
      double v = 0.0;
      MLPCHECK(hipMemcpyAsync(&v, w.scal + 1, sizeof(double), hipMemcpyDeviceToHost, s));
      MLPCHECK(hipStreamSynchronize(s));
      epoch_loss[ep] = v / (double)nbatches;
    }
  }
  return NMF_OK;
}

}  // extern "C"
