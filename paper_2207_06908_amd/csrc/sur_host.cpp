// sur_host.cpp -- host side of the surrogate library (C-ABI of include/sur.h).
//
// Owns the layer geometry, carves the caller's workspace into parameter,
// Adam, activation and gradient buffers, and sequences the kernels of
// sur_kernels.hip: forward (one product per layer with the bias/GELU
// epilogue; inference of every net in one fused launch where the widths
// allow), loss, backward (input-gradient product with the GELU-derivative
// epilogue; one launch with the forward pass where the widths allow), then
// weight and bias gradients with Adam in one launch.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <string>
#include <vector>

#include "sur.h"
#include "sur_dev.h"

using namespace mi355sur;

namespace {

constexpr int kMaxLayers = 7;

struct Layer {
  int k, kp, n;              // fan-in, fan-in padded to the product's K step, fan-out
  long long off_w, off_b;    // flat offsets
  long long w16, wt;         // element offsets of the bfloat16 copies inside a net's copy block
};

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

}  // namespace

struct sur_ctx {
  std::vector<int> w;
  int L = 0, nets = 0, R = 0, wmax = 0;
  hipStream_t stream = nullptr;
  std::string err;
  std::vector<Layer> lay;
  long long P = 0, nbf = 0;  // FP32 parameters per net, bfloat16 copy elements per net
  // workspace
  char* ws = nullptr;
  size_t ws_bytes = 0, need = 0;
  size_t o_net = 0, net_stride = 0, o_bf = 0;  // o_bf: offset of the copies inside a net block
  size_t o_X16 = 0, o_XT = 0, o_y = 0, o_part = 0, o_ys = 0;
  size_t o_a16[kMaxLayers] = {}, o_aT[kMaxLayers] = {}, o_gz[kMaxLayers] = {};
  size_t o_g16[2] = {}, o_gT = 0, o_dz = 0;
  std::vector<long long> adam_t;
  std::vector<char> ready;
  float xbound = INFINITY;   // routing bound on the inputs (sur_set_input_bound)
  int fused = 1;             // inference by the fused kernel where the widths allow (sur_set_kernel)

  template <typename T>
  T* at(size_t off) const { return (T*)(ws + off); }
  float* p(int net) const { return at<float>(o_net + net * net_stride); }
  float* m(int net) const { return p(net) + P; }
  float* v(int net) const { return p(net) + 2 * P; }
  float* g(int net) const { return p(net) + 3 * P; }
  uint16_t* bf(int net) const { return at<uint16_t>(o_net + net * net_stride + o_bf); }
};

static int fail(sur_ctx* c, int code, const std::string& msg) {
  if (c) c->err = msg;
  return code;
}

static int hip_fail(sur_ctx* c, int e, const char* what) {
  return fail(c, SUR_EDEVICE, std::string(what) + ": " + hipGetErrorString((hipError_t)e));
}

extern "C" {

int sur_create(const int* widths, int n_widths, int n_nets, int max_rows, void* hip_stream, sur_ctx** out) {
  if (!widths || !out || n_widths < 2 || n_widths > kMaxLayers + 1 || n_nets < 1 || n_nets > 16 ||
      max_rows < 64 || max_rows > 65536 || max_rows % 64)
    return SUR_EINVAL;
  if (widths[0] < 1 || widths[0] > 32) return SUR_EINVAL;
  for (int i = 1; i < n_widths; ++i)
    if (widths[i] < 64 || widths[i] > 4096 || widths[i] % 64) return SUR_EINVAL;
  sur_ctx* c = new sur_ctx;
  c->w.assign(widths, widths + n_widths);
  c->L = n_widths - 1;
  c->nets = n_nets;
  c->R = max_rows;
  c->stream = (hipStream_t)hip_stream;
  long long off = 0, bf = 0;
  for (int l = 0; l < c->L; ++l) {
    Layer y;
    y.k = c->w[l];
    y.kp = l == 0 ? 32 : c->w[l];
    y.n = c->w[l + 1];
    y.off_w = off;
    y.off_b = off + (long long)y.n * y.k;
    off = y.off_b + y.n;
    y.w16 = bf;
    y.wt = bf + (long long)y.n * y.kp;
    bf = y.wt + (long long)y.n * y.kp;
    c->lay.push_back(y);
    c->wmax = std::max(c->wmax, y.n);
  }
  c->P = off;
  c->nbf = bf;
  // workspace layout
  const size_t R = c->R, W = c->w.back();
  size_t o = 0;
  auto take = [&](size_t bytes) { const size_t r = o; o += align256(bytes); return r; };
  c->o_bf = align256((size_t)4 * c->P * 4);
  c->net_stride = align256(c->o_bf + (size_t)c->nbf * 2);
  c->o_net = take(c->net_stride * c->nets);
  c->o_X16 = take(R * 32 * 2);
  c->o_XT = take(R * 32 * 2);
  for (int l = 0; l + 1 < c->L; ++l) {
    const size_t n = c->lay[l].n;
    c->o_a16[l] = take(R * n * 2);
    c->o_aT[l] = take(R * n * 2);
    c->o_gz[l] = take(R * n * 4);
  }
  c->o_y = take(R * W * 4);
  for (int q = 0; q < 2; ++q) c->o_g16[q] = take(R * c->wmax * 2);
  c->o_gT = take(R * W * 2);
  c->o_dz = take(R * W * 4);
  c->o_part = take((size_t)loss_parts(c->R, (int)W) * 4);
  c->o_ys = take((size_t)c->nets * R * W * 4);
  c->need = o;
  c->adam_t.assign(c->nets, 0);
  c->ready.assign(c->nets, 0);
  *out = c;
  return SUR_OK;
}

size_t sur_workspace_bytes(const sur_ctx* c) { return c ? c->need : 0; }

int sur_bind_workspace(sur_ctx* c, void* dev, size_t bytes) {
  if (!c || !dev) return fail(c, SUR_EINVAL, "null workspace");
  if ((uintptr_t)dev % 256) return fail(c, SUR_EINVAL, "workspace must be 256-byte aligned");
  if (bytes < c->need) return fail(c, SUR_ENOMEM, "workspace smaller than sur_workspace_bytes()");
  c->ws = (char*)dev;
  c->ws_bytes = bytes;
  std::fill(c->ready.begin(), c->ready.end(), 0);
  return SUR_OK;
}

long long sur_num_params(const sur_ctx* c) { return c ? c->P : 0; }

static int check_net(sur_ctx* c, int net, bool need_ready) {
  if (!c) return SUR_EINVAL;
  if (net < 0 || net >= c->nets) return fail(c, SUR_EINVAL, "net index out of range");
  if (!c->ws) return fail(c, SUR_ESTATE, "no workspace bound");
  if (need_ready && !c->ready[net]) return fail(c, SUR_ESTATE, "parameters of this net were never set");
  return SUR_OK;
}

// Upload parameters, clear the Adam state and the bfloat16 copies (their
// padding columns must be zero), then rebuild the copies.
static int upload_params(sur_ctx* c, int net, const float* host) {
  hipError_t e = hipMemcpyAsync(c->p(net), host, (size_t)c->P * 4, hipMemcpyHostToDevice, c->stream);
  if (e == hipSuccess) e = hipMemsetAsync(c->m(net), 0, (size_t)c->P * 4 * 3, c->stream);
  if (e == hipSuccess) e = hipMemsetAsync(c->bf(net), 0, (size_t)c->nbf * 2, c->stream);
  if (e != hipSuccess) return hip_fail(c, e, "parameter upload");
  CopyArgs a{};
  a.p = c->p(net);
  a.bf = c->bf(net);
  a.P = (int)c->P;
  a.nl = c->L;
  for (int l = 0; l < c->L; ++l) {
    const Layer& y = c->lay[l];
    a.L[l] = CopyLayer{(int)y.off_w, y.n, y.k, y.kp, y.w16, y.wt};
  }
  const int r = launch_copies(a, c->stream);
  if (r) return hip_fail(c, r, "copy refresh");
  e = hipStreamSynchronize(c->stream);  // the host buffer may go away after return
  if (e != hipSuccess) return hip_fail(c, e, "parameter upload");
  c->adam_t[net] = 0;
  c->ready[net] = 1;
  return SUR_OK;
}

static uint64_t splitmix64(uint64_t x) {
  x += 0x9E3779B97F4A7C15ull;
  x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
  x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
  return x ^ (x >> 31);
}

int sur_init_params(sur_ctx* c, int net, unsigned long long seed) {
  int r = check_net(c, net, false);
  if (r) return r;
  std::vector<float> h((size_t)c->P);
  for (const Layer& y : c->lay) {
    const double bound = 1.0 / std::sqrt((double)y.k);
    for (long long i = y.off_w; i < y.off_b + y.n; ++i) {
      const uint64_t z = splitmix64(seed * 0xD1B54A32D192ED03ull + (uint64_t)i);
      const double u = (double)(z >> 11) * 0x1.0p-53;
      h[(size_t)i] = (float)((2.0 * u - 1.0) * bound);
    }
  }
  return upload_params(c, net, h.data());
}

int sur_set_params(sur_ctx* c, int net, const float* host) {
  int r = check_net(c, net, false);
  if (r) return r;
  if (!host) return fail(c, SUR_EINVAL, "null parameters");
  return upload_params(c, net, host);
}

static int download(sur_ctx* c, const float* dev, float* host) {
  if (!host) return fail(c, SUR_EINVAL, "null output");
  hipError_t e = hipMemcpyAsync(host, dev, (size_t)c->P * 4, hipMemcpyDeviceToHost, c->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
  if (e != hipSuccess) return hip_fail(c, e, "download");
  return SUR_OK;
}

int sur_get_params(sur_ctx* c, int net, float* host) {
  int r = check_net(c, net, true);
  return r ? r : download(c, c->p(net), host);
}

int sur_get_grads(sur_ctx* c, int net, float* host) {
  int r = check_net(c, net, true);
  return r ? r : download(c, c->g(net), host);
}

// Forward pass of rows already gathered into X16 (M rows, multiple of 64).
// train: keep every activation, its transpose and the GELU derivative.
static int forward(sur_ctx* c, int net, int M, bool train, float* y, int ldy, int m_valid) {
  const uint16_t* in = c->at<uint16_t>(c->o_X16);
  const uint16_t* bfb = c->bf(net);
  for (int l = 0; l < c->L; ++l) {
    const Layer& ly = c->lay[l];
    GemmArgs a{};
    a.A = in;
    a.lda = ly.kp;
    a.B = bfb + ly.w16;
    a.M = M;
    a.N = ly.n;
    a.K = ly.kp;
    a.bias = c->p(net) + ly.off_b;
    int epi;
    if (l + 1 < c->L) {
      epi = train ? EPI_GELU_TRAIN : EPI_GELU_INFER;
      a.o16 = c->at<uint16_t>(c->o_a16[l]);
      a.ld16 = ly.n;
      a.oT = c->at<uint16_t>(c->o_aT[l]);
      a.o32 = c->at<float>(c->o_gz[l]);
      in = a.o16;
    } else {
      epi = EPI_LINEAR;
      a.o32 = y;
      a.ld32 = ldy;
      a.m_valid = m_valid;
    }
    const int e = launch_gemm(epi, a, c->stream);
    if (e) return hip_fail(c, e, "forward product");
  }
  return SUR_OK;
}

// Whether the fused inference kernel takes this geometry: hidden widths up to
// MLP_KMAX, the output width up to MLP_NOUT.
static bool fused_ok(const sur_ctx* c) {
  if (!c->fused) return false;
  for (int l = 0; l < c->L; ++l) {
    const int n = c->lay[l].n;
    if (l + 1 < c->L ? n > MLP_KMAX : n > MLP_NOUT) return false;
  }
  return c->L <= 8;
}

// All layers of nets [net0, net0 + nets) over the m rows at x, in one launch;
// outputs to y[q ld_net + row W + col].
static int forward_fused(sur_ctx* c, int net0, int nets, const float* x, int m, float* y, long long ld_net) {
  MlpArgs a{};
  a.x = x;
  a.kin = c->w[0];
  a.bf = c->bf(net0);
  a.p = c->p(net0);
  a.bf_stride = (long long)(c->net_stride / 2);
  a.p_stride = (long long)(c->net_stride / 4);
  a.M = m;
  a.L = c->L;
  a.out = y;
  a.ld_net = ld_net;
  for (int l = 0; l < c->L; ++l) {
    const Layer& ly = c->lay[l];
    a.lay[l] = MlpLayer{ly.w16, (int)ly.off_b, ly.kp, ly.n};
  }
  const int e = launch_mlp_infer(a, nets, c->stream);
  return e ? hip_fail(c, e, "fused inference") : SUR_OK;
}

// dZ of layer l: transposed (over the layer's row-major activations, which
// only the forward product of the next layer reads) and FP32 (over its GELU
// derivatives).
static uint16_t* grad_t(const sur_ctx* c, int l) { return c->at<uint16_t>(l + 1 < c->L ? c->o_a16[l] : c->o_gT); }
static float* grad_32(const sur_ctx* c, int l) { return c->at<float>(l + 1 < c->L ? c->o_gz[l] : c->o_dz); }

// Whether one launch takes the step up to dZ of every layer: widths that fit
// its LDS buffers.  Rows do not matter (us a step, one launch / one per layer:
// 64 rows 59 / 81, 4096 102 / 176, 8192 224 / 318, 65536 1,655 / 2,015).
static bool fused_train_ok(const sur_ctx* c) { return fused_ok(c) && c->w.back() <= MLP_TOUT; }

int sur_train_step(sur_ctx* c, int net, const float* x_dev, const float* t_dev, const int* rows_dev, int batch,
                   float lr, int update, float* loss_dev) {
  int r = check_net(c, net, true);
  if (r) return r;
  if (!x_dev || !t_dev || batch < 1 || batch > c->R) return fail(c, SUR_EINVAL, "bad batch");
  if (!(lr >= 0.0f) || !std::isfinite(lr)) return fail(c, SUR_EINVAL, "bad learning rate");
  const int M = (batch + 63) / 64 * 64, W = c->w.back(), L = c->L;
  const double denom = (double)batch * W;
  const float scale = (float)(2.0 / denom);
  uint16_t* const XT = c->at<uint16_t>(c->o_XT);
  float* const part = c->at<float>(c->o_part);
  int e;
  if (fused_train_ok(c)) {
    TrainArgs a{};
    a.x = x_dev;
    a.t = t_dev;
    a.rows = rows_dev;
    a.bf = c->bf(net);
    a.p = c->p(net);
    a.M = M;
    a.m_valid = batch;
    a.kin = c->w[0];
    a.L = L;
    a.scale = scale;
    a.XT = XT;
    a.part = part;
    for (int l = 0; l < L; ++l) {
      const Layer& y = c->lay[l];
      a.lay[l] = TrainLayer{y.w16, y.wt, (int)y.off_b, y.kp, y.n, l + 1 < L ? c->at<uint16_t>(c->o_aT[l]) : nullptr,
                            grad_t(c, l), grad_32(c, l)};
    }
    if ((e = launch_mlp_train(a, c->stream))) return hip_fail(c, e, "forward and backward");
  } else {
    e = launch_gather(x_dev, rows_dev, batch, M, c->w[0], c->at<uint16_t>(c->o_X16), XT, c->stream);
    if (e) return hip_fail(c, e, "gather");
    if ((r = forward(c, net, M, true, c->at<float>(c->o_y), W, M))) return r;
    int cur = 0;
    e = launch_loss(c->at<float>(c->o_y), t_dev, rows_dev, M, batch, W, scale, c->at<uint16_t>(c->o_g16[cur]),
                    grad_t(c, L - 1), grad_32(c, L - 1), part, c->stream);
    if (e) return hip_fail(c, e, "loss");
    for (int l = L - 1; l > 0; --l) {  // dZ_{l-1} = (dZ_l W_l) * gelu'(Z_{l-1})
      const Layer& ly = c->lay[l];
      GemmArgs b{};
      b.A = c->at<uint16_t>(c->o_g16[cur]);
      b.lda = ly.n;
      b.B = c->bf(net) + ly.wt;
      b.M = M;
      b.N = ly.kp;
      b.K = ly.n;
      b.o16 = c->at<uint16_t>(c->o_g16[1 - cur]);
      b.ld16 = ly.kp;
      b.oT = grad_t(c, l - 1);
      b.o32 = grad_32(c, l - 1);
      if ((e = launch_gemm(EPI_BWD, b, c->stream))) return hip_fail(c, e, "input gradient");
      cur ^= 1;
    }
  }
  if (update) c->adam_t[net] += 1;
  DwArgs d{};
  d.p = c->p(net);
  d.m = c->m(net);
  d.v = c->v(net);
  d.g = c->g(net);
  d.bf = c->bf(net);
  d.M = M;
  d.nl = L;
  d.update = update ? 1 : 0;
  d.lr = lr;
  d.b1 = 0.9f;
  d.b2 = 0.999f;
  d.eps = 1e-8f;
  const double t = (double)c->adam_t[net];
  d.c1 = (float)(1.0 - std::pow(0.9, t));
  d.c2 = (float)(1.0 - std::pow(0.999, t));
  d.part = part;
  d.n_part = loss_parts(M, W);
  d.inv = (float)(1.0 / denom);
  d.loss = loss_dev;
  for (int l = 0; l < L; ++l) {
    const Layer& y = c->lay[l];
    d.L[l] = DwLayer{l ? c->at<uint16_t>(c->o_aT[l - 1]) : XT, grad_t(c, l), grad_32(c, l), (int)y.off_w, y.n, y.k,
                     y.kp, y.w16, y.wt, 0, 0};
  }
  if ((e = launch_dw_adam(d, c->stream))) return hip_fail(c, e, "weight gradients");
  return SUR_OK;
}

int sur_forward(sur_ctx* c, int net, const float* x_dev, int n, float* y_dev) {
  int r = check_net(c, net, true);
  if (r) return r;
  if (n < 0 || (n > 0 && (!x_dev || !y_dev))) return fail(c, SUR_EINVAL, "bad forward arguments");
  const int W = c->w.back(), k0 = c->w[0];
  // The blocks of the fused kernel read their inputs while others write
  // outputs: where the two share memory, a chunk's inputs are gathered first.
  const uintptr_t xa = (uintptr_t)x_dev, ya = (uintptr_t)y_dev;
  const bool apart = xa + (size_t)n * k0 * 4 <= ya || ya + (size_t)n * W * 4 <= xa;
  for (int c0 = 0; c0 < n; c0 += c->R) {
    const int m = std::min(c->R, n - c0), M = (m + 63) / 64 * 64;
    const float* x = x_dev + (size_t)c0 * k0;
    float* y = y_dev + (size_t)c0 * W;
    if (apart && fused_ok(c)) {
      if ((r = forward_fused(c, net, 1, x, m, y, 0))) return r;
      continue;
    }
    int e = launch_gather(x, nullptr, m, M, k0, c->at<uint16_t>(c->o_X16), nullptr, c->stream);
    if (e) return hip_fail(c, e, "gather");
    if ((r = forward(c, net, M, false, y, W, m))) return r;
  }
  return SUR_OK;
}

int sur_infer_route(sur_ctx* c, const float* x_dev, int n, float threshold, float* y_mean_dev, float* spread_dev,
                    int* fallback_dev, int* n_fallback_dev) {
  if (!c) return SUR_EINVAL;
  if (!c->ws) return fail(c, SUR_ESTATE, "no workspace bound");
  for (int q = 0; q < c->nets; ++q)
    if (!c->ready[q]) return fail(c, SUR_ESTATE, "parameters of a net were never set");
  if (n < 0 || !n_fallback_dev || (n > 0 && (!x_dev || !y_mean_dev || !spread_dev || !fallback_dev)))
    return fail(c, SUR_EINVAL, "bad routing arguments");
  const int W = c->w.back(), k0 = c->w[0];
  float* ys = c->at<float>(c->o_ys);
  int r;
  for (int c0 = 0; c0 < n; c0 += c->R) {
    const int m = std::min(c->R, n - c0), M = (m + 63) / 64 * 64;
    const float* x = x_dev + (size_t)c0 * k0;
    int e;
    if (fused_ok(c)) {
      if ((r = forward_fused(c, 0, c->nets, x, m, ys, (long long)c->R * W))) return r;
    } else {
      e = launch_gather(x, nullptr, m, M, k0, c->at<uint16_t>(c->o_X16), nullptr, c->stream);
      if (e) return hip_fail(c, e, "gather");
      for (int q = 0; q < c->nets; ++q)
        if ((r = forward(c, q, M, false, ys + (size_t)q * c->R * W, W, m))) return r;
    }
    if ((e = launch_route(ys, c->nets, c->R * W, m, W, x, k0, c->xbound,
                          y_mean_dev + (size_t)c0 * W, spread_dev + c0, c->stream)))
      return hip_fail(c, e, "route");
  }
  int e = launch_compact(spread_dev, n, threshold, fallback_dev, n_fallback_dev, c->stream);
  if (e) return hip_fail(c, e, "compact");
  return SUR_OK;
}

int sur_set_kernel(sur_ctx* c, int fused) {
  if (!c || (fused != 0 && fused != 1)) return fail(c, SUR_EINVAL, "kernel choice must be 0 or 1");
  c->fused = fused;
  return SUR_OK;
}

int sur_set_input_bound(sur_ctx* c, float bound) {
  if (!c) return SUR_EINVAL;
  if (!(bound > 0.0f)) return fail(c, SUR_EINVAL, "input bound must be positive (INFINITY: off)");
  c->xbound = bound;
  return SUR_OK;
}

const char* sur_last_error(const sur_ctx* c) { return c ? c->err.c_str() : "null handle"; }

void sur_destroy(sur_ctx* c) { delete c; }

}  // extern "C"
