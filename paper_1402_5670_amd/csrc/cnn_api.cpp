// C ABI of the learned-shrinkage network (declared in include/shearlet.h).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <string>

#include "../../include/shearlet.h"
#include "cnn.hpp"
#include "system.hpp"

namespace sl {
hipError_t render_cartoons(const float *shapes, int n, int H, int W, int max_shapes,
                           const float *sigma, uint64_t seed, float *clean, float *noisy,
                           hipStream_t st);
}

namespace {

using sl::kCnnParams;

constexpr size_t kPackLayer2 = 9 * 2 * 512;   // u16 per scale, two output blocks
constexpr size_t kPackLayer1 = 9 * 1 * 512;   // one output block
constexpr size_t kPackK1 = 2 * 512;             // layer 1, taps packed into K
constexpr int kErrBlocks = SL_SQERR_SCRATCH - 1;

size_t al(size_t v) { return (v + 255) / 256 * 256; }

struct Packed {
  const uint16_t *w1, *w2, *w3, *w2t, *w1k;
};

Packed packed_view(const void *base, int J) {
  const uint16_t *p = (const uint16_t *)base;
  Packed v;
  v.w1 = p;
  v.w2 = v.w1 + J * kPackLayer2;
  v.w3 = v.w2 + J * kPackLayer2;
  v.w2t = v.w3 + J * kPackLayer1;
  v.w1k = v.w2t + J * kPackLayer2;
  return v;
}

sl::CnnPlanes planes(const sl_system *s, int B, const float *sigma) {
  sl::CnnPlanes pl{};
  pl.R = s->R;
  pl.J = s->cfg.J;
  pl.B = B;
  pl.p0 = 0;
  int acc = 0;
  for (int j = 0; j < pl.J; ++j) {
    int n = 0, first = -1;
    for (int i = 1; i < s->R; ++i)
      if (s->subs[i].j == j) {
        if (first < 0) first = i;
        ++n;
      }
    pl.start[j] = acc;
    pl.nsub[j] = n;
    pl.first[j] = first < 0 ? 1 : first;
    acc += B * n;
  }
  pl.start[pl.J] = acc;
  pl.sigma = sigma;
  pl.l2 = s->d_l2;
  return pl;
}

size_t act_bytes(const sl_system *s, int planes) {
  return al((size_t)planes * (size_t)s->cfg.npix() * 32 * 2);
}

// SL_CNN_LAYERWISE=1 selects the layer-by-layer inference (activations in
// HBM) instead of the fused tile kernel; both compute the same network.
bool layerwise() {
  const char *e = std::getenv("SL_CNN_LAYERWISE");
  return e && std::atoi(e) != 0;
}

int apply_chunk(const sl_system *s, int B) {
  const int P = B * (s->R - 1);
  const char *env = std::getenv("SL_CNN_CHUNK_MB");
  const size_t cap = (size_t)(env ? std::max(1, std::atoi(env)) : 4096) << 20;
  const size_t per = 2 * (size_t)s->cfg.npix() * 32 * 2;
  return (int)std::max<size_t>(1, std::min<size_t>((size_t)P, cap / per));
}

int check(const sl_system *s, int B, const void *a, const void *b) {
  if (!s) return sl::set_error(SL_EINVAL, "system is NULL");
  if (B < 1 || B > 65535) return sl::set_error(SL_EINVAL, "batch must be in 1..65535");
  if (!a || !b) return sl::set_error(SL_EINVAL, "NULL buffer");
  if (s->cfg.dtype != SL_F32) return sl::set_error(SL_EINVAL, "the CNN needs SL_F32 coefficients");
  if (s->cfg.J > sl::kMaxScales) return sl::set_error(SL_EUNSUPPORTED, "too many scales");
  if (s->R < 2) return sl::set_error(SL_EINVAL, "no detail subbands");
  if (s->cfg.ndim != 2) return sl::set_error(SL_EUNSUPPORTED, "the CNN works on 2D systems");
  return SL_OK;
}

void plane_hw(const sl_system *s, int &H, int &W) {
  H = (int)s->cfg.dims[0];
  W = (int)s->cfg.dims[1];
}

#define CK(expr)                                                  \
  do {                                                            \
    hipError_t e_ = (expr);                                       \
    if (e_ != hipSuccess) return sl::hip_error(e_, #expr);        \
  } while (0)

}  // namespace

extern "C" {

size_t sl_cnn_packed_bytes(int J) {
  // w1, w2, w2t: two output blocks each; w3: one; w1k: packed layer 1
  if (J < 1) return 0;
  return (size_t)J * (3 * kPackLayer2 + kPackLayer1 + kPackK1) * sizeof(uint16_t);
}

int sl_cnn_pack(const float *params_dev, int J, void *packed_dev, void *stream) {
  if (!params_dev || !packed_dev || J < 1 || J > sl::kMaxScales)
    return sl::set_error(SL_EINVAL, "bad arguments to sl_cnn_pack");
  hipStream_t st = (hipStream_t)stream;
  uint16_t *base = (uint16_t *)packed_dev;
  Packed v = packed_view(packed_dev, J);
  CK(sl::cnn_pack(params_dev, J, 1, 0, base, 2, st));
  CK(sl::cnn_pack(params_dev, J, 2, 0, (uint16_t *)v.w2, 2, st));
  CK(sl::cnn_pack(params_dev, J, 3, 0, (uint16_t *)v.w3, 1, st));
  CK(sl::cnn_pack(params_dev, J, 2, 1, (uint16_t *)v.w2t, 2, st));
  CK(sl::cnn_pack(params_dev, J, 1, 2, (uint16_t *)v.w1k, 2, st));
  return SL_OK;
}

int sl_cnn_workspace_size(const sl_system *s, int batch, int training, size_t *bytes_out) {
  if (!s || !bytes_out || batch < 1) return sl::set_error(SL_EINVAL, "bad arguments");
  if (!training) {
    *bytes_out = layerwise() ? 2 * act_bytes(s, apply_chunk(s, batch)) : 256;
  } else {
    // one partial gradient per block of the backward kernel, which runs at
    // most one block per compute unit and one more per scale
    *bytes_out = al((size_t)(s->num_cu + s->cfg.J) * kCnnParams * sizeof(float));
  }
  return SL_OK;
}

int sl_cnn_apply(const sl_system *s, const float *params_dev, const void *packed_dev,
                 const float *coeffs_dev, const float *sigma_dev, int batch,
                 float *coeffs_out_dev, float *gains_dev, void *workspace_dev,
                 size_t workspace_bytes, void *stream) {
  int rc = check(s, batch, coeffs_dev, coeffs_out_dev);
  if (rc) return rc;
  if (!params_dev || !packed_dev || !sigma_dev || !workspace_dev)
    return sl::set_error(SL_EINVAL, "NULL argument");
  size_t need = 0;
  sl_cnn_workspace_size(s, batch, 0, &need);
  if (workspace_bytes < need)
    return sl::set_error(SL_ENOMEM, "workspace too small: need " + std::to_string(need));
  hipStream_t st = (hipStream_t)stream;
  int H, W;
  plane_hw(s, H, W);
  const int J = s->cfg.J, P = batch * (s->R - 1), Pc = apply_chunk(s, batch);
  Packed pk = packed_view(packed_dev, J);
  sl::CnnPlanes pl0 = planes(s, batch, sigma_dev);
  if (!layerwise()) {
    CK(sl::cnn_copy_lowpass(coeffs_dev, coeffs_out_dev, batch, s->R, (int)s->cfg.npix(), st));
    CK(sl::cnn_fused(coeffs_dev, pl0, P, H, W, pk.w1k, pk.w2, pk.w3, params_dev,
                     coeffs_out_dev, gains_dev, s->num_cu, st));
    return SL_OK;
  }
  uint16_t *A = (uint16_t *)workspace_dev;
  uint16_t *Bf = (uint16_t *)((char *)workspace_dev + act_bytes(s, Pc));
  sl::CnnPlanes pl = planes(s, batch, sigma_dev);
  CK(sl::cnn_copy_lowpass(coeffs_dev, coeffs_out_dev, batch, s->R, (int)s->cfg.npix(), st));
  for (int p0 = 0; p0 < P; p0 += Pc) {
    const int n = std::min(Pc, P - p0);
    pl.p0 = p0;
    CK(sl::cnn_x0(coeffs_dev, pl, n, H, W, A, st));
    CK(sl::cnn_conv(A, pk.w1, 2, params_dev + sl::kOffB1, kCnnParams, pl, n, H, W, sl::CONV_RELU,
                    Bf, nullptr, nullptr, nullptr, st));
    CK(sl::cnn_conv(Bf, pk.w2, 2, params_dev + sl::kOffB2, kCnnParams, pl, n, H, W, sl::CONV_RELU,
                    A, nullptr, nullptr, nullptr, st));
    CK(sl::cnn_conv(A, pk.w3, 1, params_dev + sl::kOffB3, kCnnParams, pl, n, H, W, sl::CONV_GAIN,
                    nullptr, coeffs_dev, coeffs_out_dev, gains_dev, st));
  }
  return SL_OK;
}

int sl_cnn_backward(const sl_system *s, const float *params_dev, const void *packed_dev,
                    const float *coeffs_dev, const float *sigma_dev, int batch,
                    const float *dcoeffs_dev, float *grads_dev, void *workspace_dev,
                    size_t workspace_bytes, void *stream) {
  int rc = check(s, batch, coeffs_dev, dcoeffs_dev);
  if (rc) return rc;
  if (!params_dev || !packed_dev || !sigma_dev || !workspace_dev || !grads_dev)
    return sl::set_error(SL_EINVAL, "NULL argument");
  size_t need = 0;
  sl_cnn_workspace_size(s, batch, 1, &need);
  if (workspace_bytes < need)
    return sl::set_error(SL_ENOMEM, "workspace too small: need " + std::to_string(need));
  hipStream_t st = (hipStream_t)stream;
  int H, W;
  plane_hw(s, H, W);
  Packed pk = packed_view(packed_dev, s->cfg.J);
  sl::CnnPlanes pl = planes(s, batch, sigma_dev);
  for (int j = 0; j < s->cfg.J; ++j)
    if (pl.start[j + 1] == pl.start[j]) return sl::set_error(SL_EINVAL, "a scale without planes");
  CK(sl::cnn_bwd(coeffs_dev, dcoeffs_dev, pl, H, W, pk.w1k, pk.w2, pk.w2t, pk.w3, params_dev,
                 s->num_cu, (float *)workspace_dev, grads_dev, st));
  return SL_OK;
}

int sl_cnn_adam(float *params_dev, const float *grads_dev, float *m_dev, float *v_dev, int n,
                float lr, int step, void *stream) {
  if (!params_dev || !grads_dev || !m_dev || !v_dev || n < 1 || step < 1)
    return sl::set_error(SL_EINVAL, "bad arguments to sl_cnn_adam");
  CK(sl::cnn_adam(params_dev, grads_dev, m_dev, v_dev, n, lr, 0.9, 0.999, 1e-8, step,
                  (hipStream_t)stream));
  return SL_OK;
}

int sl_sq_error_grad(const float *a_dev, const float *b_dev, size_t n, float scale,
                     float *out_dev, float *loss_dev, void *stream) {
  if (!a_dev || !b_dev || !out_dev || !loss_dev || n == 0)
    return sl::set_error(SL_EINVAL, "bad arguments to sl_sq_error_grad");
  // loss_dev[1 .. SL_SQERR_SCRATCH) holds the per-block partial sums
  CK(sl::sq_error_grad(a_dev, b_dev, n, scale, out_dev, loss_dev + 1, kErrBlocks, loss_dev,
                       (hipStream_t)stream));
  return SL_OK;
}

int sl_render_cartoons(const float *shapes_dev, int n, int H, int W, int max_shapes,
                       const float *sigma_dev, uint64_t noise_seed, float *clean_dev,
                       float *noisy_dev, void *stream) {
  if (!shapes_dev || !clean_dev || n < 1 || n > 65535 || H < 1 || W < 1 || max_shapes < 0 ||
      (noisy_dev && !sigma_dev))
    return sl::set_error(SL_EINVAL, "bad arguments to sl_render_cartoons");
  CK(sl::render_cartoons(shapes_dev, n, H, W, max_shapes, sigma_dev, noise_seed, clean_dev,
                         noisy_dev, (hipStream_t)stream));
  return SL_OK;
}

}  // extern "C"
