// C-ABI of the surrogate MLP: parameters, forward with input gradient,
// full gradients and the Adam training step.  Kernels in mlp_kernels.h.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "internal.h"
#include "mlp_fused.h"
#include "mlp_train.h"

namespace pcsdf {

// Rows per partial of the weight gradient: at most kMaxParts partials
// while each covers at most kChunk rows (65,536 rows: 128 partials of 512
// rows, so that the 128 x 5 workgroups fill the chip and the partials, 216
// KB each, stay a fifth of the bytes the kernel reads).
constexpr int kChunk = 1024, kMaxParts = 128;
// Row tiles of the fused inference in flight at once: two workgroups per
// CU on 256 CUs.
constexpr int kInferBlocks = 512;
constexpr int kWofs[5] = {0, 4096, 20480, 36864, 53248};
constexpr int kWbfTotal = 53376;

struct Mlp {
  Handle *h = nullptr;
  int n_in = 0;    // inputs per row, 1..kInPad
  int nparam = 0;  // mlp_nparam(n_in)
  DevBuf params, grad, m1, m2, wbf, wtbf, norm, wofs;
  float out_scale = 1.f;
  int64_t step = 0;  // Adam steps taken
  // workspace, grown with the batch
  int cap = 0;
  DevBuf a0, act, dz, seed, wpart, lpart;
};

static int chunk_rows(int npad) {
  const int r = (npad + kMaxParts - 1) / kMaxParts;
  return std::min(kChunk, (r + kSlabRows - 1) / kSlabRows * kSlabRows);
}
static int chunk_count(int npad) {
  const int r = chunk_rows(npad);
  return (npad + r - 1) / r;
}

static int ws(Mlp *m, int npad, hipStream_t s) {
  Handle *h = m->h;
  if (npad <= m->cap) return PCSDF_OK;
  const size_t r = (size_t)npad;
  // a smaller batch may use more, shorter chunks, but never more than
  // kMaxParts where a larger one does not
  const size_t parts = std::max(chunk_count(npad), std::min(kMaxParts, npad / kSlabRows));
  int rc;
  if ((rc = ensure_buffer(h, m->a0, r * kInPad * 2, s)) ||
      (rc = ensure_buffer(h, m->act, 4 * r * kHid * 2, s)) ||
      (rc = ensure_buffer(h, m->dz, 4 * r * kHid * 2, s)) ||
      (rc = ensure_buffer(h, m->seed, r * 4, s)) ||
      (rc = ensure_buffer(h, m->wpart, parts * kPartLen * 4, s)) ||
      (rc = ensure_buffer(h, m->lpart, r / 32 * 4, s)))
    return rc;
  m->cap = npad;
  return PCSDF_OK;
}

static const uint16_t *wb(Mlp *m, int l) {
  return reinterpret_cast<const uint16_t *>(m->wbf.ptr) + kWofs[l];
}
static const uint16_t *wtb(Mlp *m, int l) {
  return reinterpret_cast<const uint16_t *>(m->wtbf.ptr) + kWofs[l];
}
static int np(const Mlp *m) { return m->nparam; }
static const float *pf(Mlp *m) {
  return reinterpret_cast<const float *>(m->params.ptr);
}

static unsigned blocks(int64_t n, int per) {
  return (unsigned)((n + per - 1) / per);
}

static NetWeights weights(Mlp *m) {
  NetWeights w;
  for (int l = 0; l <= kLayers; ++l) w.W[l] = wb(m, l);
  for (int l = 0; l < kLayers; ++l) w.Wt[l] = wtb(m, l);
  return w;
}

// Parameter gradient gp of the loss whose seed is 2 (y - tgt) / n or, when
// dy is given, dy; and, if given, the mean squared residual and the
// gradient of the inputs.
static int gradients(Mlp *m, int n, const float *x, const float *tgt,
                     const float *dy, float *gp, float *loss, float *grad_x,
                     hipStream_t s) {
  const int npad = (n + kRowTile - 1) / kRowTile * kRowTile;
  int rc;
  if ((rc = ws(m, npad, s))) return rc;
  uint16_t *a0 = reinterpret_cast<uint16_t *>(m->a0.ptr);
  uint16_t *act = reinterpret_cast<uint16_t *>(m->act.ptr);
  uint16_t *dz = reinterpret_cast<uint16_t *>(m->dz.ptr);
  float *seed = reinterpret_cast<float *>(m->seed.ptr);
  float *wpart = reinterpret_cast<float *>(m->wpart.ptr);
  float *lpart = reinterpret_cast<float *>(m->lpart.ptr);
  const int64_t stride = (int64_t)npad * kHid;
  hipLaunchKernelGGL(k_mlp_train_rows, dim3(npad / kRowTile),
                     dim3(64 * kRowWaves), 0, s, x, n, m->n_in,
                     reinterpret_cast<const float *>(m->norm.ptr), weights(m),
                     pf(m), m->out_scale, tgt, dy, a0, act, dz, stride, seed,
                     lpart, grad_x);
  const int chunks = chunk_count(npad);
  hipLaunchKernelGGL(k_mlp_wgrad, dim3(chunks, 5), dim3(256), 0, s, a0, act,
                     dz, stride, seed, npad, chunk_rows(npad), wpart);
  hipLaunchKernelGGL(k_grad_sum, dim3(blocks(kPartLen, 64) + 1), dim3(256), 0,
                     s, wpart, chunks, m->n_in, gp, lpart, npad / 32,
                     1.f / (float)n, loss);
  return check_launch(m->h, "mlp gradients");
}

static int check_rows(Mlp *m, int n, const void *x) {
  if (n < 0 || n > (1 << 28))
    return fail(m->h, PCSDF_ERR_INVALID_ARG, "n must be in [0, 2^28]");
  if (n > 0 && !x) return fail(m->h, PCSDF_ERR_INVALID_ARG, "x is NULL");
  return PCSDF_OK;
}

// Fused inference (value and input gradient) of rows [0, n) (with n_dev,
// [0, min(n, *n_dev)) read on the device).
static int mlp_infer(Mlp *m, int n, const int *n_dev, const float *x,
                     float *y, float *gx, hipStream_t s) {
  if (n == 0) return PCSDF_OK;
  const bool few = n <= kFewRows;
  const int rows = few ? 32 : kRowTile;
  const int grid = std::min((n + rows - 1) / rows, kInferBlocks);
  hipLaunchKernelGGL(few ? k_mlp_infer_few : k_mlp_infer, dim3(grid),
                     dim3(64 * kRowWaves), 0, s, x, n, n_dev, m->n_in,
                     reinterpret_cast<const float *>(m->norm.ptr), weights(m),
                     pf(m), m->out_scale, y, gx);
  return check_launch(m->h, "mlp inference");
}

}  // namespace pcsdf

using namespace pcsdf;

struct pcsdf_mlp : Mlp {};

Handle *pcsdf::mlp_handle(pcsdf_mlp *m) { return m ? m->h : nullptr; }
int pcsdf::mlp_inputs(const pcsdf_mlp *m) { return m ? m->n_in : 0; }
int pcsdf::mlp_rows(pcsdf_mlp *m, int n, const int32_t *n_dev,
                    const float *x, float *y, float *gx, hipStream_t s) {
  return mlp_infer(m, n, n_dev, x, y, gx, s);
}

extern "C" int pcsdf_mlp_param_count(int32_t n_in) {
  return n_in >= 1 && n_in <= kInPad ? mlp_nparam(n_in) : -1;
}

extern "C" int pcsdf_mlp_create(pcsdf_handle *hp, int32_t n_in,
                                pcsdf_mlp **out) {
  Handle *h = reinterpret_cast<Handle *>(hp);
  if (!h) return PCSDF_ERR_INVALID_ARG;
  if (!out) return fail(h, PCSDF_ERR_INVALID_ARG, "out is NULL");
  *out = nullptr;
  if (n_in < 1 || n_in > kInPad)
    return fail(h, PCSDF_ERR_INVALID_ARG, "n_in must be in [1, 32]");
  int rc;
  if ((rc = bind_device(h))) return rc;
  pcsdf_mlp *m = new (std::nothrow) pcsdf_mlp();
  if (!m) return fail(h, PCSDF_ERR_OOM, "mlp allocation failed");
  m->h = h;
  m->n_in = n_in;
  m->nparam = mlp_nparam(n_in);
  const size_t P = (size_t)m->nparam * 4;
  if ((rc = ensure_buffer(h, m->params, P, nullptr)) ||
      (rc = ensure_buffer(h, m->grad, P, nullptr)) ||
      (rc = ensure_buffer(h, m->m1, P, nullptr)) ||
      (rc = ensure_buffer(h, m->m2, P, nullptr)) ||
      (rc = ensure_buffer(h, m->wbf, kWbfTotal * 2, nullptr)) ||
      (rc = ensure_buffer(h, m->wtbf, kWbfTotal * 2, nullptr)) ||
      (rc = ensure_buffer(h, m->norm, 2 * kInPad * 4, nullptr)) ||
      (rc = ensure_buffer(h, m->wofs, 5 * 4, nullptr))) {
    pcsdf_mlp_destroy(m);
    return rc;
  }
  if (hipMemset(m->wbf.ptr, 0, m->wbf.bytes) != hipSuccess ||
      hipMemset(m->wtbf.ptr, 0, m->wtbf.bytes) != hipSuccess ||
      hipMemcpy(m->wofs.ptr, kWofs, sizeof(kWofs), hipMemcpyHostToDevice) !=
          hipSuccess) {
    pcsdf_mlp_destroy(m);
    return fail(h, PCSDF_ERR_HIP, "mlp initialisation failed");
  }
  *out = m;
  return PCSDF_OK;
}

extern "C" void pcsdf_mlp_destroy(pcsdf_mlp *m) {
  if (!m) return;
  DevBuf *bufs[] = {&m->params, &m->grad, &m->m1,   &m->m2,  &m->wbf,
                    &m->wtbf,   &m->norm, &m->wofs, &m->a0,  &m->act,
                    &m->dz,     &m->seed, &m->wpart, &m->lpart};
  bool any = false;
  for (DevBuf *b : bufs) any = any || b->ptr;
  if (any) (void)hipDeviceSynchronize();
  for (DevBuf *b : bufs)
    if (b->ptr) (void)hipFree(b->ptr);
  delete m;
}

extern "C" int pcsdf_mlp_set_params(pcsdf_mlp *m, const float *params_host,
                                    const float *in_offset_host,
                                    const float *in_scale_host,
                                    float out_scale) {
  if (!m) return PCSDF_ERR_INVALID_ARG;
  Handle *h = m->h;
  if (!params_host || !in_offset_host || !in_scale_host)
    return fail(h, PCSDF_ERR_INVALID_ARG, "params, offset and scale required");
  const int P = np(m), ni = m->n_in;
  for (int i = 0; i < P; ++i)
    if (!std::isfinite(params_host[i]))
      return fail(h, PCSDF_ERR_NUMERIC,
                  "non-finite parameter at index " + std::to_string(i));
  for (int i = 0; i < ni; ++i)
    if (!std::isfinite(in_offset_host[i]) || !std::isfinite(in_scale_host[i]))
      return fail(h, PCSDF_ERR_NUMERIC, "non-finite normalisation");
  if (!std::isfinite(out_scale))
    return fail(h, PCSDF_ERR_NUMERIC, "non-finite output scale");
  // [offset 32][scale 32]; padding columns read offset 0, scale 1
  std::vector<float> norm(2 * kInPad, 0.f);
  std::fill(norm.begin() + kInPad, norm.end(), 1.f);
  std::memcpy(norm.data(), in_offset_host, (size_t)ni * 4);
  std::memcpy(norm.data() + kInPad, in_scale_host, (size_t)ni * 4);
  if (hipDeviceSynchronize() != hipSuccess ||
      hipMemcpy(m->params.ptr, params_host, (size_t)P * 4,
                hipMemcpyHostToDevice) != hipSuccess ||
      hipMemcpy(m->norm.ptr, norm.data(), norm.size() * 4,
                hipMemcpyHostToDevice) != hipSuccess ||
      hipMemset(m->m1.ptr, 0, (size_t)P * 4) != hipSuccess ||
      hipMemset(m->m2.ptr, 0, (size_t)P * 4) != hipSuccess)
    return fail(h, PCSDF_ERR_HIP, "uploading the parameters failed");
  m->out_scale = out_scale;
  m->step = 0;
  hipLaunchKernelGGL(k_cast_weights, dim3(blocks(P, 256)), dim3(256), 0,
                     nullptr, reinterpret_cast<const float *>(m->params.ptr),
                     reinterpret_cast<uint16_t *>(m->wbf.ptr),
                     reinterpret_cast<uint16_t *>(m->wtbf.ptr),
                     reinterpret_cast<const int *>(m->wofs.ptr), ni);
  if (hipDeviceSynchronize() != hipSuccess)
    return fail(h, PCSDF_ERR_HIP, "casting the weights failed");
  return PCSDF_OK;
}

extern "C" int pcsdf_mlp_get_params(pcsdf_mlp *m, float *params_host) {
  if (!m) return PCSDF_ERR_INVALID_ARG;
  if (!params_host) return fail(m->h, PCSDF_ERR_INVALID_ARG, "params NULL");
  if (hipDeviceSynchronize() != hipSuccess ||
      hipMemcpy(params_host, m->params.ptr, (size_t)np(m) * 4,
                hipMemcpyDeviceToHost) != hipSuccess)
    return fail(m->h, PCSDF_ERR_HIP, "reading the parameters failed");
  return PCSDF_OK;
}

extern "C" int pcsdf_mlp_forward(pcsdf_mlp *m, int32_t n, const float *x_dev,
                                 float *y_dev, float *grad_x_dev,
                                 void *stream) {
  if (!m) return PCSDF_ERR_INVALID_ARG;
  int rc = check_rows(m, n, x_dev);
  if (rc || n == 0) return rc;
  if (!y_dev) return fail(m->h, PCSDF_ERR_INVALID_ARG, "y_dev is NULL");
  if (((uintptr_t)x_dev | (uintptr_t)y_dev | (uintptr_t)grad_x_dev) & 3)
    return fail(m->h, PCSDF_ERR_ALIGN, "device buffers must be 4-byte aligned");
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  ProfScope ps(m->h, PCSDF_KERNEL_MLP, s);
  return mlp_infer(m, n, nullptr, x_dev, y_dev, grad_x_dev, s);
}

extern "C" int pcsdf_mlp_gradients(pcsdf_mlp *m, int32_t n,
                                   const float *x_dev, const float *dy_dev,
                                   float *grad_params_dev, float *grad_x_dev,
                                   void *stream) {
  if (!m) return PCSDF_ERR_INVALID_ARG;
  int rc = check_rows(m, n, x_dev);
  if (rc) return rc;
  if (n == 0 || !dy_dev || !grad_params_dev)
    return fail(m->h, PCSDF_ERR_INVALID_ARG, "need n > 0, dy and grad");
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  return gradients(m, n, x_dev, nullptr, dy_dev, grad_params_dev, nullptr,
                   grad_x_dev, s);
}

// One bias-corrected Adam step from the gradient g (device, fp32
// [nparam]); the step counter advances first, so the first step uses
// c1 = 1 - beta1, c2 = 1 - beta2.
static int adam(Mlp *m, const float *g, float lr, float beta1, float beta2,
                float eps, hipStream_t s) {
  m->step += 1;
  const float c1 = (float)(1.0 - std::pow((double)beta1, (double)m->step));
  const float c2 = (float)(1.0 - std::pow((double)beta2, (double)m->step));
  hipLaunchKernelGGL(k_adam, dim3(blocks(np(m), 256)), dim3(256), 0, s,
                     reinterpret_cast<float *>(m->params.ptr), g,
                     reinterpret_cast<float *>(m->m1.ptr),
                     reinterpret_cast<float *>(m->m2.ptr), lr, beta1, beta2,
                     eps, c1, c2, reinterpret_cast<uint16_t *>(m->wbf.ptr),
                     reinterpret_cast<uint16_t *>(m->wtbf.ptr),
                     reinterpret_cast<const int *>(m->wofs.ptr), m->n_in);
  return check_launch(m->h, "mlp adam step");
}

static int check_adam(Mlp *m, float lr, float beta1, float beta2, float eps) {
  if (!(lr >= 0) || !(beta1 >= 0 && beta1 < 1) || !(beta2 >= 0 && beta2 < 1) ||
      !(eps > 0) || !std::isfinite(lr) || !std::isfinite(eps))
    return fail(m->h, PCSDF_ERR_NUMERIC, "bad optimiser hyper-parameters");
  return PCSDF_OK;
}

extern "C" int pcsdf_mlp_loss_gradients(pcsdf_mlp *m, int32_t n,
                                        const float *x_dev,
                                        const float *target_dev,
                                        float *grad_params_dev,
                                        float *loss_dev, void *stream) {
  if (!m) return PCSDF_ERR_INVALID_ARG;
  int rc = check_rows(m, n, x_dev);
  if (rc) return rc;
  if (n == 0 || !target_dev || !grad_params_dev)
    return fail(m->h, PCSDF_ERR_INVALID_ARG,
                "need n > 0, targets and a gradient buffer");
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  if (((uintptr_t)x_dev | (uintptr_t)target_dev | (uintptr_t)grad_params_dev |
       (uintptr_t)loss_dev) & 3)
    return fail(m->h, PCSDF_ERR_ALIGN, "device buffers must be 4-byte aligned");
  return gradients(m, n, x_dev, target_dev, nullptr, grad_params_dev,
                   loss_dev, nullptr, s);
}

extern "C" int pcsdf_mlp_adam_step(pcsdf_mlp *m, const float *grad_params_dev,
                                   float lr, float beta1, float beta2,
                                   float eps, void *stream) {
  if (!m) return PCSDF_ERR_INVALID_ARG;
  if (!grad_params_dev)
    return fail(m->h, PCSDF_ERR_INVALID_ARG, "gradient is NULL");
  if ((uintptr_t)grad_params_dev & 3)
    return fail(m->h, PCSDF_ERR_ALIGN, "gradient must be 4-byte aligned");
  int rc;
  if ((rc = check_adam(m, lr, beta1, beta2, eps))) return rc;
  return adam(m, grad_params_dev, lr, beta1, beta2, eps,
              reinterpret_cast<hipStream_t>(stream));
}

extern "C" int pcsdf_mlp_train_step(pcsdf_mlp *m, int32_t n,
                                    const float *x_dev,
                                    const float *target_dev, float lr,
                                    float beta1, float beta2, float eps,
                                    float *loss_dev, void *stream) {
  if (!m) return PCSDF_ERR_INVALID_ARG;
  int rc = check_rows(m, n, x_dev);
  if (rc) return rc;
  if (n == 0 || !target_dev)
    return fail(m->h, PCSDF_ERR_INVALID_ARG, "need n > 0 and targets");
  if ((rc = check_adam(m, lr, beta1, beta2, eps))) return rc;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  ProfScope ps(m->h, PCSDF_KERNEL_MLP_TRAIN, s);
  float *gp = reinterpret_cast<float *>(m->grad.ptr);
  if ((rc = gradients(m, n, x_dev, target_dev, nullptr, gp, loss_dev, nullptr,
                      s)))
    return rc;
  return adam(m, gp, lr, beta1, beta2, eps, s);
}

extern "C" int pcsdf_mlp_get_state(pcsdf_mlp *m, float *params_host,
                                   float *m1_host, float *m2_host,
                                   int64_t *step) {
  if (!m) return PCSDF_ERR_INVALID_ARG;
  if (!params_host || !m1_host || !m2_host || !step)
    return fail(m->h, PCSDF_ERR_INVALID_ARG, "every output is required");
  const size_t P = (size_t)np(m) * 4;
  if (hipDeviceSynchronize() != hipSuccess ||
      hipMemcpy(params_host, m->params.ptr, P, hipMemcpyDeviceToHost) !=
          hipSuccess ||
      hipMemcpy(m1_host, m->m1.ptr, P, hipMemcpyDeviceToHost) != hipSuccess ||
      hipMemcpy(m2_host, m->m2.ptr, P, hipMemcpyDeviceToHost) != hipSuccess)
    return fail(m->h, PCSDF_ERR_HIP, "reading the optimiser state failed");
  *step = m->step;
  return PCSDF_OK;
}

extern "C" int pcsdf_mlp_set_state(pcsdf_mlp *m, const float *params_host,
                                   const float *m1_host, const float *m2_host,
                                   int64_t step, const float *in_offset_host,
                                   const float *in_scale_host,
                                   float out_scale) {
  if (!m) return PCSDF_ERR_INVALID_ARG;
  if (!m1_host || !m2_host)
    return fail(m->h, PCSDF_ERR_INVALID_ARG, "moments are required");
  if (step < 0 || step > (int64_t)1 << 40)
    return fail(m->h, PCSDF_ERR_INVALID_ARG, "step out of range");
  for (int i = 0; i < np(m); ++i)
    if (!std::isfinite(m1_host[i]) || !std::isfinite(m2_host[i]) ||
        m2_host[i] < 0.f)
      return fail(m->h, PCSDF_ERR_NUMERIC,
                  "bad moment at index " + std::to_string(i));
  int rc = pcsdf_mlp_set_params(m, params_host, in_offset_host,
                                in_scale_host, out_scale);
  if (rc) return rc;
  const size_t P = (size_t)np(m) * 4;
  if (hipMemcpy(m->m1.ptr, m1_host, P, hipMemcpyHostToDevice) != hipSuccess ||
      hipMemcpy(m->m2.ptr, m2_host, P, hipMemcpyHostToDevice) != hipSuccess)
    return fail(m->h, PCSDF_ERR_HIP, "uploading the moments failed");
  m->step = step;
  return PCSDF_OK;
}
