// C ABI of the MLP subgrid closure (declared in include/oc.h): workspace
// carving, parameter upload, and the forward / backward / Adam sequences
// built from the kernels of mlp.hip.
#include <cmath>
#include <cstring>
#include <new>
#include <vector>

#include "oc_internal.h"

using namespace oc;

#define OC_CHECK_HIP(expr)                                        \
  do {                                                            \
    hipError_t e_ = (expr);                                       \
    if (e_ != hipSuccess) {                                       \
      set_error("%s failed: %s", #expr, hipGetErrorString(e_));   \
      return OC_ERR_DEVICE;                                       \
    }                                                             \
  } while (0)

struct oc_mlp {
  int max_batch;
  MlpParams p;
  float* m1;
  float* m2;
  float* grad;
  float* y;         // max_batch x 4: outputs inside a model's step
  MlpTrain t;
  int step;
};

namespace {

struct MlpLayout {
  uint64_t master, m1, m2, grad, w1f, w2f, w2tf, w3f, w3tf, y, xf, h1f, h2f, dyf, dz2f, dz1f, biasp,
      lossp, loss, part, total;
};

uint64_t a256(uint64_t x) { return (x + 255) & ~uint64_t(255); }

MlpLayout mlp_layout(int B) {
  MlpLayout L;
  uint64_t o = 0;
  auto take = [&](uint64_t bytes) { uint64_t r = o; o += a256(bytes); return r; };
  const uint64_t kb = (uint64_t)B / 32, block = 1024;   // 32-row blocks; bytes of an operand block
  L.master = take((uint64_t)MLP_NPARAM * 4);
  L.m1 = take((uint64_t)MLP_NPARAM * 4);
  L.m2 = take((uint64_t)MLP_NPARAM * 4);
  L.grad = take((uint64_t)MLP_NPARAM * 4);
  L.w1f = take((uint64_t)MLP_NH * MLP_KIN * 2);
  L.w2f = take((uint64_t)MLP_NH * MLP_NH * 2);
  L.w2tf = take((uint64_t)MLP_NH * MLP_NH * 2);
  L.w3f = take((uint64_t)16 * MLP_NH * 2);
  L.w3tf = take((uint64_t)MLP_NH * 32 * 2);
  L.y = take((uint64_t)B * MLP_NOUT * 4);
  L.xf = take(kb * 32 * block);
  L.h1f = take(kb * 16 * block);
  L.h2f = take(kb * 16 * block);
  L.dyf = take(kb * block);
  L.dz2f = take(kb * 16 * block);
  L.dz1f = take(kb * 16 * block);
  L.biasp = take((uint64_t)TR_MAXWG * TR_NB * 4);
  L.lossp = take((uint64_t)TR_MAXWG * 8);
  L.loss = take(8);
  L.part = take((uint64_t)TR_MAXSPLIT * MLP_NPARAM * 4);
  L.total = o;
  return L;
}

int check_batch(const oc_mlp* m, int B) {
  if (!m) { set_error("mlp is NULL"); return OC_ERR_ARG; }
  if (B < 32 || B > m->max_batch || B % 32) {
    set_error("batch must be a multiple of 32 in [32, %d]", m->max_batch);
    return OC_ERR_ARG;
  }
  return OC_OK;
}

int read_loss(oc_mlp* m, int B, double* loss, hipStream_t s) {
  if (!loss) return OC_OK;
  double sum = 0.0;
  OC_CHECK_HIP(hipMemcpyAsync(&sum, m->t.loss, sizeof(sum), hipMemcpyDeviceToHost, s));
  OC_CHECK_HIP(hipStreamSynchronize(s));
  *loss = sum / ((double)B * MLP_NOUT);
  return OC_OK;
}

}  // namespace

namespace oc {

const float* mlp_output(oc_mlp* net) { return net->y; }
float* mlp_output_rw(oc_mlp* net) { return net->y; }
const MlpParams& mlp_params(const oc_mlp* net) { return net->p; }
int mlp_max_batch(const oc_mlp* net) { return net->max_batch; }

int mlp_params_finite(oc_mlp* net, hipStream_t s) {
  std::vector<float> p(MLP_NPARAM);
  OC_CHECK_HIP(hipMemcpyAsync(p.data(), net->p.master, p.size() * 4, hipMemcpyDeviceToHost, s));
  OC_CHECK_HIP(hipStreamSynchronize(s));
  for (float x : p)
    if (!std::isfinite(x)) return 0;
  return 1;
}

}  // namespace oc

extern "C" {

int oc_mlp_workspace_size(int32_t max_batch, uint64_t* bytes) {
  if (!bytes || max_batch < 32 || max_batch % 32) {
    set_error("max_batch must be a positive multiple of 32");
    return OC_ERR_ARG;
  }
  *bytes = mlp_layout(max_batch).total;
  return OC_OK;
}

int oc_mlp_create(int32_t max_batch, void* workspace, uint64_t bytes, oc_mlp** out) {
  if (!out || !workspace || max_batch < 32 || max_batch % 32) {
    set_error("need a workspace, an output handle and max_batch a multiple of 32");
    return OC_ERR_ARG;
  }
  if ((uintptr_t)workspace % 256) { set_error("workspace must be 256-byte aligned"); return OC_ERR_ARG; }
  const MlpLayout L = mlp_layout(max_batch);
  if (bytes < L.total) {
    set_error("workspace has %llu bytes, needs %llu", (unsigned long long)bytes,
              (unsigned long long)L.total);
    return OC_ERR_ARG;
  }
  hipPointerAttribute_t attr;
  if (hipPointerGetAttributes(&attr, workspace) != hipSuccess || attr.type != hipMemoryTypeDevice) {
    (void)hipGetLastError();
    set_error("workspace is not device memory");
    return OC_ERR_ARG;
  }
  oc_mlp* m = new (std::nothrow) oc_mlp;
  if (!m) { set_error("out of host memory"); return OC_ERR_ARG; }
  char* w = (char*)workspace;
  m->max_batch = max_batch;
  m->p.master = (float*)(w + L.master);
  m->m1 = (float*)(w + L.m1);
  m->m2 = (float*)(w + L.m2);
  m->grad = (float*)(w + L.grad);
  m->p.W1f = (__bf16*)(w + L.w1f);
  m->p.W2f = (__bf16*)(w + L.w2f);
  m->p.W2Tf = (__bf16*)(w + L.w2tf);
  m->p.W3f = (__bf16*)(w + L.w3f);
  m->p.W3Tf = (__bf16*)(w + L.w3tf);
  m->y = (float*)(w + L.y);
  m->t.xf = (__bf16*)(w + L.xf);
  m->t.h1f = (__bf16*)(w + L.h1f);
  m->t.h2f = (__bf16*)(w + L.h2f);
  m->t.dyf = (__bf16*)(w + L.dyf);
  m->t.dz2f = (__bf16*)(w + L.dz2f);
  m->t.dz1f = (__bf16*)(w + L.dz1f);
  m->t.biasp = (float*)(w + L.biasp);
  m->t.lossp = (double*)(w + L.lossp);
  m->t.loss = (double*)(w + L.loss);
  m->t.part = (float*)(w + L.part);
  m->step = 0;
  // zero everything: padded weight rows/columns stay zero for good
  if (hipMemset(workspace, 0, L.total) != hipSuccess || hipDeviceSynchronize() != hipSuccess) {
    set_error("mlp setup failed");
    delete m;
    return OC_ERR_DEVICE;
  }
  *out = m;
  return OC_OK;
}

int oc_mlp_destroy(oc_mlp* m) {
  delete m;
  return OC_OK;
}

int oc_mlp_set_params(oc_mlp* m, const float* params, void* stream) {
  if (!m || !params) { set_error("NULL argument"); return OC_ERR_ARG; }
  for (int i = 0; i < MLP_NPARAM; ++i)
    if (!std::isfinite(params[i])) { set_error("parameter %d is not finite", i); return OC_ERR_NONFINITE; }
  hipStream_t s = (hipStream_t)stream;
  OC_CHECK_HIP(hipMemcpyAsync(m->p.master, params, (size_t)MLP_NPARAM * 4, hipMemcpyHostToDevice, s));
  OC_CHECK_HIP(launch_refresh_bf16(m->p, MLP_NPARAM, s));
  // a fresh optimiser state
  OC_CHECK_HIP(hipMemsetAsync(m->m1, 0, (size_t)MLP_NPARAM * 4, s));
  OC_CHECK_HIP(hipMemsetAsync(m->m2, 0, (size_t)MLP_NPARAM * 4, s));
  OC_CHECK_HIP(hipStreamSynchronize(s));
  m->step = 0;
  return OC_OK;
}

int oc_mlp_get_params(oc_mlp* m, float* params, void* stream) {
  if (!m || !params) { set_error("NULL argument"); return OC_ERR_ARG; }
  hipStream_t s = (hipStream_t)stream;
  OC_CHECK_HIP(hipMemcpyAsync(params, m->p.master, (size_t)MLP_NPARAM * 4, hipMemcpyDeviceToHost, s));
  OC_CHECK_HIP(hipStreamSynchronize(s));
  return OC_OK;
}

int oc_mlp_forward(oc_mlp* m, const float* x, int32_t batch, float* y, void* stream) {
  int rc = check_batch(m, batch);
  if (rc) return rc;
  if (!x || !y) { set_error("NULL argument"); return OC_ERR_ARG; }
  hipStream_t s = (hipStream_t)stream;
  // outputs that lie in the rows: the kernel's workgroups store theirs while
  // others still read, so they go through the handle's own
  const uintptr_t x0 = (uintptr_t)x, y0 = (uintptr_t)y;
  const size_t nx = (size_t)batch * MLP_NIN * 4, ny = (size_t)batch * MLP_NOUT * 4;
  const bool overlap = y0 < x0 + nx && x0 < y0 + ny;
  float* out = overlap ? m->y : y;
  OC_CHECK_HIP(launch_mlp_forward(m->p, x, batch, out, s));
  if (overlap) OC_CHECK_HIP(hipMemcpyAsync(y, out, ny, hipMemcpyDeviceToDevice, s));
  return OC_OK;
}

int oc_mlp_gradients(oc_mlp* m, const float* x, const float* target, int32_t batch, float* grad,
                     double* loss, void* stream) {
  int rc = check_batch(m, batch);
  if (rc) return rc;
  if (!x || !target || !grad) { set_error("NULL argument"); return OC_ERR_ARG; }
  hipStream_t s = (hipStream_t)stream;
  OC_CHECK_HIP(launch_mlp_gradients(m->p, m->t, x, target, batch, grad, nullptr, nullptr, 0.f, 0, s));
  return read_loss(m, batch, loss, s);
}

int oc_mlp_train_step(oc_mlp* m, const float* x, const float* target, int32_t batch, float lr,
                      double* loss, void* stream) {
  int rc = check_batch(m, batch);
  if (rc) return rc;
  if (!x || !target || !(lr > 0)) { set_error("need inputs, targets and lr > 0"); return OC_ERR_ARG; }
  hipStream_t s = (hipStream_t)stream;
  m->step += 1;
  OC_CHECK_HIP(launch_mlp_gradients(m->p, m->t, x, target, batch, m->grad, m->m1, m->m2, lr, m->step,
                                    s));
  return read_loss(m, batch, loss, s);
}

}  // extern "C"
