// Host runtime of the surrogate network (C ABI in include/fib.h).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/fib.h"
#include "mlp_internal.h"

namespace fib {
int set_error(int code, const char* msg);  // fib_api.hip
}

struct fib_mlp {
  fib::MlpShape shape{};
  hipStream_t stream = nullptr;
  int device = 0;             // device the network lives on
  float* d_params = nullptr;  // FP32 master parameters
  float* d_m = nullptr;       // Adam first moment
  float* d_v = nullptr;       // Adam second moment
  float* d_grad = nullptr;
  void* d_frags = nullptr;    // BF16 operand fragments of d_params, always current
  float* d_work = nullptr;    // work space of the gradient
  int work_chunks = 0;        // chunks it holds
  int64_t t = 0;              // Adam step count
};

// Scratch of fib_mlp_gradient_noalloc: the gradient's work space, in a fixed
// array of every device's code object instead of memory allocated
// per call.  The array's name is a host-side stand-in: host code uses only
// the device address that hipGetSymbolAddress returns, looked up once per
// device with that device current (at fib_mlp_create) and kept in g_scratch
// below.  Every call on a device shares that device's array.
static __device__ __align__(256) float scratch[fib::kScratchFloats];

// Work space of fib_column_stats, one per device (its address as above); a
// call holds its device's lock while it uses it.
static __device__ __align__(256) char col_work[sizeof(fib::ColWork)];

// Batches fib_mlp_gradient_noalloc takes: ceil(B / 32) (n_params + 1) floats
// at most.
static constexpr int64_t kNoallocFloats = (int64_t)1 << 22;

namespace fib {
const MlpShape& mlp_shape(const fib_mlp* n) { return n->shape; }
const float* mlp_device_params(const fib_mlp* n) { return n->d_params; }
hipStream_t mlp_stream(const fib_mlp* n) { return n->stream; }
}  // namespace fib

namespace {

int mfail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  return fib::set_error(code, buf);
}

#define MHIP(expr)                                                                    \
  do {                                                                                \
    hipError_t e_ = (expr);                                                           \
    if (e_ != hipSuccess) return mfail(FIB_EHIP, "%s: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float* g_scratch[kMaxDevices] = {};
std::mutex g_col_mu[kMaxDevices];

// Looks up (once) the scratch address of `dev`, which must be current.
int scratch_setup(int dev) {
  if (dev < 0 || dev >= kMaxDevices) return mfail(FIB_EUNSUPPORTED, "device %d out of range", dev);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch[dev]) return FIB_OK;
  void* p = nullptr;
  const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess || !p)
    return mfail(FIB_EHIP, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
  g_scratch[dev] = static_cast<float*>(p);
  return FIB_OK;
}

float* scratch_of(int dev) {
  if (dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  return g_scratch[dev];
}

// LDS of a chunk's activations, pre-activations and two gradient blocks in
// FP32: the network widths this library takes are those for which it fits a
// workgroup (the kernels' own LDS is smaller, whatever the widths).
size_t chunk_fp32_bytes(const fib::MlpShape& s) {
  int64_t f = 0, pmax = 0;
  for (int l = 0; l <= s.L; ++l) {
    f += s.pad[l] * (l > 0 && l < s.L ? 2 : 1);
    pmax = std::max<int64_t>(pmax, s.pad[l]);
  }
  return sizeof(float) * fib::kChunk * (size_t)(f + 2 * pmax);
}

// Work space for passes of `chunks` chunks; it grows with the largest batch,
// up to one pass.
int ensure_work(fib_mlp* n, int chunks) {
  if (chunks <= n->work_chunks) return FIB_OK;
  (void)hipStreamSynchronize(n->stream);
  (void)hipFree(n->d_work);
  n->d_work = nullptr;
  n->work_chunks = 0;
  if (hipMalloc(&n->d_work, sizeof(float) * (size_t)chunks * fib::mlp_chunk_floats(n->shape)) !=
      hipSuccess)
    return mfail(FIB_ENOMEM, "device allocation of %d gradient chunks failed", chunks);
  n->work_chunks = chunks;
  return FIB_OK;
}

}  // namespace

extern "C" {

int fib_mlp_create(int32_t n_layers, const int32_t* sizes, int32_t activation, void* stream,
                   fib_mlp_t** out) {
  if (!out) return mfail(FIB_EINVAL, "null output pointer");
  *out = nullptr;
  if (n_layers < 1 || n_layers > fib::kMaxLayers || !sizes)
    return mfail(FIB_EINVAL, "the network needs 1..%d weight layers", fib::kMaxLayers);
  if (activation != FIB_ACT_SILU && activation != FIB_ACT_RELU)
    return mfail(FIB_EINVAL, "unknown activation %d", activation);
  fib::MlpShape s{};
  s.L = n_layers;
  s.act = activation;
  int64_t off = 0;
  for (int l = 0; l <= n_layers; ++l) {
    if (sizes[l] < 1 || sizes[l] > 512) return mfail(FIB_EINVAL, "layer width %d not in 1..512", sizes[l]);
    s.size[l] = sizes[l];
    s.pad[l] = (sizes[l] + fib::kPad - 1) / fib::kPad * fib::kPad;
  }
  for (int l = 1; l <= n_layers; ++l) {
    s.w_off[l] = (int)off;
    off += (int64_t)s.size[l] * s.size[l - 1];
    s.b_off[l] = (int)off;
    off += s.size[l];
  }
  s.n_params = (int)off;
  for (int l = 1; l <= n_layers; ++l) {
    s.f_off[l] = s.n_frag;
    s.n_frag += s.pad[l] * s.pad[l - 1];
    s.r_off[l] = s.n_frag;
    if (l > 1) s.n_frag += s.pad[l] * s.pad[l - 1];
    const int ib = (s.size[l - 1] + 15) / 16, ob = (s.size[l] + 15) / 16;
    s.a_ops[l] = s.n_ops;
    s.d_ops[l] = s.n_ops + ib;
    s.n_ops += ib + ob;
    s.n_tiles += ob * ib;
    s.bias_off[l] = s.n_bias;
    s.n_bias += s.size[l];
  }
  hipDeviceProp_t prop;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess)
    return mfail(FIB_EHIP, "no HIP device");
  if (chunk_fp32_bytes(s) > prop.sharedMemPerBlock)
    return mfail(FIB_EUNSUPPORTED, "network too wide for one workgroup's LDS");
  if (int rc = scratch_setup(dev)) return rc;
  fib_mlp* n = new (std::nothrow) fib_mlp();
  if (!n) return mfail(FIB_ENOMEM, "host allocation failed");
  n->shape = s;
  n->stream = (hipStream_t)stream;
  n->device = dev;
  const size_t bytes = sizeof(float) * (size_t)s.n_params;
  if (hipMalloc(&n->d_params, bytes) != hipSuccess || hipMalloc(&n->d_m, bytes) != hipSuccess ||
      hipMalloc(&n->d_v, bytes) != hipSuccess || hipMalloc(&n->d_grad, bytes) != hipSuccess ||
      hipMalloc(&n->d_frags, 2 * (size_t)s.n_frag) != hipSuccess) {
    fib_mlp_destroy(n);
    return mfail(FIB_ENOMEM, "device allocation failed");
  }
  if (hipMemset(n->d_params, 0, bytes) != hipSuccess || hipMemset(n->d_m, 0, bytes) != hipSuccess ||
      hipMemset(n->d_v, 0, bytes) != hipSuccess ||
      hipMemset(n->d_frags, 0, 2 * (size_t)s.n_frag) != hipSuccess) {
    fib_mlp_destroy(n);
    return mfail(FIB_EHIP, "device initialization failed");
  }
  *out = n;
  return FIB_OK;
}

void fib_mlp_destroy(fib_mlp_t* n) {
  if (!n) return;
  (void)hipStreamSynchronize(n->stream);
  (void)hipFree(n->d_params);
  (void)hipFree(n->d_m);
  (void)hipFree(n->d_v);
  (void)hipFree(n->d_grad);
  (void)hipFree(n->d_frags);
  (void)hipFree(n->d_work);
  delete n;
}

int64_t fib_mlp_n_params(const fib_mlp_t* n) { return n ? n->shape.n_params : 0; }

int fib_mlp_set_params(fib_mlp_t* n, const float* params, int64_t count) {
  if (!n || !params) return mfail(FIB_EINVAL, "null argument");
  if (count != n->shape.n_params) return mfail(FIB_EINVAL, "expected %d parameters", n->shape.n_params);
  MHIP(hipMemcpyAsync(n->d_params, params, sizeof(float) * count, hipMemcpyHostToDevice, n->stream));
  MHIP(fib::launch_mlp_pack(n->shape, n->d_params, n->d_frags, n->stream));
  MHIP(hipStreamSynchronize(n->stream));
  return FIB_OK;
}

int fib_mlp_get_params(fib_mlp_t* n, float* params, int64_t count) {
  if (!n || !params) return mfail(FIB_EINVAL, "null argument");
  if (count != n->shape.n_params) return mfail(FIB_EINVAL, "expected %d parameters", n->shape.n_params);
  MHIP(hipMemcpyAsync(params, n->d_params, sizeof(float) * count, hipMemcpyDeviceToHost, n->stream));
  MHIP(hipStreamSynchronize(n->stream));
  return FIB_OK;
}

int fib_mlp_forward(fib_mlp_t* n, const float* X, int64_t B, float* O) {
  if (!n || B < 0 || (B > 0 && (!X || !O))) return mfail(FIB_EINVAL, "bad arguments");
  MHIP(fib::launch_mlp_forward(n->shape, n->d_params, n->d_frags, X, B, O, n->stream));
  return FIB_OK;
}

int fib_mlp_gradient(fib_mlp_t* n, const float* X, const float* T, int64_t B, float* grad,
                     float* loss) {
  if (!n || B < 1 || !X || !T) return mfail(FIB_EINVAL, "bad arguments");
  if (int rc = ensure_work(n, fib::mlp_pass_chunks(n->shape, B))) return rc;
  MHIP(fib::launch_mlp_grad(n->shape, n->d_params, n->d_frags, X, T, B, n->d_work,
                            grad ? grad : n->d_grad, loss, nullptr, n->stream));
  return FIB_OK;
}

int fib_mlp_gradient_noalloc(fib_mlp_t* n, const float* X, const float* T, int64_t B,
                             float* grad, float* loss) {
  if (!n || B < 1 || !X || !T) return mfail(FIB_EINVAL, "bad arguments");
  const int64_t chunks = (B + fib::kChunk - 1) / fib::kChunk;
  const int64_t need = chunks * (int64_t)n->shape.n_params + chunks;
  if (need > kNoallocFloats)
    return mfail(FIB_EINVAL, "batch of %lld samples needs %lld scratch floats, more than the "
                 "%lld this entry point holds (at most %lld samples for this network)",
                 (long long)B, (long long)need, (long long)kNoallocFloats,
                 (long long)(kNoallocFloats / (n->shape.n_params + 1) * fib::kChunk));
  float* base = scratch_of(n->device);
  if (!base) return mfail(FIB_ESTATE, "scratch of device %d not set up", n->device);
  MHIP(fib::launch_mlp_grad(n->shape, n->d_params, n->d_frags, X, T, B, base,
                            grad ? grad : n->d_grad, loss, nullptr, n->stream));
  return FIB_OK;
}

int fib_column_stats(const float* A, int64_t rows, int32_t cols, void* stream, double* mean,
                     double* std, float* cmin, float* cmax) {
  if (!A || rows < 1 || cols < 1 || cols > fib::kStatCols || !mean || !std || !cmin || !cmax)
    return mfail(FIB_EINVAL, "bad arguments (1 <= cols <= 64, rows >= 1)");
  hipStream_t st = (hipStream_t)stream;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices)
    return mfail(FIB_EHIP, "no HIP device");
  // the call waits for its results, so it holds its device's work space
  // until then
  std::lock_guard<std::mutex> lock(g_col_mu[dev]);
  void* w = nullptr;
  hipError_t e = hipGetSymbolAddress(&w, HIP_SYMBOL(col_work));
  if (e == hipSuccess)
    e = fib::launch_col_stats(A, rows, cols, static_cast<fib::ColWork*>(w), st);
  fib::ColStats h;
  if (e == hipSuccess) e = hipMemcpyAsync(&h, w, sizeof h, hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e != hipSuccess) return mfail(FIB_EHIP, "column statistics: %s", hipGetErrorString(e));
  for (int k = 0; k < cols; ++k) {
    mean[k] = h.mean[k];
    std[k] = rows > 1 ? std::sqrt(h.sq[k] / (double)(rows - 1)) : 0.0;
    cmin[k] = h.lo[k];
    cmax[k] = h.hi[k];
  }
  return FIB_OK;
}

int fib_normalize_rows(const float* A, int64_t rows, int32_t cols, const float* shift,
                       const float* scale, double extra, float* Y, int32_t ldy, void* stream) {
  if (!A || !Y || !shift || !scale || rows < 0 || cols < 1 || cols > fib::kStatCols || ldy < cols)
    return mfail(FIB_EINVAL, "bad arguments (1 <= cols <= 64, ldy >= cols)");
  if (rows == 0) return FIB_OK;
  hipStream_t st = (hipStream_t)stream;
  fib::ColScale cs{};
  std::copy(shift, shift + cols, cs.shift);
  std::copy(scale, scale + cols, cs.scale);
  hipError_t e = fib::launch_normalize(A, rows, cols, cs, (float)extra, Y, ldy, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e != hipSuccess) return mfail(FIB_EHIP, "normalize: %s", hipGetErrorString(e));
  return FIB_OK;
}

int fib_mlp_adam_step(fib_mlp_t* n, const float* X, const float* T, int64_t B, double lr,
                      float* loss) {
  if (!n || B < 1 || !X || !T || !(lr > 0.0)) return mfail(FIB_EINVAL, "bad arguments");
  if (int rc = ensure_work(n, fib::mlp_pass_chunks(n->shape, B))) return rc;
  const fib::MlpAdam adam{n->d_params, n->d_m, n->d_v, n->d_frags, (float)lr, 0.9f, 0.999f, 1e-8f,
                          n->t + 1};
  MHIP(fib::launch_mlp_grad(n->shape, n->d_params, n->d_frags, X, T, B, n->d_work, n->d_grad,
                            loss, &adam, n->stream));
  n->t += 1;
  return FIB_OK;
}

int fib_mlp_reset_optimizer(fib_mlp_t* n) {
  if (!n) return mfail(FIB_EINVAL, "null network");
  const size_t bytes = sizeof(float) * (size_t)n->shape.n_params;
  MHIP(hipMemsetAsync(n->d_m, 0, bytes, n->stream));
  MHIP(hipMemsetAsync(n->d_v, 0, bytes, n->stream));
  n->t = 0;
  return FIB_OK;
}

}  // extern "C"
