// Internal shape description of the surrogate network, shared by the host
// runtime and the network kernels.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace fib {

constexpr int kMaxLayers = 6;  // weight layers
constexpr int kChunk = 32;     // samples per training workgroup
constexpr int kPad = 32;       // feature dimensions are padded to multiples of this

// Flat parameter layout (FP32): for every layer l = 1..L the weight matrix
// W_l (size[l] x size[l-1], row-major) followed by the bias b_l.
struct MlpShape {
  int L;                        // number of weight layers
  int size[kMaxLayers + 1];     // features per layer, size[0] = inputs
  int pad[kMaxLayers + 1];      // size rounded up to kPad
  int w_off[kMaxLayers + 1];    // offset of W_l in the flat parameters
  int b_off[kMaxLayers + 1];    // offset of b_l
  int n_params;
  // BF16 operand fragments (elements): forward ones of W_l, backward (transposed)
  // ones of l > 1, and their total
  int f_off[kMaxLayers + 1];
  int r_off[kMaxLayers + 1];
  int n_frag;
  // operands of the weight gradients a chunk leaves (fragments of 16 features
  // x 32 samples): the inputs of layer l from a_ops[l], its gradients from
  // d_ops[l]; the 16 x 16 tiles of all W_l; and all biases, layer l's from
  // bias_off[l]
  int a_ops[kMaxLayers + 1];
  int d_ops[kMaxLayers + 1];
  int n_ops;
  int n_tiles;
  int bias_off[kMaxLayers + 1];
  int n_bias;
  int act;                      // hidden activation: FIB_ACT_SILU or FIB_ACT_RELU
};

// Floats of work space per chunk: its operand fragments (512 BF16 each), bias
// gradients and loss.
inline int64_t mlp_chunk_floats(const MlpShape& s) { return (int64_t)s.n_ops * 256 + s.n_bias + 1; }
// Floats of the allocation-free entry point's fixed scratch: the work space
// of at least 150 chunks whatever the widths (794 chunks of the 57-128-128-57
// network's, batches of 25 408).
constexpr int64_t kScratchFloats = (int64_t)1 << 23;  // 32 MiB per device
int mlp_pass_chunks(const MlpShape& s, int64_t B);

// One Adam step: the masters, their moments and fragments.
struct MlpAdam {
  float *params, *m, *v;
  void* frags;
  float lr, b1, b2, eps;
  int64_t t;
};

// BF16 operand fragments of the parameters.
hipError_t launch_mlp_pack(const MlpShape& s, const float* params, void* frags, hipStream_t st);
hipError_t launch_mlp_forward(const MlpShape& s, const float* params, const void* frags,
                              const float* X, int64_t B, float* O, hipStream_t st);
// Gradient into grad and loss into loss (nullable), and with `adam` the
// parameter update; work holds mlp_pass_chunks x mlp_chunk_floats values.
hipError_t launch_mlp_grad(const MlpShape& s, const float* params, const void* frags,
                           const float* X, const float* T, int64_t B, float* work, float* grad,
                           float* loss, const MlpAdam* adam, hipStream_t st);
// Column statistics: results, and their work space in device memory.
constexpr int kStatCols = 64, kStatBlocks = 2048;
struct ColStats {
  double mean[kStatCols], sq[kStatCols];  // sq: sum of squared deviations
  float lo[kStatCols], hi[kStatCols];
};
struct ColWork {
  ColStats stats;
  double part[kStatBlocks * kStatCols];
  float pmin[kStatBlocks * kStatCols], pmax[kStatBlocks * kStatCols];
};
// Statistics of the columns of A (rows x cols, cols <= kStatCols) into
// w->stats (two passes over A).
hipError_t launch_col_stats(const float* A, int64_t rows, int cols, ColWork* w, hipStream_t st);
// Shift and scale of every column, passed to the kernel by value.
struct ColScale {
  float shift[kStatCols], scale[kStatCols];
};
// Y[r][k] = (A[r][k] - shift[k]) scale[k]; Y[r][cols] = extra if ldy > cols.
hipError_t launch_normalize(const float* A, int64_t rows, int cols, const ColScale& cs, float extra,
                            float* Y, int ldy, hipStream_t st);

}  // namespace fib

struct fib_mlp;
namespace fib {
// Shape and device parameters of a network object (mlp_api.hip).
const MlpShape& mlp_shape(const fib_mlp* n);
const float* mlp_device_params(const fib_mlp* n);
hipStream_t mlp_stream(const fib_mlp* n);

}  // namespace fib
