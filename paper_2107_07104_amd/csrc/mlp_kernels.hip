// Surrogate network kernels (gfx950): batched forward pass, backpropagation
// and Adam for a multilayer perceptron with SiLU or ReLU hidden layers and
// a linear output, trained on the mean squared error.  Every matrix product runs on
// the matrix cores (v_mfma_f32_16x16x32_bf16: BF16 operands, FP32
// accumulation); the master weights, moments and gradients are FP32.
//
// Operand layout of v_mfma_f32_16x16x32_bf16 on a 64-lane wave (checked on
// the device): lane l supplies A[l % 16][8 (l / 16) + i] and
// B[8 (l / 16) + i][l % 16] for i = 0..7, and receives
// D[4 (l / 16) + j][l % 16] for j = 0..3.
//
// The weights' BF16 operand fragments are kept beside the FP32 masters (the
// kernels that change the masters write them), so every product reads its
// weights ready for the matrix cores.
#include <algorithm>

#include "../../include/fib.h"
#include "fib_internal.h"
#include "mlp_internal.h"

namespace fib {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef __bf16 v4bf __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float silu(float z) { return z * __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }
__device__ __forceinline__ float silu_grad(float z) {
  const float s = __builtin_amdgcn_rcpf(1.0f + __expf(-z));
  return s * fmaf(z, 1.0f - s, 1.0f);
}
// Hidden activation and its derivative (ReLU'(0) taken as 0).
__device__ __forceinline__ float act_fn(int act, float z) {
  return act == FIB_ACT_RELU ? fmaxf(z, 0.0f) : silu(z);
}
__device__ __forceinline__ float act_grad(int act, float z) {
  return act == FIB_ACT_RELU ? (z > 0.0f ? 1.0f : 0.0f) : silu_grad(z);
}

constexpr int kTS = kChunk + 8;  // row stride of the feature-major operands (BF16)
constexpr int kWaves = 8;        // waves of a training workgroup

// LDS plan of the network kernels (byte offsets).  xs: two sample-major
// operand blocks (kChunk rows of xstride BF16), alternating by layer: layer
// l's activations, on the way back its gradient; xt[l]: the activations of
// layer l < L feature-major (pad[l] rows of kTS BF16), the operand of the
// weight gradients; dt: two blocks of the gradient feature-major; z[l]: the
// pre-activations of hidden layer l in FP32, in the accumulators' own order;
// db: per-feature sums of the gradient over the samples.
struct NetLds {
  int xstride;
  int xs[2];
  int xt[kMaxLayers + 1];
  int dt[2];
  int z[kMaxLayers + 1];
  int db[2];
  int loss;
  int total;
};

static NetLds net_lds(const MlpShape& s, bool grad) {
  NetLds t{};
  int pmax = 0;
  for (int l = 0; l <= s.L; ++l) pmax = s.pad[l] > pmax ? s.pad[l] : pmax;
  t.xstride = pmax + 8;
  int o = 0;
  for (int b = 0; b < 2; ++b) {
    t.xs[b] = o;
    o += 2 * kChunk * t.xstride;
  }
  if (grad) {
    for (int l = 0; l < s.L; ++l) {
      t.xt[l] = o;
      o += 2 * kTS * s.pad[l];
    }
    for (int b = 0; b < 2; ++b) {
      t.dt[b] = o;
      o += 2 * kTS * pmax;
    }
    for (int l = 1; l < s.L; ++l) {
      t.z[l] = o;
      o += 4 * kChunk * s.pad[l];
    }
    for (int b = 0; b < 2; ++b) {
      t.db[b] = o;
      o += 4 * pmax;
    }
    t.loss = o;  // (doubles: every block before it is a multiple of 8 bytes)
    o += 8 * kWaves;
  }
  t.total = o;
  return t;
}

// Chunks one pass of the gradient kernels takes: all of a batch's, up to what
// the fixed scratch of the allocation-free entry point holds, so that both
// entry points sum the same chunks in the same order.
int mlp_pass_chunks(const MlpShape& s, int64_t B) {
  const int64_t chunks = (B + kChunk - 1) / kChunk;
  return (int)std::min<int64_t>(chunks, kScratchFloats / mlp_chunk_floats(s));
}

// Position of parameter W_l[out][in] in the forward operand fragments (rows
// = outputs, K = inputs) and in the backward ones (rows = inputs, K =
// outputs): fragment-major, 64 lanes x 8 BF16 each.
__device__ __forceinline__ int fwd_index(const MlpShape& s, int l, int out, int in) {
  const int frag = (out >> 4) * (s.pad[l - 1] >> 5) + (in >> 5);
  return s.f_off[l] + frag * 512 + (((in >> 3) & 3) * 16 + (out & 15)) * 8 + (in & 7);
}
__device__ __forceinline__ int bwd_index(const MlpShape& s, int l, int out, int in) {
  const int frag = (in >> 4) * (s.pad[l] >> 5) + (out >> 5);
  return s.r_off[l] + frag * 512 + (((out >> 3) & 3) * 16 + (in & 15)) * 8 + (out & 7);
}

// BF16 operand fragments of every weight, from the FP32 parameters (the
// padding stays zero from the network's creation).
__global__ __launch_bounds__(256) void k_mlp_pack(MlpShape s, const float* __restrict__ params,
                                                  __bf16* __restrict__ frags) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  int l = 1;
  while (l <= s.L && e >= s.b_off[l] + s.size[l]) ++l;
  if (l > s.L || e >= s.b_off[l]) return;  // past the end, or a bias
  const int k = e - s.w_off[l], out = k / s.size[l - 1], in = k % s.size[l - 1];
  const __bf16 w = (__bf16)params[e];
  frags[fwd_index(s, l, out, in)] = w;
  if (l > 1) frags[bwd_index(s, l, out, in)] = w;
}

// acc += A B over K = 32 kb: A's fragments of one 16-row block from global
// memory, B's columns (the 16 samples of half sb) from a sample-major block.
__device__ __forceinline__ v4f block_product(const v8bf* __restrict__ a, const __bf16* xs,
                                             int xstride, int kb, int sb, int lane) {
  const __bf16* row = xs + (16 * sb + (lane & 15)) * xstride + 8 * (lane >> 4);
  v4f acc = {0.0f, 0.0f, 0.0f, 0.0f};
  // four weight fragments in flight at a time
  for (int k0 = 0; k0 < kb; k0 += 4) {
    v8bf av[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (k0 + q < kb) av[q] = a[(k0 + q) * 64 + lane];
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (k0 + q < kb)
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            av[q], *reinterpret_cast<const v8bf*>(row + 32 * (k0 + q)), acc, 0, 0, 0);
  }
  return acc;
}

// Stores a lane's four features f .. f + 3 of sample n as BF16 operands,
// sample-major and (xt non-null) feature-major.
__device__ __forceinline__ void store_operand(const v4f& v, __bf16* xs, int xstride, __bf16* xt,
                                              int n, int f) {
  const v4bf b = __builtin_convertvector(v, v4bf);
  *reinterpret_cast<v4bf*>(xs + n * xstride + f) = b;
  if (xt) {
#pragma unroll
    for (int j = 0; j < 4; ++j) xt[(f + j) * kTS + n] = b[j];
  }
}

// Sum of v over the 16 samples of a lane row, one after the other from
// `carry`, in the row's last lane: FP32 sums keep one fixed order over the
// batch's samples.
__device__ __forceinline__ float scan_samples(float v, float carry, int r) {
  v += r == 0 ? carry : 0.0f;
  float acc = v;
#pragma unroll
  for (int k = 1; k < 16; ++k)  // lane k takes lane k - 1's sum (row_shr:1, 0 into lane 0)
    acc = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
              0, __builtin_bit_cast(int, acc), 0x111, 0xf, 0xf, true)) + v;
  return acc;
}

// v plus the value of another lane (CTRL, ROWS: a DPP move and the rows it
// writes; 0 elsewhere).
template <int CTRL, int ROWS>
__device__ __forceinline__ double plus_lane(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, ROWS, 0xf, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, ROWS, 0xf, true);
  return v + __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// Sum over the wave, in lane 63 (shuffles through LDS took 0.4 us a chunk).
__device__ __forceinline__ double wave_sum(double v) {
  v = plus_lane<0x111, 0xf>(v);  // row_shr:1, 2, 4, 8
  v = plus_lane<0x112, 0xf>(v);
  v = plus_lane<0x114, 0xf>(v);
  v = plus_lane<0x118, 0xf>(v);
  v = plus_lane<0x142, 0xa>(v);     // row_bcast:15 into rows 1 and 3
  return plus_lane<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
}

// Sums of a lane's four features over the chunk's samples (v[0]: the first
// 16, v[1]: the others) to db[f .. f + 3].
__device__ __forceinline__ void sum_samples(const v4f (&v)[2], float* db, int f, int lane) {
  v4f s;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float half = scan_samples(v[0][j], 0.0f, lane & 15);
    s[j] = scan_samples(v[1][j], __shfl(half, lane | 15), lane & 15);
  }
  if ((lane & 15) == 15) *reinterpret_cast<v4f*>(db + f) = s;
}

// The network kernels: a workgroup of eight waves takes a chunk of kChunk =
// 32 samples (chunk0 + blockIdx.x, + gridDim.x, ...).  Every product of a
// layer is cut into units of 16 features x 16 samples that the waves share;
// weights are read as ready-made BF16 fragments (16 bytes a lane, from L2),
// activations and gradients pass through LDS as BF16, in the two orders the
// products need.  GRAD: backpropagation of loss = sum (O - T)^2 / (2 B n_out)
// down to the first layer's pre-activations; the operands of the weight
// gradients (activations and gradients, feature-major) go to `ops` as
// fragments, the chunk's bias gradients to `db` and its loss to loss_part,
// all indexed by blockIdx.x, for k_mlp_update.
//
// Bound by the chain of 2 L layer phases and their barriers (a chunk is 4
// MFLOP, half a microsecond of a compute unit's matrix cores), so the chunk
// is small enough that a training batch of 8192 fills all 256 compute units.
// On the 57-128-128-57 network that batch's gradient took 553 us with one
// wave per chunk (FP32 operands in LDS, 115 KB: one wave per compute unit)
// and every chunk's whole weight gradient (32 MB in all) written out and
// summed; 50 us with these workgroups doing the same; 35 us (this kernel 21)
// with the operands (10 MB) written instead and contracted by k_mlp_update.
template <bool GRAD>
__global__ __launch_bounds__(64 * kWaves) void k_mlp(MlpShape s, NetLds t,
                                                     const float* __restrict__ params,
                                                     const __bf16* __restrict__ frags,
                                                     const float* __restrict__ X,
                                                     const float* __restrict__ T, int64_t B,
                                                     int64_t chunk0, float* __restrict__ O,
                                                     v8bf* __restrict__ ops,
                                                     float* __restrict__ db_part,
                                                     float* __restrict__ loss_part) {
  extern __shared__ __align__(16) char lds[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, g = lane >> 4;
  const int nL = s.size[s.L];
  const float scale = 1.0f / ((float)B * (float)nL);
  const int64_t chunks = (B + kChunk - 1) / kChunk;
  double lsum = 0.0;
  for (int64_t chunk = chunk0 + blockIdx.x; chunk < chunks; chunk += gridDim.x) {
    const int64_t s0 = chunk * kChunk;
    // inputs, zero padded: each wave takes four samples
    {
      __bf16* xs = reinterpret_cast<__bf16*>(lds + t.xs[0]);
      __bf16* xt = GRAD ? reinterpret_cast<__bf16*>(lds + t.xt[0]) : nullptr;
      const int n0 = s.size[0], p0 = s.pad[0];
      for (int j = lane; j < p0; j += 64) {
        float x[kChunk / kWaves];
#pragma unroll
        for (int q = 0; q < kChunk / kWaves; ++q) {
          const int64_t sr = s0 + wave * (kChunk / kWaves) + q;
          x[q] = sr < B && j < n0 ? X[sr * n0 + j] : 0.0f;
        }
#pragma unroll
        for (int q = 0; q < kChunk / kWaves; ++q) {
          const int i = wave * (kChunk / kWaves) + q;
          const __bf16 b = (__bf16)x[q];
          xs[i * t.xstride + j] = b;
          if (GRAD) xt[j * kTS + i] = b;
        }
      }
    }
    __syncthreads();
    for (int l = 1; l <= s.L; ++l) {
      const __bf16* src = reinterpret_cast<const __bf16*>(lds + t.xs[(l - 1) & 1]);
      __bf16* dst = reinterpret_cast<__bf16*>(lds + t.xs[l & 1]);
      const int nout = s.size[l], ob_n = s.pad[l] >> 4, kb_n = s.pad[l - 1] >> 5;
      const v8bf* fr = reinterpret_cast<const v8bf*>(frags + s.f_off[l]);
      const float* bias = params + s.b_off[l];
      // the last layer's gradient sums need both halves of the samples in one
      // wave; the other layers' units go to whichever wave is next
      const bool pair = GRAD && l == s.L;
      for (int u = wave; u < (pair ? ob_n : 2 * ob_n); u += kWaves) {
        const int ob = u % ob_n, f = 16 * ob + 4 * g;
        float bj[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) bj[j] = f + j < nout ? bias[f + j] : 0.0f;
        if (pair) {
          v4f d[2];
          float tj[2][4];
#pragma unroll
          for (int sb = 0; sb < 2; ++sb)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              const int64_t sr = s0 + 16 * sb + r;
              tj[sb][j] = sr < B && f + j < nout ? T[sr * nout + f + j] : 0.0f;
            }
#pragma unroll
          for (int sb = 0; sb < 2; ++sb) {
            const int n = 16 * sb + r;
            v4f v = block_product(fr + (int64_t)ob * kb_n * 64, src, t.xstride, kb_n, sb, lane);
            // output gradient (O - T) / (B n_L), zero on padding and past B
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              const float o = v[j] + bj[j];
              const float diff = s0 + n < B && f + j < nout ? o - tj[sb][j] : 0.0f;
              lsum += (double)diff * diff;
              d[sb][j] = diff * scale;
            }
            store_operand(d[sb], dst, t.xstride, reinterpret_cast<__bf16*>(lds + t.dt[l & 1]), n, f);
          }
          sum_samples(d, reinterpret_cast<float*>(lds + t.db[l & 1]), f, lane);
          continue;
        }
        const int sb = u / ob_n, n = 16 * sb + r;
        v4f v = block_product(fr + (int64_t)ob * kb_n * 64, src, t.xstride, kb_n, sb, lane);
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] += bj[j];
        if (l < s.L) {
          if (GRAD)
            *reinterpret_cast<v4f*>(lds + t.z[l] + 16 * ((sb * ob_n + ob) * 64 + lane)) = v;
#pragma unroll
          for (int j = 0; j < 4; ++j)  // padding stays 0 where an activation is not finite
            v[j] = f + j < nout ? act_fn(s.act, v[j]) : 0.0f;
          store_operand(v, dst, t.xstride,
                        GRAD ? reinterpret_cast<__bf16*>(lds + t.xt[l]) : nullptr, n, f);
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (s0 + n < B && f + j < nout) O[(s0 + n) * nout + f + j] = v[j];
        }
      }
      __syncthreads();
    }
    if constexpr (GRAD) {
      // fragments of 16 features x 32 samples from a feature-major block
      auto put = [&](const __bf16* xt, int frag0, int n) {
        v8bf* out = ops + ((int64_t)blockIdx.x * s.n_ops + frag0) * 64 + lane;
        for (int q = wave; q < n; q += kWaves)
          out[q * 64] = *reinterpret_cast<const v8bf*>(xt + (16 * q + r) * kTS + 8 * g);
      };
      for (int l = s.L; l >= 1; --l) {
        const int nin = s.size[l - 1], nout = s.size[l];
        if (l > 1) {
          // gradient of layer l - 1: (W_l^T dz_l) act'(z_{l-1})
          const __bf16* src = reinterpret_cast<const __bf16*>(lds + t.xs[l & 1]);
          __bf16* dst = reinterpret_cast<__bf16*>(lds + t.xs[(l - 1) & 1]);
          const int ib_n = s.pad[l - 1] >> 4, kb_n = s.pad[l] >> 5;
          const v8bf* fr = reinterpret_cast<const v8bf*>(frags + s.r_off[l]);
          for (int ib = wave; ib < ib_n; ib += kWaves) {
            const int f = 16 * ib + 4 * g;
            v4f d[2];
#pragma unroll
            for (int sb = 0; sb < 2; ++sb) {
              d[sb] = block_product(fr + (int64_t)ib * kb_n * 64, src, t.xstride, kb_n, sb, lane);
              const v4f z = *reinterpret_cast<const v4f*>(
                  lds + t.z[l - 1] + 16 * ((sb * ib_n + ib) * 64 + lane));
#pragma unroll
              for (int j = 0; j < 4; ++j)
                d[sb][j] = f + j < nin ? d[sb][j] * act_grad(s.act, z[j]) : 0.0f;
              store_operand(d[sb], dst, t.xstride,
                            reinterpret_cast<__bf16*>(lds + t.dt[(l - 1) & 1]), 16 * sb + r, f);
            }
            sum_samples(d, reinterpret_cast<float*>(lds + t.db[(l - 1) & 1]), f, lane);
          }
        }
        put(reinterpret_cast<const __bf16*>(lds + t.xt[l - 1]), s.a_ops[l], (nin + 15) >> 4);
        put(reinterpret_cast<const __bf16*>(lds + t.dt[l & 1]), s.d_ops[l], (nout + 15) >> 4);
        const float* db = reinterpret_cast<const float*>(lds + t.db[l & 1]);
        float* rb = db_part + (int64_t)blockIdx.x * s.n_bias + s.bias_off[l];
        for (int j = threadIdx.x; j < nout; j += 64 * kWaves) rb[j] = db[j];
        __syncthreads();
      }
      // (launched with one chunk per workgroup)
      lsum = wave_sum(lsum);
      double* sl = reinterpret_cast<double*>(lds + t.loss);
      if (lane == 63) sl[wave] = lsum;
      __syncthreads();
      if (threadIdx.x == 0) {
        double a = 0.0;
        for (int w = 0; w < kWaves; ++w) a += sl[w];
        loss_part[blockIdx.x] = (float)(0.5 * a / ((double)B * nL));
      }
      return;
    }
  }
}

// Adam of one training step; p null: gradient only.
struct AdamArgs {
  float* p;
  float* m;
  float* v;
  __bf16* frags;
  float lr, b1, b2, eps, bc1, bc2;
};

// Position of a parameter (in < 0: a bias).
__device__ __forceinline__ int param_index(const MlpShape& s, int l, int out, int in) {
  return in < 0 ? s.b_off[l] + out : s.w_off[l] + out * s.size[l - 1] + in;
}

// The gradient of one parameter is ready: grad, and with Adam the FP32
// master and its BF16 fragments.
__device__ __forceinline__ void finish_param(const MlpShape& s, int l, int out, int in, float acc,
                                             float* __restrict__ grad, const AdamArgs& ad) {
  const int p = param_index(s, l, out, in);
  grad[p] = acc;
  if (!ad.p) return;
  const float mm = fmaf(ad.b1, ad.m[p], (1.0f - ad.b1) * acc);
  const float vv = fmaf(ad.b2, ad.v[p], (1.0f - ad.b2) * acc * acc);
  ad.m[p] = mm;
  ad.v[p] = vv;
  const float mh = mm / ad.bc1, vh = vv / ad.bc2;
  const float q = ad.p[p] - ad.lr * mh / (sqrtf(vh) + ad.eps);
  ad.p[p] = q;
  if (in >= 0) {
    ad.frags[fwd_index(s, l, out, in)] = (__bf16)q;
    if (l > 1) ad.frags[bwd_index(s, l, out, in)] = (__bf16)q;
  }
}

constexpr int kUpdWaves = 16;    // waves of an update workgroup
constexpr int kAheadChunks = 8;  // chunks of each wave whose operands are in flight

// Gradients from the operands of a pass: block b < n_tiles contracts one 16
// x 16 tile of some dW_l = sum over chunks of dz_l act_{l-1}^T, a wave per
// chunk and sixteen at a time (one instruction per chunk, K = its 32 samples;
// eight chunks' operands of every wave in flight), which 256 threads add up in
// the chunks' order through LDS; the blocks after the tiles sum 64 biases
// each over the chunks, the last one the loss (in FP64).  Every sum has one
// fixed order, over the samples of a chunk and then the chunks, so gradients are
// deterministic and do not depend on how the work is split (Adam's first
// steps are signs of gradients: an order of its own would send training
// elsewhere).  add: a later pass of a batch too large for one, which carries
// the sums on; the parameters are updated (ad.p non-null) with the last.
//
// Bound by reading the operands, 2 KB per tile and chunk (64 MB from the
// last-level cache for a batch of 8192 on the 57-128-128-57 network), and then
// by the ordered sums: 15 us with Adam (10 us with each wave's chunks summed
// in its accumulators); one thread per parameter walking 256 whole gradients
// one by one took 71 us, and Adam a launch of 5 us more.
__global__ __launch_bounds__(64 * kUpdWaves) void k_mlp_update(
    MlpShape s, const v8bf* __restrict__ ops, const float* __restrict__ db_part,
    const float* __restrict__ loss_part, int chunks, int add, float* __restrict__ grad,
    float* __restrict__ loss, AdamArgs ad) {
  __shared__ __align__(16) float sh[2][kUpdWaves][256];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, w = threadIdx.x;
  float sum = 0.0f;
  if ((int)blockIdx.x < s.n_tiles) {
    int l = 1, tile = blockIdx.x, ib_n;
    for (;; ++l) {
      ib_n = (s.size[l - 1] + 15) >> 4;
      const int nt = ((s.size[l] + 15) >> 4) * ib_n;
      if (tile < nt) break;
      tile -= nt;
    }
    const int ob = tile / ib_n, ib = tile % ib_n;
    // thread w < 256: element w of the tile
    const int out = 16 * ob + 4 * (w >> 6) + (w & 3), in = 16 * ib + ((w >> 2) & 15);
    const bool mine = w < 256 && out < s.size[l] && in < s.size[l - 1];
    if (add && mine) sum = grad[param_index(s, l, out, in)];
    const v8bf* pa = ops + (int64_t)(s.d_ops[l] + ob) * 64 + lane;
    const v8bf* pb = ops + (int64_t)(s.a_ops[l] + ib) * 64 + lane;
    const int64_t stride = (int64_t)s.n_ops * 64;
    int par = 0;
    for (int c0 = 0; c0 < chunks; c0 += kAheadChunks * kUpdWaves) {
      v8bf a[kAheadChunks], b[kAheadChunks];
#pragma unroll
      for (int q = 0; q < kAheadChunks; ++q) {
        const int c = c0 + q * kUpdWaves + wave;
        if (c < chunks) {
          a[q] = pa[c * stride];
          b[q] = pb[c * stride];
        }
      }
#pragma unroll
      for (int q = 0; q < kAheadChunks; ++q) {
        const int r0 = c0 + q * kUpdWaves;
        if (r0 >= chunks) break;
        if (r0 + wave < chunks) {
          const v4f zero = {0.0f, 0.0f, 0.0f, 0.0f};
          *reinterpret_cast<v4f*>(&sh[par][wave][4 * lane]) =
              __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[q], b[q], zero, 0, 0, 0);
        }
        __syncthreads();
        if (w < 256) {
          const int n = min(kUpdWaves, chunks - r0);
          for (int v = 0; v < n; ++v) sum += sh[par][v][w];
        }
        par ^= 1;
      }
    }
    if (mine) finish_param(s, l, out, in, sum, grad, ad);
    return;
  }
  const int j = ((int)blockIdx.x - s.n_tiles) * 64 + lane;
  int l = 1;
  while (l < s.L && j >= s.bias_off[l + 1]) ++l;
  if (add && j < s.n_bias) sum = grad[param_index(s, l, j - s.bias_off[l], -1)];
  // the waves fetch four chunks each, the first one adds them in order
  for (int c0 = 0; c0 < chunks; c0 += 4 * kUpdWaves) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int c = c0 + 4 * wave + q;
      sh[0][wave][64 * q + lane] = c < chunks && j < s.n_bias ? db_part[(int64_t)c * s.n_bias + j]
                                                              : 0.0f;
    }
    __syncthreads();
    if (wave == 0) {
      const int n = min(4 * kUpdWaves, chunks - c0);
      for (int v = 0; v < n; ++v) sum += sh[0][v >> 2][64 * (v & 3) + lane];
    }
    __syncthreads();
  }
  if (wave > 0) return;
  if (blockIdx.x + 1 == gridDim.x && loss) {
    double a = 0.0;
    for (int c = lane; c < chunks; c += 64) a += (double)loss_part[c];
    for (int off = 32; off > 0; off >>= 1) a += __shfl_xor(a, off);
    if (lane == 0) loss[0] = (float)(add ? loss[0] + a : a);
  }
  if (j < s.n_bias) finish_param(s, l, j - s.bias_off[l], -1, sum, grad, ad);
}

// ---------------------------------------------------------------------------
// Training data: column statistics and normalization of row-major arrays
// ---------------------------------------------------------------------------

// Row-major arrays of at most 64 columns are walked flat: a block's threads
// cover whole rows (floor(256 / width) of them at a time), thread t keeps
// column t % width, so that loads are coalesced whatever the width and no
// element needs a division.  kAhead rows of each thread are in flight.
constexpr int kColThreads = 256, kAhead = 8;

// Per-block partial statistics of the columns of A (rows x cols): block b
// takes rows [b rb, (b + 1) rb).  Without `mean` it sums x and records min and
// max; with `mean` it sums (x - mean)^2.  FP64 sums, combined in a fixed
// order, so the statistics are deterministic.  Bound by reading A: 135 MB
// (592 400 x 57) in 42 us, and in 22 us the second time (partly from the
// last-level cache); one column per lane and one row per wave took 66 us.
template <bool SQUARES>
__global__ __launch_bounds__(kColThreads) void k_col_partial(
    const float* __restrict__ A, int64_t rows, int cols, int64_t rb,
    const double* __restrict__ mean, double* __restrict__ part, float* __restrict__ pmin,
    float* __restrict__ pmax) {
  __shared__ double ssum[kColThreads];
  __shared__ float smin[kColThreads], smax[kColThreads];
  const int t = threadIdx.x, step = kColThreads / cols;
  const int x = t % cols, y = t / cols;
  double acc = 0.0;
  float lo = __builtin_inff(), hi = -__builtin_inff();
  if (y < step) {
    const double m = SQUARES ? mean[x] : 0.0;
    auto take = [&](float v) {
      if (SQUARES) {
        const double d = (double)v - m;
        acc += d * d;
      } else {
        acc += (double)v;
        lo = fminf(lo, v);
        hi = fmaxf(hi, v);
      }
    };
    const int64_t r0 = (int64_t)blockIdx.x * rb;
    const int64_t r1 = r0 + rb < rows ? r0 + rb : rows;
    int64_t r = r0 + y;
    for (; r + (kAhead - 1) * step < r1; r += kAhead * step) {
      float v[kAhead];
#pragma unroll
      for (int q = 0; q < kAhead; ++q) v[q] = A[(r + q * step) * cols + x];
#pragma unroll
      for (int q = 0; q < kAhead; ++q) take(v[q]);
    }
    for (; r < r1; r += step) take(A[r * cols + x]);
  }
  ssum[t] = acc;
  if (!SQUARES) {
    smin[t] = lo;
    smax[t] = hi;
  }
  __syncthreads();
  if (t < cols) {
    for (int j = 1; j < step; ++j) {
      acc += ssum[t + j * cols];
      if (!SQUARES) {
        lo = fminf(lo, smin[t + j * cols]);
        hi = fmaxf(hi, smax[t + j * cols]);
      }
    }
    part[(int64_t)blockIdx.x * cols + t] = acc;
    if (!SQUARES) {
      pmin[(int64_t)blockIdx.x * cols + t] = lo;
      pmax[(int64_t)blockIdx.x * cols + t] = hi;
    }
  }
}

// Column blockIdx.x's total over the blocks, in a fixed order (a thread every
// 256th block, then a tree): the mean with the minimum and maximum, or the
// sum of squares.  One wave walking 1024 blocks one by one took 288 us for
// 57 columns; this 9 us (6 without minimum and maximum).
template <bool SQUARES>
__global__ __launch_bounds__(kColThreads) void k_col_final(
    const double* __restrict__ part, const float* __restrict__ pmin,
    const float* __restrict__ pmax, int blocks, int cols, int64_t rows, ColStats* __restrict__ st) {
  __shared__ double ssum[kColThreads];
  __shared__ float smin[kColThreads], smax[kColThreads];
  const int t = threadIdx.x, x = blockIdx.x;
  double acc = 0.0;
  float lo = __builtin_inff(), hi = -__builtin_inff();
  for (int b = t; b < blocks; b += kColThreads) {
    acc += part[(int64_t)b * cols + x];
    if (!SQUARES) {
      lo = fminf(lo, pmin[(int64_t)b * cols + x]);
      hi = fmaxf(hi, pmax[(int64_t)b * cols + x]);
    }
  }
  ssum[t] = acc;
  smin[t] = lo;
  smax[t] = hi;
  __syncthreads();
  for (int d = kColThreads / 2; d > 0; d >>= 1) {
    if (t < d) {
      ssum[t] += ssum[t + d];
      smin[t] = fminf(smin[t], smin[t + d]);
      smax[t] = fmaxf(smax[t], smax[t + d]);
    }
    __syncthreads();
  }
  if (t == 0) {
    if (SQUARES) {
      st->sq[x] = ssum[0];
    } else {
      st->mean[x] = ssum[0] / (double)rows;
      st->lo[x] = smin[0];
      st->hi[x] = smax[0];
    }
  }
}

// Y[r][k] = (A[r][k] - shift[k]) * scale[k] for k < cols, Y[r][cols] = extra
// when ldy > cols, other columns of Y untouched.  Bound by the copy: 270 MB
// read and written (592 400 x 57) in 59 us; one element per thread with
// its 64-bit division took 89 us.
__global__ __launch_bounds__(kColThreads) void k_normalize(const float* __restrict__ A,
                                                           int64_t rows, int cols, ColScale cs,
                                                           float extra, float* __restrict__ Y,
                                                           int ldy) {
  const int t = threadIdx.x, w = ldy > cols ? cols + 1 : cols, step = kColThreads / w;
  const int k = t % w, y = t / w;
  if (y >= step) return;
  const bool from = k < cols;
  const float sh = from ? cs.shift[k] : 0.0f, sc = from ? cs.scale[k] : 0.0f;
  const int64_t stride = (int64_t)gridDim.x * step;
  int64_t r = (int64_t)blockIdx.x * step + y;
  for (; r + (kAhead - 1) * stride < rows; r += kAhead * stride) {
    float v[kAhead];
#pragma unroll
    for (int q = 0; q < kAhead; ++q) v[q] = from ? A[(r + q * stride) * cols + k] : 0.0f;
#pragma unroll
    for (int q = 0; q < kAhead; ++q)
      Y[(r + q * stride) * ldy + k] = from ? (v[q] - sh) * sc : extra;
  }
  for (; r < rows; r += stride) Y[r * ldy + k] = from ? (A[r * cols + k] - sh) * sc : extra;
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------

hipError_t launch_col_stats(const float* A, int64_t rows, int cols, ColWork* w, hipStream_t st) {
  const int blocks = (int)std::min<int64_t>(kStatBlocks, (rows + 63) / 64);
  const int64_t rb = (rows + blocks - 1) / blocks;
  const dim3 g((unsigned)blocks), gc((unsigned)cols), blk(kColThreads);
  hipLaunchKernelGGL(k_col_partial<false>, g, blk, 0, st, A, rows, cols, rb,
                     (const double*)nullptr, w->part, w->pmin, w->pmax);
  hipLaunchKernelGGL(k_col_final<false>, gc, blk, 0, st, w->part, w->pmin, w->pmax, blocks, cols,
                     rows, &w->stats);
  hipLaunchKernelGGL(k_col_partial<true>, g, blk, 0, st, A, rows, cols, rb, w->stats.mean, w->part,
                     (float*)nullptr, (float*)nullptr);
  hipLaunchKernelGGL(k_col_final<true>, gc, blk, 0, st, w->part, (const float*)nullptr,
                     (const float*)nullptr, blocks, cols, rows, &w->stats);
  return hipGetLastError();
}

hipError_t launch_normalize(const float* A, int64_t rows, int cols, const ColScale& cs, float extra,
                            float* Y, int ldy, hipStream_t st) {
  if (rows == 0) return hipSuccess;
  const int step = kColThreads / (ldy > cols ? cols + 1 : cols);
  const int64_t need = (rows + step - 1) / step;
  hipLaunchKernelGGL(k_normalize, dim3((unsigned)std::min<int64_t>(need, 4096)), dim3(kColThreads),
                     0, st, A, rows, cols, cs, extra, Y, ldy);
  return hipGetLastError();
}

hipError_t launch_mlp_pack(const MlpShape& s, const float* params, void* frags, hipStream_t st) {
  hipLaunchKernelGGL(k_mlp_pack, dim3((unsigned)((s.n_params + 255) / 256)), dim3(256), 0, st, s,
                     params, static_cast<__bf16*>(frags));
  return hipGetLastError();
}

hipError_t launch_mlp_forward(const MlpShape& s, const float* params, const void* frags,
                              const float* X, int64_t B, float* O, hipStream_t st) {
  if (B == 0) return hipSuccess;
  // a workgroup per chunk, up to the grid's limit (the kernel strides on)
  const unsigned grid = (unsigned)std::min<int64_t>((B + kChunk - 1) / kChunk, 1 << 20);
  const NetLds t = net_lds(s, false);
  hipLaunchKernelGGL(k_mlp<false>, dim3(grid), dim3(64 * kWaves), t.total, st, s, t, params,
                     static_cast<const __bf16*>(frags), X, (const float*)nullptr, B, (int64_t)0, O,
                     (v8bf*)nullptr, (float*)nullptr, (float*)nullptr);
  return hipGetLastError();
}

hipError_t launch_mlp_grad(const MlpShape& s, const float* params, const void* frags,
                           const float* X, const float* T, int64_t B, float* work, float* grad,
                           float* loss, const MlpAdam* adam, hipStream_t st) {
  const int64_t chunks = (B + kChunk - 1) / kChunk;
  const int pass = mlp_pass_chunks(s, B);
  v8bf* ops = reinterpret_cast<v8bf*>(work);
  float* db = work + (int64_t)pass * s.n_ops * 256;
  float* loss_part = db + (int64_t)pass * s.n_bias;
  const NetLds t = net_lds(s, true);
  const dim3 ugrid((unsigned)(s.n_tiles + (s.n_bias + 63) / 64));
  for (int64_t c0 = 0; c0 < chunks; c0 += pass) {
    const int n = (int)std::min<int64_t>(pass, chunks - c0);
    hipLaunchKernelGGL(k_mlp<true>, dim3(n), dim3(64 * kWaves), t.total, st, s, t, params,
                       static_cast<const __bf16*>(frags), X, T, B, c0, (float*)nullptr, ops, db,
                       loss_part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    AdamArgs ad{};
    if (adam && c0 + n == chunks) {
      ad = AdamArgs{adam->params, adam->m, adam->v, static_cast<__bf16*>(adam->frags), adam->lr,
                    adam->b1, adam->b2, adam->eps, 1.0f - powf(adam->b1, (float)adam->t),
                    1.0f - powf(adam->b2, (float)adam->t)};
    }
    hipLaunchKernelGGL(k_mlp_update, ugrid, dim3(64 * kUpdWaves), 0, st, s, ops, db, loss_part, n,
                       c0 > 0 ? 1 : 0, grad, loss, ad);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace fib
