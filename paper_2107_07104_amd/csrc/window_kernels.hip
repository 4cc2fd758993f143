// Windowed diffusion and whole split steps on windows of nodes (gfx950).
//
// The diffusion step V+ = V + A^{-1} dt L V couples a node to its neighbours
// through the inverse of a tridiagonal matrix with constant rows, whose
// entries fall off geometrically: on an endless fiber A^{-1} is the
// convolution with g_0 lambda^|k|, lambda the smaller root of w l^2 - (1 + 2
// w) l + w = 0 for row weight w = theta c dt / h^2, g_0 = 1 / sqrt(1 + 4 w).
// The no-flux ends (one-sided rows of doubled weight) make a fiber the even
// reflection of itself about its end nodes, so A^{-1} on a fiber is the same
// convolution with reflected indices, and the whole step is
//   V+_i = V_i + sum_{k = 1..W} h_k ((V_{i-k} - V_i) + (V_{i+k} - V_i)),
//   h_k = w g_0 (1 - lambda)^2 lambda^{k - 1} / theta,
// in increment form: a constant field stays exactly.  W is where lambda^W
// falls below 2^-40, the bound at which the partitioned solve stops its
// parallel cyclic reduction too: 9 at dt = 1e-3 ms, 7 at 5e-4 ms, 15 at 5e-3 ms
// (sigma = 3.828 mS/cm, h = 0.01 cm).  No barrier chain and no whole fiber per
// workgroup: a node needs 2 W neighbours.
//
// That locality also blocks time: a workgroup that holds the states of a
// window of nodes can take several split steps at once, each of which spoils W
// nodes at either end; neighbouring windows overlap by
// what is spoiled and the overlap is computed twice.
#include <algorithm>
#include <cmath>

#include "fib_internal.h"
#include "hh_model.h"

namespace fib {

namespace {

// Values reserved around a window in LDS for the reads of its outermost
// nodes (their results are spoiled).
template <int W>
constexpr int kPad = W;

// The diffusion of one node from its window's V in LDS (s: the node's own
// slot), distances dl and dr to its fiber's ends (clipped; W or more apart in
// sum).  Smallest terms first.  The reflected form reads the values an
// extended fiber would hold, so both forms give the same bits.
template <int W>
__device__ __forceinline__ float reflected(const float* s, float V, int dl, int dr,
                                           const WindowStencil& st) {
  float d = 0.0f;
#pragma unroll
  for (int k = W; k >= 1; --k) {
    const float l = s[k <= dl ? -k : k - 2 * dl], r = s[k <= dr ? k : 2 * dr - k];
    d = fmaf(st.h[k - 1], (l - V) + (r - V), d);
  }
  return V + d;
}

template <int W>
__device__ __forceinline__ float window_diffuse(const float* s, float V, int dl, int dr,
                                                const WindowStencil& st) {
  if (__any(dl < W || dr < W)) return reflected<W>(s, V, dl, dr, st);
  float d = 0.0f;
#pragma unroll
  for (int k = W; k >= 1; --k) d = fmaf(st.h[k - 1], (s[-k] - V) + (s[k] - V), d);
  return V + d;
}

}  // namespace

// Distances of every node to its fiber's ends, clipped to 255, as dl | dr <<
// 8, from the fibers' first nodes (first[n_fibers] = n_total).
__global__ __launch_bounds__(256) void k_node_ends(const int32_t* __restrict__ first, int n_fibers,
                                                   int64_t nt, uint16_t* __restrict__ ends) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= nt) return;
  int lo = 0, hi = n_fibers - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (first[mid] <= i) lo = mid; else hi = mid - 1;
  }
  const int dl = (int)(i - first[lo]), dr = (int)(first[lo + 1] - 1 - i);
  ends[i] = (uint16_t)(min(dl, 255) | min(dr, 255) << 8);
}

// One diffusion substep of every node, from row `in` to row `out` (different
// rows): 1024 nodes per block through LDS, four consecutive ones per thread,
// whose 4 + 2 W neighbours it then holds in registers.  With adaptive
// computation (fiber_any) fibers without a solved node keep V, and every
// fiber's flag of the step after next is cleared by its first node.  Bound by
// HBM (8 B per node): 4e6 nodes in DIFF4 us, 2e7 in DIFF20; one node per
// thread, with its 2 W reads from LDS, took 21 us for 4e6, the partitioned
// solve in its place (six barriers per bin of one fiber) 15 us.
constexpr int kDiffNodes = 1024;

template <int W>
__global__ __launch_bounds__(256) void k_diffuse_window(KArgs A, WindowStencil st,
                                                        const float* __restrict__ in,
                                                        float* __restrict__ out) {
  constexpr int PAD = (W + 3) / 4 * 4, Q = PAD / 4;
  __shared__ float4 s_v4[kDiffNodes / 4 + 2 * Q];
  const int t = threadIdx.x;
  const int64_t nt = A.n_total, b0 = (int64_t)blockIdx.x * kDiffNodes, i = b0 + 4 * t;
  auto load4 = [&](int64_t j) {
    if (j >= 0 && j + 3 < nt) return *reinterpret_cast<const float4*>(in + j);
    float4 v = {0.0f, 0.0f, 0.0f, 0.0f};
    if (j >= 0 && j < nt) v.x = in[j];
    if (j + 1 >= 0 && j + 1 < nt) v.y = in[j + 1];
    if (j + 2 >= 0 && j + 2 < nt) v.z = in[j + 2];
    return v;
  };
  s_v4[Q + t] = load4(i);
  if (t < Q) s_v4[t] = load4(b0 - PAD + 4 * t);
  else if (t < 2 * Q) s_v4[kDiffNodes / 4 + t] = load4(b0 + kDiffNodes + 4 * (t - Q));
  int ends[4];
  bool live[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const bool real = i + q < nt;
    ends[q] = real ? A.node_ends[i + q] : 0xffff;
    live[q] = true;
    if (A.fiber_any && real) {
      const int32_t f = A.node_fiber[i + q];
      live[q] = A.fiber_any[f];
      if ((ends[q] & 255) == 0) A.fiber_any_next[f] = 0;
    }
  }
  __syncthreads();
  float v[4 + 2 * PAD];
#pragma unroll
  for (int q = 0; q < 1 + 2 * Q; ++q) {
    const float4 x = s_v4[t + q];
    v[4 * q] = x.x;
    v[4 * q + 1] = x.y;
    v[4 * q + 2] = x.z;
    v[4 * q + 3] = x.w;
  }
  bool near = false;
#pragma unroll
  for (int q = 0; q < 4; ++q) near |= (ends[q] & 255) < W || (ends[q] >> 8) < W;
  float o[4];
  if (!__any(near)) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float V = v[PAD + q];
      float d = 0.0f;
#pragma unroll
      for (int k = W; k >= 1; --k)
        d = fmaf(st.h[k - 1], (v[PAD + q - k] - V) + (v[PAD + q + k] - V), d);
      o[q] = V + d;
    }
  } else {
    const float* s = reinterpret_cast<const float*>(s_v4) + PAD + 4 * t;
#pragma unroll
    for (int q = 0; q < 4; ++q) o[q] = reflected<W>(s + q, s[q], ends[q] & 255, ends[q] >> 8, st);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) o[q] = live[q] ? o[q] : v[PAD + q];
  if (i + 3 < nt) {
    *reinterpret_cast<float4*>(out + i) = make_float4(o[0], o[1], o[2], o[3]);
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (i + q < nt) out[i + q] = o[q];
  }
}

// Split steps step0 .. step0 + wa.steps - 1 on windows, Hodgkin-Huxley: block
// b owns nodes b U .. b U + U - 1 and computes wa.halo more at either side
// (one node per thread), from state rows `in` to rows `out` (different
// buffers: neighbours read what this block owns).  Per step as in k_run_hh:
// V_m prescriptions, R(dt/2) D(dt) R(dt/2) (Godunov: R(dt) D(dt)), the
// observables; the states stay in registers throughout.
//
// Bound by vector issue like k_run_hh (0.35-0.45 us per step for each wave a
// SIMD holds) and by one step's own chain (0.5 us: four right-hand sides and
// one barrier, where the fused kernel has 3 + L), and by the launch (2.7 us)
// shared by wa.steps steps.  Where fibers are few or short this fills the chip
// as whole-fiber workgroups cannot: one fiber of 1000 nodes 2.5 -> 1.07 us per
// step, 200 fibers of 301-977 nodes 2.7 -> 1.9 us against the fused kernel and
// 10.5 -> 2.1 us against one reaction and one diffusion launch per step.
template <bool APX, int W>
__global__ __launch_bounds__(1024) void k_window_hh(KArgs A, WindowStencil st, WindowArgs wa,
                                                    int32_t step0) {
  extern __shared__ float s_v[];  // two buffers of blockDim.x + 2 kPad
  const int T = blockDim.x, t = threadIdx.x, row = T + 2 * kPad<W>;
  const int64_t nt = A.n_total;
  const int64_t i = (int64_t)blockIdx.x * wa.own + t - wa.halo;
  const bool real = i >= 0 && i < nt;
  const bool mine = real && t >= wa.halo && t < wa.halo + wa.own;
  const int64_t ic = real ? i : (i < 0 ? 0 : nt - 1);
  step0 += step_base_of(A);
  hh::State y{wa.in[ic], wa.in[nt + ic], wa.in[2 * nt + ic], wa.in[3 * nt + ic]};
  const int ends = real ? A.node_ends[ic] : 0xffff;
  const int dl = ends & 255, dr = ends >> 8;
  const uint32_t sid = real ? (uint32_t)A.node_stim[ic] : 0u;
  const StimDev e = sid ? A.stim[sid - 1] : StimDev{INT32_MAX, 0, 0, 0.0f, 0};
  bool watch = mine && isinf(A.t_act[ic]);  // not activated yet
  const hh::Ref ref{A.rest[0], A.rest[1], A.rest[2], A.rest[3]};
  const float uth = A.v_th - A.rest[0];
  // padding of both buffers
  for (int p = t; p < 2 * kPad<W>; p += T) {
    const int at = p < kPad<W> ? p : T + p;
    s_v[at] = s_v[row + at] = 0.0f;
  }
  // the next step that writes samples, and its row
  int64_t row_at = 0;
  int32_t sample_at = -1;
  if (A.sample_every > 0) {
    row_at = step0 / A.sample_every - A.sample_row0;
    const int64_t at = (step0 / A.sample_every + 1) * A.sample_every - 1;
    sample_at = at < step0 + wa.steps ? (int32_t)at : -1;
  }
  int par = 0;
  for (int32_t n = step0; n < step0 + wa.steps; ++n) {
    const float v0 = y.V;
    float I = 0.0f;
    if (sid && stim_on(e, n)) {
      if (e.voltage) y.V = e.amp;
      else I = e.amp;
    }
    for (int s = 0; s < A.n_sub; ++s) hh::heun<APX>(y, I, A.tau, A.inv_cm, ref);
    float* s = s_v + par + kPad<W> + t;
    *s = y.V;
    __syncthreads();
    y.V = window_diffuse<W>(s, y.V, dl, dr, st);
    par = row - par;
    for (int s = 0; s < A.n_sub2; ++s) hh::heun<APX>(y, I, A.tau, A.inv_cm, ref);
    if (watch && v0 < uth && y.V >= uth) {
      A.t_act[i] = fmaf(A.dt, (uth - v0) / (y.V - v0), (float)n * A.dt);
      watch = false;
    }
    if (n == sample_at) {
      if (mine) A.samples[row_at * nt + i] = y.V + A.rest[0];
      ++row_at;
      const int64_t at = (int64_t)n + A.sample_every;
      sample_at = at < step0 + wa.steps ? (int32_t)at : -1;
    }
  }
  if (mine) {
    wa.out[i] = y.V;
    wa.out[nt + i] = y.m;
    wa.out[2 * nt + i] = y.h;
    wa.out[3 * nt + i] = y.n;
    A.v_prev[i] = y.V;
    if (!isfinite(y.V) || !isfinite(y.m) || !isfinite(y.h) || !isfinite(y.n)) atomicOr(A.flag, 1);
  }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------

// Stencil widths the kernels are built for (a stencil takes the next one, its
// further weights zero).
#define FIB_FOR_EACH_WIDTH(X) X(8) X(10) X(12) X(16) X(24) X(32)

bool window_stencil(double w, double theta, WindowStencil& st) {
  st = WindowStencil{};
  if (!(w >= 0.0) || !std::isfinite(w)) return false;
  double lambda = 0.0;
  int need = 0;
  if (w > 0.0) {
    const double a = (1.0 + 2.0 * w) / w;
    lambda = 2.0 / (a + std::sqrt(a * a - 4.0));
    need = (int)std::ceil(40.0 / -std::log2(lambda));
  }
#define FIB_PICK(W) \
  if (st.width == 0 && need <= W) st.width = W;
  FIB_FOR_EACH_WIDTH(FIB_PICK)
#undef FIB_PICK
  if (st.width == 0) return false;
  const double g0 = 1.0 / std::sqrt(1.0 + 4.0 * w);
  double p = w * g0 * (1.0 - lambda) * (1.0 - lambda) / theta;
  for (int k = 0; k < need; ++k, p *= lambda) st.h[k] = (float)p;
  return true;
}

hipError_t launch_node_ends(const int32_t* first, int n_fibers, int64_t nt, uint16_t* ends,
                            hipStream_t s) {
  if (nt == 0) return hipSuccess;
  hipLaunchKernelGGL(k_node_ends, dim3((unsigned)((nt + 255) / 256)), dim3(256), 0, s, first,
                     n_fibers, nt, ends);
  return hipGetLastError();
}

hipError_t launch_diffuse_window(const WindowStencil& st, const float* in, float* out,
                                 const KArgs& a, hipStream_t s) {
  if (a.n_total == 0) return hipSuccess;
  const dim3 grid((unsigned)((a.n_total + kDiffNodes - 1) / kDiffNodes)), block(256);
#define FIB_LAUNCH(W) \
  if (st.width == W) hipLaunchKernelGGL(k_diffuse_window<W>, grid, block, 0, s, a, st, in, out);
  FIB_FOR_EACH_WIDTH(FIB_LAUNCH)
#undef FIB_LAUNCH
  return hipGetLastError();
}

hipError_t launch_window_hh(bool apx, const WindowStencil& st, const WindowArgs& wa,
                            const WindowPlan& p, int32_t step0, const KArgs& a, hipStream_t s) {
  if (a.n_total == 0) return hipSuccess;
  const dim3 grid((unsigned)((a.n_total + wa.own - 1) / wa.own)), block((unsigned)p.threads);
  const size_t lds = 2 * sizeof(float) * (size_t)(p.threads + 2 * st.width);
#define FIB_LAUNCH(W)                                                                       \
  if (st.width == W) {                                                                      \
    if (apx) hipLaunchKernelGGL((k_window_hh<true, W>), grid, block, lds, s, a, st, wa, step0); \
    else hipLaunchKernelGGL((k_window_hh<false, W>), grid, block, lds, s, a, st, wa, step0);    \
  }
  FIB_FOR_EACH_WIDTH(FIB_LAUNCH)
#undef FIB_LAUNCH
  return hipGetLastError();
}

}  // namespace fib
