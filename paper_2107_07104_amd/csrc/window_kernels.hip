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
#include "st57_model.h"

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
// HBM (8 B per node): 4e6 nodes in 14.5 us; one node per thread, with its
// 2 W reads from LDS, took 21 us, the partitioned solve in its place (six
// barriers per bin of one fiber) 15 us.
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
// Bound by vector issue like k_run_hh (0.35 us per step for each wave a SIMD
// holds; paced as that is, 0.42 without) and by one step's own chain (0.5 us:
// four right-hand sides and one barrier, where the fused kernel has 3 + L),
// and by the launch (2.7 us) shared by wa.steps steps.  Where fibers are few
// or short this fills the chip as whole-fiber workgroups cannot: one fiber of
// 1000 nodes 2.25 -> 1.06 us per step, 200 fibers of 301-977 nodes 2.3 -> 1.8
// us against the fused kernel and 10.5 -> 1.9 us against one reaction and one
// diffusion launch per step.
template <bool APX, int W, bool PACED>
__global__ __launch_bounds__(1024) void k_window_hh(KArgs A, WindowStencil st, WindowArgs wa,
                                                    int32_t step0) {
  FIB_PACED(PACED);
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
// Adaptive computation of the 57-state model, a fiber per workgroup
// ---------------------------------------------------------------------------

// LDS of k_run_st57_adapt for a fiber of n nodes (bytes): V_m twice with the
// stencil's padding, V_m at the end of the previous step, the list of solved
// nodes, the verdicts of two steps; then kStimCache stimulus entries, two
// list lengths and the range of the fiber's entries.
constexpr int kStimCache = 8;
__host__ __device__ inline int adapt_v_row(int n) { return n + 2 * kMaxWidth; }
__host__ __device__ inline size_t adapt_fiber_lds(int n) {
  const size_t rows = sizeof(float) * (2 * (size_t)adapt_v_row(n) + n) + 4 * (size_t)n;
  return (rows + 15) / 16 * 16 + kStimCache * sizeof(StimDev) + 4 * sizeof(int32_t);
}

// Split steps step0 .. step0 + n_steps - 1 of one fiber per workgroup with the
// adaptive computation's rules (k_adapt_decide / k_adapt_solve, which take a
// launch for each part): V_m, the verdicts and the list of solved nodes stay in
// LDS; the other states are read from and written to memory for solved nodes
// only.  Per step:
//   1. each node is solved if the last check found it or a neighbour active
//      or a stimulus entry that is on covers one of them; the solved nodes go
//      to a list (before the fiber's first stimulus none);
//   2. the first reaction part over the list (Godunov: the only part, with
//      the check);
//   3. the windowed diffusion of the whole fiber;
//   4. Strang: the second half and the check, on the states still in registers
//      where the list fits one round;
//   5. the observables.
// A step without a solved node skips 2 to 4.
//
// Bound by the reaction's chain (six right-hand sides per half, 6-7 us) on the
// few waves the solved nodes fill; the four launches it replaces took 65 us
// per step on 400 x 1481 nodes with 6 % firing (22 of them reading flags), this
// 30 (34 before it was paced).  Fibers are independent, so no other
// synchronization is needed; with more fibers than compute units workgroups
// of four waves run two to a unit, else of eight.
template <bool GODUNOV, int W>
__global__ __launch_bounds__(512, 2) void k_run_st57_adapt(KArgs A, WindowStencil st,
                                                           const int32_t* __restrict__ first) {
  FIB_PACED(true);
  constexpr int S = st57::S;
  extern __shared__ __align__(16) char smem[];
  const int f = blockIdx.x, t = threadIdx.x, T = blockDim.x, lane = t & 63;
  const int64_t off = first[f], nt = A.n_total;
  const int N = first[f + 1] - first[f];
  const int vrow = adapt_v_row(N);
  float* v_in = reinterpret_cast<float*>(smem) + kMaxWidth;  // node i at [i]
  float* v_new = v_in + vrow;
  float* v_prev = reinterpret_cast<float*>(smem) + 2 * vrow;
  uint16_t* list = reinterpret_cast<uint16_t*>(v_prev + N);
  uint8_t* act[2] = {reinterpret_cast<uint8_t*>(list + N),
                     reinterpret_cast<uint8_t*>(list + N) + N};
  char* tail = smem + adapt_fiber_lds(N) - kStimCache * sizeof(StimDev) - 4 * sizeof(int32_t);
  StimDev* cache = reinterpret_cast<StimDev*>(tail);
  int32_t* cnt = reinterpret_cast<int32_t*>(tail + kStimCache * sizeof(StimDev));
  int32_t* sid_lo = cnt + 2;  // smallest and largest entry + 1 of the fiber
  int32_t* sid_hi = cnt + 3;

  if (t == 0) {
    cnt[0] = cnt[1] = 0;
    *sid_lo = INT32_MAX;
    *sid_hi = 0;
  }
  for (int p = t; p < kMaxWidth; p += T) {
    v_in[-1 - p] = v_new[-1 - p] = 0.0f;
    v_in[N + p] = v_new[N + p] = 0.0f;
  }
  __syncthreads();
  // bit j of a mask: node t + j T
  uint32_t watch = 0, stim = 0;
  for (int j = 0, i = t; i < N; ++j, i += T) {
    const float v = A.state[off + i];
    v_in[i] = v;
    v_prev[i] = v;
    act[0][i] = (A.pt_prev[off + i] & PT_ACTIVE) ? 1 : 0;
    if (isinf(A.t_act[off + i])) watch |= 1u << j;
    // the node's own entry or a neighbour's
    const int32_t s0 = A.node_stim[off + i];
    const int32_t sl = i > 0 ? A.node_stim[off + i - 1] : 0;
    const int32_t sr = i + 1 < N ? A.node_stim[off + i + 1] : 0;
    if (s0 | sl | sr) stim |= 1u << j;
    if (s0) {
      atomicMin(sid_lo, s0);
      atomicMax(sid_hi, s0);
    }
  }
  __syncthreads();
  const int32_t lo = *sid_lo, n_ent = *sid_hi - lo + 1;
  const bool cached = *sid_hi > 0 && n_ent <= kStimCache;
  if (cached && t < n_ent) cache[t] = A.stim[lo - 1 + t];
  __syncthreads();
  auto entry = [&](int32_t sid) { return cached ? cache[sid - lo] : A.stim[sid - 1]; };
  auto on_at = [&](int i, int32_t n) {
    const int32_t sid = A.node_stim[off + i];
    return sid != 0 && stim_on(entry(sid), n);
  };
  const int32_t first_on = A.fiber_first_on[f];

  unsigned long long solved = 0;
  const int32_t n_end = A.step0 + A.n_steps;
  int par = 0;
  for (int32_t n = A.step0; n < n_end; ++n, par ^= 1) {
    // 1. nodes to solve; verdicts of the others
    const bool on = n >= first_on;
    if (on) {
      const uint8_t* a = act[par];
      for (int j = 0, i0 = t - lane; i0 < N; ++j, i0 += T) {
        const int i = i0 + lane;
        bool solve = false;
        if (i < N) {
          const int il = i > 0 ? i - 1 : i, ir = i + 1 < N ? i + 1 : i;
          solve = (a[i] | a[il] | a[ir]) != 0;
          if (!solve && ((stim >> j) & 1u)) solve = on_at(i, n) || on_at(il, n) || on_at(ir, n);
          if (!solve) act[par ^ 1][i] = 0;
        }
        const uint64_t mask = __ballot(solve);
        if (mask) {
          int base = 0;
          if (lane == 0) base = atomicAdd(&cnt[par], __popcll(mask));
          base = __builtin_amdgcn_readfirstlane(base);
          if (solve) list[base + __popcll(mask & ((1ull << lane) - 1ull))] = (uint16_t)i;
        }
      }
    } else {
      for (int i = t; i < N; i += T) act[par ^ 1][i] = act[par][i];
    }
    if (t == 0) cnt[par ^ 1] = 0;
    __syncthreads();
    const int c = cnt[par];
    if (c) {
      solved += t == 0 ? (unsigned)c : 0u;
      float u[S];
      float I = 0.0f;
      // whether the state moved over a reaction part from V offset vb and the
      // other states still in memory
      auto moved = [&](int64_t g, float vb) {
        gfloat* col = (gfloat*)(A.state + g);
        __asm__("" : "+v"(col));  // read again, not kept through the substeps
        bool m = fabsf(u[0] - vb) > A.adapt_tol * fabsf(vb + A.rest[0]);
#pragma unroll
        for (int k = 1; k < S; ++k) {
          const float b = col[k * nt];
          m |= fabsf(u[k] - b) > A.adapt_tol * fabsf(b + A.rest[k]);
        }
        return m;
      };
      // 2. first part
      for (int e = t; e < c; e += T) {
        const int i = list[e];
        const int64_t g = off + i;
#pragma unroll
        for (int k = 1; k < S; ++k) u[k] = A.state[k * nt + g];
        u[0] = v_in[i];
        I = 0.0f;
        const int32_t sid = A.node_stim[g];
        if (sid) {
          const StimDev en = entry(sid);
          if (stim_on(en, n)) {
            if (en.voltage) u[0] = en.amp;
            else I = en.amp;
          }
        }
        const float vb = u[0];
        for (int s = 0; s < A.n_sub; ++s) st57::heun(u, A.rest, I, A.tau, A.inv_cm);
        if (GODUNOV) act[par ^ 1][i] = moved(g, vb) ? 1 : 0;
        v_in[i] = u[0];
#pragma unroll
        for (int k = 1; k < S; ++k) A.state[k * nt + g] = u[k];
      }
      __syncthreads();
      // 3. diffusion
      for (int i0 = t - lane; i0 < N; i0 += T) {
        const int i = i0 + lane < N ? i0 + lane : N - 1;
        const float v = window_diffuse<W>(v_in + i, v_in[i], i, N - 1 - i, st);
        if (i0 + lane < N) v_new[i] = v;
      }
      __syncthreads();
      float* sw = v_in;
      v_in = v_new;
      v_new = sw;
      // 4. second half and the check
      if (!GODUNOV) {
        for (int e = t; e < c; e += T) {
          const int i = list[e];
          const int64_t g = off + i;
          if (c > T) {
#pragma unroll
            for (int k = 1; k < S; ++k) u[k] = A.state[k * nt + g];
            const int32_t sid = A.node_stim[g];
            I = 0.0f;
            if (sid) {
              const StimDev en = entry(sid);
              if (!en.voltage && stim_on(en, n)) I = en.amp;
            }
          }
          const float vb = v_in[i];
          u[0] = vb;
          for (int s = 0; s < A.n_sub; ++s) st57::heun(u, A.rest, I, A.tau, A.inv_cm);
          act[par ^ 1][i] = moved(g, vb) ? 1 : 0;
          v_in[i] = u[0];
#pragma unroll
          for (int k = 1; k < S; ++k) A.state[k * nt + g] = u[k];
        }
        __syncthreads();
      }
    }
    // 5. observables of this thread's nodes
    const bool sample = A.sample_every > 0 && ((int64_t)n + 1) % A.sample_every == 0;
    if (c || sample) {
      const float uth = A.v_th - A.rest[0];
      const int64_t r = sample ? ((int64_t)n + 1) / A.sample_every - 1 - A.sample_row0 : 0;
      for (int j = 0, i = t; i < N; ++j, i += T) {
        const float v0 = v_prev[i], v1 = v_in[i];
        if (((watch >> j) & 1u) && v0 < uth && v1 >= uth) {
          A.t_act[off + i] = fmaf(A.dt, (uth - v0) / (v1 - v0), (float)n * A.dt);
          watch &= ~(1u << j);
        }
        if (sample) A.samples[r * nt + off + i] = v1 + A.rest[0];
        v_prev[i] = v1;
      }
    }
  }
  __syncthreads();
  bool bad = false;
  for (int i = t; i < N; i += T) {
    const float v = v_in[i];
    A.state[off + i] = v;
    A.pt_cur[off + i] = act[par][i] ? PT_ACTIVE : 0;
    bad |= !isfinite(v);
  }
  if (bad) atomicOr(A.flag, 1);
  if (solved) atomicAdd(&A.adapt_count[f % kAdaptCounters], solved);
  // for a surrogate step that may follow (in the loop above it cost the steps'
  // loop registers: 29.1 -> 29.5 us per step on 400 x 1481 nodes)
  for (int i = t; i < N; i += T) A.v_prev[off + i] = v_in[i];
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

// Threads of a fiber's workgroup: with more fibers than compute units two
// workgroups of four waves share a unit.
static int adapt_fiber_threads(int n_fibers, int cus) { return n_fibers > cus ? 256 : 512; }

// Whether the longest fiber (n nodes) fits a workgroup (a thread's masks hold 32
// nodes), and is not behind the launches even with every node solved.  A
// workgroup then takes its list in rounds of a node per thread, 24 us a step
// each, 29 where every unit has one; the launches take 30 us a step and 0.52
// us per 1000 nodes of the chip (us per step, workgroup / launches, a tenth and
// all nodes solved: 1 x 101 19 19 / 28 28, 1 x 1000 20 48 / 30 33, 1 x 2000 23 93
// / 31 34, 64 x 2000 24 97 / 42 88, 256 x 1000 22 59 / 56 167, 400 x 1481 33 160
// / 69 354, 1500 x 2000 110 739 / 238 1637).  Few long fibers keep the launches:
// as a tenth of them is solved a workgroup would save a third of a step, and
// lose two steps where all are.
bool adapt_fiber_fits(int n, int n_fibers, int64_t nt, int cus, size_t lds) {
  if (n > 32 * 256 || adapt_fiber_lds(n) > lds) return false;
  const int threads = adapt_fiber_threads(n_fibers, cus), resident = cus * (512 / threads);
  const double rounds = (double)((n + threads - 1) / threads) *
                        (double)((n_fibers + resident - 1) / resident);
  const double busy = n_fibers < cus ? (double)n_fibers / cus : 1.0;
  return rounds * (24.0 + 5.0 * busy) <= 1.1 * (30.0 + 0.52e-3 * (double)nt);
}

hipError_t launch_run_st57_adapt(bool godunov, const WindowStencil& st, const int32_t* first,
                                 int n_fibers, int max_nodes, int cus, const KArgs& a,
                                 hipStream_t s) {
  if (a.n_total == 0) return hipSuccess;
  const dim3 grid((unsigned)n_fibers), block((unsigned)adapt_fiber_threads(n_fibers, cus));
  const size_t lds = adapt_fiber_lds(max_nodes);
#define FIB_LAUNCH(W)                                                                          \
  if (st.width == W) {                                                                         \
    if (godunov)                                                                               \
      hipLaunchKernelGGL((k_run_st57_adapt<true, W>), grid, block, lds, s, a, st, first);      \
    else                                                                                       \
      hipLaunchKernelGGL((k_run_st57_adapt<false, W>), grid, block, lds, s, a, st, first);     \
  }
  FIB_FOR_EACH_WIDTH(FIB_LAUNCH)
#undef FIB_LAUNCH
  return hipGetLastError();
}

hipError_t launch_window_hh(bool apx, const WindowStencil& st, const WindowArgs& wa,
                            const WindowPlan& p, int32_t step0, const KArgs& a, hipStream_t s) {
  if (a.n_total == 0) return hipSuccess;
  const dim3 grid((unsigned)((a.n_total + wa.own - 1) / wa.own)), block((unsigned)p.threads);
  const size_t lds = 2 * sizeof(float) * (size_t)(p.threads + 2 * st.width);
  const bool paced = two_waves(grid.x, p.threads);
#define FIB_LAUNCH_(APX, W, PACED) \
  hipLaunchKernelGGL((k_window_hh<APX, W, PACED>), grid, block, lds, s, a, st, wa, step0)
#define FIB_LAUNCH(W)                                       \
  if (st.width == W) {                                      \
    if (apx && paced) FIB_LAUNCH_(true, W, true);           \
    else if (apx) FIB_LAUNCH_(true, W, false);              \
    else if (paced) FIB_LAUNCH_(false, W, true);            \
    else FIB_LAUNCH_(false, W, false);                      \
  }
  FIB_FOR_EACH_WIDTH(FIB_LAUNCH)
#undef FIB_LAUNCH
#undef FIB_LAUNCH_
  return hipGetLastError();
}

}  // namespace fib
