// EMG step: the static bidomain solve on the structured 3D mesh (gfx950).
//
// The mesh nodes are every m-th node of an nx x ny bundle of equal fibers
// (thesis eq. discretized_fibers_2: V_3D = P V_m is an injection), and the
// elements are trilinear hexahedra with widths (hx, hy, m h).  For a
// diagonal conduction tensor D the Q1 stiffness matrix is
//   K_D = dx Kx (x) My (x) Mz + dy Mx (x) Ky (x) Mz + dz Mx (x) My (x) Kz
// with the 1D linear-element stiffness K and consistent mass M, so a row of
// K_D is a 27-point stencil whose weights are products of three 1D weights
// (each 1D factor knows whether its neighbour exists: that is the Neumann
// boundary).  The operator is applied matrix-free: no matrix is stored, the
// weights of a node are formed from its (i, j, k) in registers.
//
// A row is applied as sum_{j != t} w_tj (u_j - u_t): K_D u with the diagonal
// taken as minus the row's off-diagonal weights, which is exact for K_D
// (its rows sum to zero).  In any precision this keeps the constant vector an exact
// null vector of the operator, as it is of K_D, so the projected Neumann
// system stays consistent and semi-definite.  Applied with the centre weight
// rounded on its own, the operator's constant mode has an eigenvalue of the
// size of the rounding and of either sign (about -3e-8 of the diagonal on a
// 3 x 7 x 121 mesh), and CG diverges once it resolves that mode.
//
// The solve (eq. discretized_fibers_3) is preconditioned conjugate gradients
// on the Neumann system, preconditioned with the operator's own inverse by
// cosine transforms (below, k_fdm_*), or, for bundles too large for those,
// with the diagonal of K_{sigma_i + sigma_e} (k_cg_*).  The iterates are kept
// in the range of the operator: the stored residual r is the raw update, and
// its mean c is removed wherever it is used (diagonal: z = (r - c) / diag).  Rounding
// in r -= alpha q moves the residual's sum away from zero by a random walk
// that no CG step can reduce (the constant is the operator's null vector);
// left in, it dominates r.z once the residual is small and CG diverges.
// The projected scalars come from four sums of the raw r:
//   r.z = sum r^2/d - 2 c sum r/d + c^2 sum 1/d,  r.r = sum r^2 - n c^2.
// Each iteration k of the diagonal form is two launches:
//   k_cg_q:  the totals of the previous launch's per-block sums of r give
//            c, r.z, r.r and the convergence test; then p <- (r - c)/d +
//            beta p (the previous p in the other buffer; the stencil forms
//            its neighbours' p itself), q = A p, per-block sums of p.q;
//   k_cg_x:  alpha = r.z / p.q from the totals of those sums; x += alpha p,
//            r <- (r - c) - alpha q, per-block sums of r, r^2, r/d, r^2/d.
// Every block forms the totals itself, from FP64 per-block sums added in a
// fixed order, so all blocks agree bit for bit and every solve is
// deterministic; the kernel boundaries order the sums and scalars without
// device-wide fences.  Sums and scalars alternate between two buffers by
// the parity of k, so a launch never overwrites what its own blocks read.
// Once converged, launches return at once, so the host enqueues batches and
// checks the
// flag between them.  The grid is (blocks per layer, layers): a thread
// finds (i, j) from its index in the layer and k from the block row.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <vector>

#include "../../include/fib.h"
#include "fib_internal.h"

namespace {

constexpr int kB = 256;  // threads per block (four waves)

struct Grid3 {
  int nx, ny, nz;
  float hx, hy, hz;
  int64_t n;
  double h64[3];  // hx, hy, hz
};

// Scalars of the solve, in device memory.  slot[k & 1] holds iteration
// k's projected scalars, written by block 0 of its k_cg_q.
struct Slot {
  double c;   // mean of the stored (raw) residual
  double rz;  // r.z of the projected residual
};

struct Scal {
  double mean_b;  // mean of the raw right-hand side
  double bb;      // ||b||^2 after the projection
  double sd;      // sum of 1 / diag(A)
  double tol2;    // tol^2
  double rr;      // r.r of the last residual tested
  Slot slot[2];
  int32_t it;     // iterations taken
  int32_t done;   // converged (or b = 0)
};

// Projected c, r.z, r.r from the sums of the raw residual (S1 = sum r,
// S2 = sum r^2, S1d = sum r/d, S2d = sum r^2/d).
struct Proj {
  double c, rz, rr;
};

__device__ __forceinline__ Proj project(const double* t, int64_t n, double sd) {
  const double c = t[0] / (double)n;
  return {c, fmax(t[3] - 2.0 * c * t[2] + c * c * sd, 0.0), fmax(t[1] - (double)n * c * c, 0.0)};
}

__device__ __forceinline__ bool first_thread() {
  return blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0;
}

__device__ __forceinline__ float fma_of(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double fma_of(double a, double b, double c) { return fma(a, b, c); }

// 1D linear-element stiffness and mass weights of node i (of n, spacing h)
// towards its neighbours i - 1, i, i + 1; a missing neighbour weighs 0.
template <class R>
__device__ __forceinline__ void weights_1d(int i, int n, R h, R (&K)[3], R (&M)[3]) {
  const R lo = i > 0 ? R(1) : R(0), hi = i + 1 < n ? R(1) : R(0);
  const R ih = R(1) / h;
  K[0] = -lo * ih;
  K[1] = (lo + hi) * ih;
  K[2] = -hi * ih;
  M[0] = lo * h * R(1.0 / 6.0);
  M[1] = (lo + hi) * h * R(1.0 / 3.0);
  M[2] = hi * h * R(1.0 / 6.0);
}

template <class R>
__device__ __forceinline__ R spacing(const Grid3& g, int axis);
template <>
__device__ __forceinline__ float spacing<float>(const Grid3& g, int axis) {
  return axis == 0 ? g.hx : axis == 1 ? g.hy : g.hz;
}
template <>
__device__ __forceinline__ double spacing<double>(const Grid3& g, int axis) {
  return g.h64[axis];
}

// Row (i, j, k) of K_D applied to a field u in the difference form
// sum_{j != t} w_tj (u_j - u_t), by sum factorization over the axes:
//     dx sum_c Mz_c sum_b My_b sum_a Kx_a du
//   + dy sum_c Mz_c sum_b Ky_b sum_a Mx_a du
//   + dz sum_c Kz_c sum_b My_b sum_a Mx_a du,
// du = u(i + a - 1, j + b - 1, k + c - 1) - u(i, j, k) (the centre term is
// zero).  get(kk, l) returns u at layer kk and in-layer index l = j' nx + i'.
// A missing neighbour has 1D weight 0, and its offset is clamped to the node
// itself so that every read stays in the mesh.  diag receives the diagonal
// weight of K_D (the Jacobi preconditioner).  R: the arithmetic (float, or
// double on the same FP32 field).  Z: only the last term (dx = dy = 0).
template <class R, bool Z = false, class Get>
__device__ __forceinline__ R apply_row(const Grid3& g, R dx, R dy, R dz, int i, int j, int k,
                                       Get get, R& diag) {
  R Kx[3], Mx[3], Ky[3], My[3], Kz[3], Mz[3];
  weights_1d<R>(i, g.nx, spacing<R>(g, 0), Kx, Mx);
  weights_1d<R>(j, g.ny, spacing<R>(g, 1), Ky, My);
  weights_1d<R>(k, g.nz, spacing<R>(g, 2), Kz, Mz);
  diag = dx * Kx[1] * My[1] * Mz[1] + dy * Mx[1] * Ky[1] * Mz[1] + dz * Mx[1] * My[1] * Kz[1];
  const uint32_t l0 = (uint32_t)(j * g.nx + i);
  const uint32_t ox[3] = {i > 0 ? ~0u : 0u, 0u, i + 1 < g.nx ? 1u : 0u};
  const uint32_t oy[3] = {j > 0 ? 0u - (uint32_t)g.nx : 0u, 0u, j + 1 < g.ny ? (uint32_t)g.nx : 0u};
  const uint32_t kz[3] = {(uint32_t)(k > 0 ? k - 1 : k), (uint32_t)k,
                          (uint32_t)(k + 1 < g.nz ? k + 1 : k)};
  const R uc = (R)get((uint32_t)k, l0);
  R s1 = 0, s2 = 0, s3 = 0;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    R y1 = 0, y2 = 0, y3 = 0;
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      const uint32_t l = l0 + oy[b];
      const R d0 = (R)get(kz[c], l + ox[0]) - uc;
      const R d1 = (R)get(kz[c], l) - uc;
      const R d2 = (R)get(kz[c], l + ox[2]) - uc;
      const R sk = Z ? R(0) : fma_of(Kx[0], d0, fma_of(Kx[1], d1, Kx[2] * d2));
      const R sm = fma_of(Mx[0], d0, fma_of(Mx[1], d1, Mx[2] * d2));
      if (!Z) {
        y1 = fma_of(My[b], sk, y1);
        y2 = fma_of(Ky[b], sm, y2);
      }
      y3 = fma_of(My[b], sm, y3);
    }
    if (!Z) {
      s1 = fma_of(Mz[c], y1, s1);
      s2 = fma_of(Mz[c], y2, s2);
    }
    s3 = fma_of(Kz[c], y3, s3);
  }
  return Z ? dz * s3 : fma_of(dx, s1, fma_of(dy, s2, dz * s3));
}

// Node of this thread in the (blocks per layer, layers) grid; false past
// the end of its layer.
__device__ __forceinline__ bool node_of(const Grid3& g, int& i, int& j, int& k, uint32_t& t) {
  const int tl = (int)blockIdx.x * kB + (int)threadIdx.x;  // index in the layer
  if (tl >= g.nx * g.ny) return false;
  i = tl % g.nx;
  j = tl / g.nx;
  k = (int)blockIdx.y;
  t = (uint32_t)k * (uint32_t)(g.nx * g.ny) + (uint32_t)tl;
  return true;
}

// Element idx of a vector through a 32-bit byte offset (vectors hold at
// most 2^30 elements), so that the load takes the base address from scalar
// registers and only the offset from a vector register.
__device__ __forceinline__ float at(const float* __restrict__ v, uint32_t idx) {
  return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(v) + (idx << 2));
}

// Accessor of a mesh vector for apply_row.
struct MeshVec {
  const float* __restrict__ v;
  uint32_t nxy;
  __device__ __forceinline__ float operator()(uint32_t kk, uint32_t l) const {
    return at(v, kk * nxy + l);
  }
};

// Per-block sums of NV doubles into the block's record partials[block * NV
// + v], in a fixed order (waves by shuffles, then the four waves in order).
// Each (NV, TAG) has its own LDS array: a kernel that calls it twice gives
// each call its own.
template <int NV, int TAG = 0>
__device__ __forceinline__ void block_sums(double (&v)[NV], double* partials) {
  __shared__ double sh[NV][kB / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int blk = (int)(blockIdx.y * gridDim.x + blockIdx.x);
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    double x = v[q];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) x += __shfl_down(x, d);
    if (lane == 0) sh[q][wave] = x;
  }
  __syncthreads();
  if (threadIdx.x < NV) {
    double x = 0.0;
    for (int w = 0; w < kB / 64; ++w) x += sh[threadIdx.x][w];
    partials[(size_t)blk * NV + threadIdx.x] = x;
  }
}

// Totals of the per-block records, the same in every block that forms them:
// thread t adds records t, t + kB, t + 2 kB, ... in that order (loaded four
// at a time, so one memory latency covers up to 4 kB blocks), then the
// waves reduce by shuffles and the four wave sums are added in order (the
// first kB threads of a larger block).  Each (NV, TAG) has its own LDS array,
// as above.
template <int NV, int TAG = 0>
__device__ __forceinline__ void total_sums(const double* partials, int nblocks, double (&tot)[NV]) {
  __shared__ double sh[NV][kB / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double x[NV];
#pragma unroll
  for (int q = 0; q < NV; ++q) x[q] = 0.0;
  for (int b0 = wave < kB / 64 ? (int)threadIdx.x : nblocks; b0 < nblocks; b0 += 4 * kB) {
    double rec[4][NV];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int b = b0 + u * kB;
#pragma unroll
      for (int q = 0; q < NV; ++q) rec[u][q] = b < nblocks ? partials[(size_t)b * NV + q] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
#pragma unroll
      for (int q = 0; q < NV; ++q) x[q] += rec[u][q];
    }
  }
#pragma unroll
  for (int q = 0; q < NV; ++q) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) x[q] += __shfl_down(x[q], d);
    if (lane == 0 && wave < kB / 64) sh[q][wave] = x[q];
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    double y = 0.0;
    for (int w = 0; w < kB / 64; ++w) y += sh[q][w];
    tot[q] = y;
  }
}

// b = -K_{sigma_i} P V_m from the fiber state (row 0: V_m - rest; the
// difference form sees only differences of V_m), formed in FP64 and rounded
// once; per-block sums of b.
__global__ __launch_bounds__(kB) void k_emg_rhs(Grid3 g, const float* __restrict__ vm,
                                                int32_t n_fib, int32_t m, double sigma_i,
                                                float* __restrict__ b, double* partials) {
  int i, j, k;
  uint32_t t;
  double v[1] = {0.0};
  if (node_of(g, i, j, k, t)) {
    // 3D node (i', j', k') is fiber j' nx + i' at its node k' m
    auto get = [&](uint32_t kk, uint32_t f) {
      return at(vm, f * (uint32_t)n_fib + kk * (uint32_t)m);
    };
    double d;
    const float val = (float)-apply_row<double, true>(g, 0.0, 0.0, sigma_i, i, j, k, get, d);
    b[t] = val;
    v[0] = val;
  }
  block_sums<1>(v, partials);
}

__global__ __launch_bounds__(kB) void k_emg_mean(const double* partials, int nblocks, int64_t n,
                                                 Scal* s) {
  double tot[1];
  total_sums<1>(partials, nblocks, tot);
  if (threadIdx.x == 0) s->mean_b = tot[0] / (double)n;
}

// 1 / diag(A) of every node and per-block sums of it.
__global__ __launch_bounds__(kB) void k_emg_invd(Grid3 g, float dx, float dy, float dz,
                                                 float* __restrict__ invd, double* partials) {
  int i, j, k;
  uint32_t t;
  double v[1] = {0.0};
  if (node_of(g, i, j, k, t)) {
    float Kx[3], Mx[3], Ky[3], My[3], Kz[3], Mz[3];
    weights_1d<float>(i, g.nx, g.hx, Kx, Mx);
    weights_1d<float>(j, g.ny, g.hy, Ky, My);
    weights_1d<float>(k, g.nz, g.hz, Kz, Mz);
    const float d = dx * Kx[1] * My[1] * Mz[1] + dy * Mx[1] * Ky[1] * Mz[1] +
                    dz * Mx[1] * My[1] * Kz[1];
    const float w = 1.0f / d;
    invd[t] = w;
    v[0] = w;
  }
  block_sums<1>(v, partials);
}

__global__ __launch_bounds__(kB) void k_emg_sd(const double* partials, int nblocks, Scal* s) {
  double tot[1];
  total_sums<1>(partials, nblocks, tot);
  if (threadIdx.x == 0) s->sd = tot[0];
}

// Sums of the raw residual rt for project(): r, r^2, r/d, r^2/d.
__device__ __forceinline__ void residual_sums(float rt, float wd, double* v) {
  const double r = rt, rw = (double)rt * wd;
  v[0] = r;
  v[1] = r * r;
  v[2] = rw;
  v[3] = rw * r;
}

// Start of CG from the last solution x: bp = b - mean(b), r = bp - A x;
// per-block sums of r, r^2, r/d, r^2/d into part_r and of bp.bp into part_b.
__global__ __launch_bounds__(kB) void k_emg_start(Grid3 g, float dx, float dy, float dz,
                                                  const float* __restrict__ b,
                                                  const float* __restrict__ x,
                                                  const float* __restrict__ invd,
                                                  float* __restrict__ r, double* part_r,
                                                  double* part_b, const Scal* s) {
  int i, j, k;
  uint32_t t;
  double v[4] = {0.0, 0.0, 0.0, 0.0}, vb[1] = {0.0};
  if (node_of(g, i, j, k, t)) {
    float d;
    const float ax =
        apply_row<float>(g, dx, dy, dz, i, j, k, MeshVec{x, (uint32_t)(g.nx * g.ny)}, d);
    const float bp = b[t] - (float)s->mean_b;
    const float rt = bp - ax;
    r[t] = rt;
    residual_sums(rt, invd[t], v);
    vb[0] = (double)bp * bp;
  }
  block_sums<4>(v, part_r);
  block_sums<1>(vb, part_b);
}

__global__ __launch_bounds__(kB) void k_emg_started(const double* part_r, const double* part_b,
                                                    int nblocks, int64_t n, Scal* s) {
  double tot[4], tb[1];
  total_sums<4>(part_r, nblocks, tot);
  total_sums<1>(part_b, nblocks, tb);
  if (threadIdx.x == 0) {
    const Proj pr = project(tot, n, s->sd);
    s->bb = tb[0];
    s->rr = pr.rr;
    s->it = 0;
    s->slot[1].rz = INFINITY;  // beta = 0 in the first iteration
    s->done = (tb[0] == 0.0 || pr.rr <= s->tol2 * tb[0]) ? 1 : 0;
  }
}

// Iteration k (parity P): the test and beta from the sums of r in part_r,
// then p_new = (r - c)/d + beta p_old and q = A p_new; per-block sums of
// p.q into part_pq.
__global__ __launch_bounds__(kB) void k_cg_q(Grid3 g, float dx, float dy, float dz,
                                             const float* __restrict__ r,
                                             const float* __restrict__ invd,
                                             const float* __restrict__ p_old,
                                             float* __restrict__ p_new, float* __restrict__ q,
                                             const double* part_r, double* part_pq, int nblocks,
                                             int P, Scal* s) {
  if (s->done) return;
  double tot[4];
  total_sums<4>(part_r, nblocks, tot);
  const Proj pr = project(tot, g.n, s->sd);
  const bool done = pr.rr <= s->tol2 * s->bb;
  const double rz_prev = s->slot[P ^ 1].rz;
  if (first_thread()) {
    s->rr = pr.rr;
    s->slot[P].c = pr.c;
    s->slot[P].rz = pr.rz;
    if (done) s->done = 1;
    else s->it += 1;
  }
  if (done) return;
  const float beta = (rz_prev > 0.0 && rz_prev < INFINITY) ? (float)(pr.rz / rz_prev) : 0.0f;
  const float c = (float)pr.c;
  int i, j, k;
  uint32_t t;
  double v[1] = {0.0};
  if (node_of(g, i, j, k, t)) {
    const uint32_t nxy = (uint32_t)(g.nx * g.ny);
    auto pn = [&](uint32_t kk, uint32_t l) {
      const uint32_t n = kk * nxy + l;
      return fmaf(beta, at(p_old, n), (at(r, n) - c) * at(invd, n));
    };
    float d;
    const float qt = apply_row<float>(g, dx, dy, dz, i, j, k, pn, d);
    const float pt = fmaf(beta, p_old[t], (r[t] - c) * invd[t]);
    p_new[t] = pt;
    q[t] = qt;
    v[0] = (double)pt * qt;
  }
  block_sums<1>(v, part_pq);
}

// Iteration k (parity P): alpha from the sums of p.q, x += alpha p,
// r <- (r - c) - alpha q; per-block sums of r, r^2, r/d, r^2/d into
// part_r (the buffer of parity P ^ 1).
__global__ __launch_bounds__(kB) void k_cg_x(Grid3 g, const float* __restrict__ p,
                                             const float* __restrict__ q,
                                             const float* __restrict__ invd,
                                             float* __restrict__ x, float* __restrict__ r,
                                             const double* part_pq, double* part_r, int nblocks,
                                             int P, const Scal* s) {
  if (s->done) return;
  double tot[1];
  total_sums<1>(part_pq, nblocks, tot);
  const float alpha = tot[0] > 0.0 ? (float)(s->slot[P].rz / tot[0]) : 0.0f;
  const float c = (float)s->slot[P].c;
  int i, j, k;
  uint32_t t;
  double v[4] = {0.0, 0.0, 0.0, 0.0};
  if (node_of(g, i, j, k, t)) {
    x[t] = fmaf(alpha, p[t], x[t]);
    const float rt = fmaf(-alpha, q[t], r[t] - c);
    r[t] = rt;
    residual_sums(rt, invd[t], v);
  }
  block_sums<4>(v, part_r);
}

// ---------------------------------------------------------------------------
// Conjugate gradients preconditioned by the operator's own inverse
// ---------------------------------------------------------------------------
//
// On a uniform axis of n nodes with spacing h the linear-element stiffness K
// and mass M share the cosines V[i][k] = cos(pi i k / (n - 1)): with D =
// diag(1/2, 1, ..., 1, 1/2) and t = pi k / (n - 1),
//   K V = D V diag((2 - 2 cos t) / h),  M V = D V diag(h (2 + cos t) / 3),
//   V^T D V = diag((n - 1) (1 at k = 0 and n - 1, else 1/2)).
// So K_D is diagonal in the products of the three axes' cosines (the fast
// diagonalization of tensor-product operators, Lynch, Rice and Thomas 1964),
// and its inverse is a cosine transform along each axis, a division and the
// same transforms back (V is symmetric).  In exact arithmetic the first
// iteration solves the system; with z and p in FP32 the second takes the
// residual to 1e-11 where the diagonal preconditioner took 230 to 1e-7 on 37 x
// 37 x 149 nodes (14.4 us each, 3.5 ms a solve; now 0.25 ms).
//
// The residual r, q = A p and the rows' arithmetic are FP64 (of FP32 fields p,
// x and V_m): two iterations average no rounding away, and with r, q and the
// rows in FP32 what the operator's largest terms rounded off stood in the
// smooth modes of phi_e (relative error 8e-7 on 6 x 5 x 48 nodes, 8.2e-7 on
// 37 x 37 x 149; now 1.1e-7 and 5.6e-8).  It costs 8 us of 231 a solve there:
// the right-hand side 17.0 -> 20.1, k_fdm_xy 9.1 -> 11.2, k_pcg_q 6.9 -> 7.4 us.
// An iteration is five launches:
//   k_fdm_xy:   the residual test, then the x and y transforms of one layer;
//   k_fdm_z:    z transform, division, z transform back, 16 columns;
//   k_fdm_back: x and y back to z = A^+ r, per-block sums of r.z and z;
//   k_pcg_q:    beta, p <- z + beta p and q = A p, per-block sums of p.q;
//   k_pcg_x:    alpha, x += alpha p, r <- (r - c) - alpha q, per-block sums of
//               r, r^2 and x (for the final shift to zero mean).
// The transforms are matrix products on the matrix cores in FP32
// (v_mfma_f32_16x16x4_f32): 4 (nx + ny + nz) operations per node, 182 MFLOP on
// 37 x 37 x 149 nodes, so an iteration is bound by its launches and their
// load latencies (11.2, 14.5, 8.2, 7.4 and 6.1 us there under the tracer).

typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kFdmPlane = 128;   // the most fibers along x or y
constexpr int kFdmLayers = 2048; // the most layers (a z panel of 16 columns in LDS)

// One axis of the transform: V padded with zeros to np x np, np = n rounded
// up to 16, and per k the stiffness and mass eigenvalues times the norm.
struct Axis {
  int n, np;
  const float* V;
  const float2* km;
};

struct Fdm {
  Axis x, y, z;
  float dx, dy, dz;
};

// V (FP64 cosines rounded once) and the eigenvalue table of an axis.
__global__ __launch_bounds__(kB) void k_fdm_axis(int n, int np, double h, float* __restrict__ V,
                                                 float2* __restrict__ km) {
  const int e = (int)blockIdx.x * kB + (int)threadIdx.x;
  if (e >= np * np) return;
  const int i = e / np, k = e % np;
  const int period = 2 * (n - 1);
  V[e] = i < n && k < n ? (float)cospi((double)((int64_t)i * k % period) / (double)(n - 1)) : 0.0f;
  if (i == 0) {
    const double c = cospi((double)k / (double)(n - 1));
    const double norm = (n - 1) * (k == 0 || k == n - 1 ? 1.0 : 0.5);
    km[k] = k < n ? make_float2((float)((2.0 - 2.0 * c) / h * norm),
                                (float)(h * (2.0 + c) / 3.0 * norm))
                  : make_float2(0.0f, 1.0f);
  }
}

// acc += A B over K = 0 .. k_n - 1 (padding of the operands past the axis is
// zero): lane l supplies A[l % 16][l / 16 + 4 s] = a(row, k) and B[l / 16 + 4
// s][l % 16] = b(k, column), eight steps' operands in flight.
template <class FA, class FB>
__device__ __forceinline__ v4f mma_f32(FA a, FB b, int k_n, int lane) {
  const int m = lane & 15, k0 = lane >> 4;
  v4f acc = {0.0f, 0.0f, 0.0f, 0.0f};
  for (int s = 0; s < k_n; s += 32) {
    float av[8], bv[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int k = s + 4 * q + k0;
      const bool in = s + 4 * q < k_n;
      av[q] = in ? a(m, k) : 0.0f;
      bv[q] = in ? b(k, m) : 0.0f;
    }
#pragma unroll
    for (int q = 0; q < 8; ++q)
      if (s + 4 * q < k_n) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[q], bv[q], acc, 0, 0, 0);
  }
  return acc;
}

// The x and y transforms of one layer U (ny x nx): out = Vy U Vx, through an
// LDS plane T = U Vx of y.np rows of x.np + 1.  Every wave takes 16 x 16
// tiles.  put(j, i, v) receives the results inside the layer.
template <class U, class Put>
__device__ __forceinline__ void plane_transform(const Axis& X, const Axis& Y,
                                                const U* __restrict__ in, float* T, Put put) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
  const int xt = X.np >> 4, yt = Y.np >> 4, ts = X.np + 1;
  const int r = lane & 15, g = lane >> 4;
  for (int t = wave; t < xt * yt; t += waves) {
    const int jb = 16 * (t / xt), ib = 16 * (t % xt);
    const v4f v = mma_f32(
        [&](int m, int k) {
          return jb + m < Y.n && k < X.n ? (float)in[(jb + m) * X.n + k] : 0.0f;
        },
        [&](int k, int c) { return k < X.np ? X.V[k * X.np + ib + c] : 0.0f; }, X.n, lane);
#pragma unroll
    for (int j = 0; j < 4; ++j) T[(jb + 4 * g + j) * ts + ib + r] = v[j];
  }
  __syncthreads();
  for (int t = wave; t < xt * yt; t += waves) {
    const int jb = 16 * (t / xt), ib = 16 * (t % xt);
    const v4f v = mma_f32([&](int m, int k) { return k < Y.np ? Y.V[k * Y.np + jb + m] : 0.0f; },
                          [&](int k, int c) { return k < Y.np ? T[k * ts + ib + c] : 0.0f; }, Y.n,
                          lane);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int jj = jb + 4 * g + j, ii = ib + r;
      if (jj < Y.n && ii < X.n) put(jj, ii, v[j]);
    }
  }
}

// Iteration k (parity P): the test from the sums of r in part_r, then u = the
// x and y transforms of r, one layer per block (its constant mode, which c
// belongs to, is dropped by k_fdm_z).
__global__ __launch_bounds__(1024) void k_fdm_xy(Fdm f, const double* __restrict__ r,
                                                 float* __restrict__ u, const double* part_r,
                                                 int nblocks, int64_t n, int P, Scal* s) {
  extern __shared__ float plane[];
  if (s->done) return;
  double tot[2];
  total_sums<2>(part_r, nblocks, tot);
  const double c = tot[0] / (double)n, rr = fmax(tot[1] - (double)n * c * c, 0.0);
  const bool done = rr <= s->tol2 * s->bb;
  if (first_thread()) {
    s->rr = rr;
    s->slot[P].c = c;
    if (done) s->done = 1;
  }
  if (done) return;
  const int64_t base = (int64_t)blockIdx.x * f.x.n * f.y.n;
  plane_transform(f.x, f.y, r + base, plane,
                  [&](int j, int i, float v) { u[base + j * f.x.n + i] = v; });
}

// u <- Vz (Vz u / (eigenvalue norm)) on 16 columns (modes of a layer, `cols`
// of them) per block; the constant mode becomes 0.  The panel of 16 columns
// lies in LDS, beside the divided one where both fit (`two`), else the
// latter passes through u.
__global__ __launch_bounds__(1024) void k_fdm_z(Fdm f, float* __restrict__ u, int cols, int two,
                                                const Scal* s) {
  extern __shared__ float panel[];  // z.np x 17, once or twice
  if (s->done) return;
  const Axis& Z = f.z;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
  const int r = lane & 15, g = lane >> 4, c0 = (int)blockIdx.x * 16;
  const bool real = c0 + r < cols;
  auto load = [&]() {
    for (int e = threadIdx.x; e < Z.np * 16; e += blockDim.x) {
      const int k = e >> 4, c = e & 15;
      panel[k * 17 + c] = k < Z.n && c0 + c < cols ? u[(int64_t)k * cols + c0 + c] : 0.0f;
    }
    __syncthreads();
  };
  auto product = [&](const float* in, int t) {
    return mma_f32([&](int m, int k) { return Z.V[k * Z.np + 16 * t + m]; },
                   [&](int k, int c) { return in[k * 17 + c]; }, Z.n, lane);
  };
  load();
  // eigenvalues of this lane's column
  const int col = real ? c0 + r : 0;
  const float2 ex = f.x.km[col % f.x.n], ey = f.y.km[col / f.x.n];
  const float la = f.dx * ex.x * ey.y + f.dy * ex.y * ey.x, lb = f.dz * ex.y * ey.y;
  for (int t = wave; t < (Z.np >> 4); t += waves) {
    const v4f v = product(panel, t);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int k = 16 * t + 4 * g + j;
      const float2 ez = Z.km[k];
      const float lam = fmaf(la, ez.y, lb * ez.x);
      const bool zero = !real || k >= Z.n || (k == 0 && c0 + r == 0);
      const float w = zero ? 0.0f : v[j] / lam;
      if (two)
        panel[(Z.np + k) * 17 + r] = w;
      else if (real && k < Z.n)
        u[(int64_t)k * cols + c0 + r] = w;
    }
  }
  __syncthreads();
  if (!two) load();
  const float* mid = two ? panel + Z.np * 17 : panel;
  for (int t = wave; t < (Z.np >> 4); t += waves) {
    const v4f v = product(mid, t);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int k = 16 * t + 4 * g + j;
      if (k < Z.n && real) u[(int64_t)k * cols + c0 + r] = v[j];
    }
  }
}

// z = the x and y transforms of u back, one layer per block; per-block sums
// of r z and z into part_z.
__global__ __launch_bounds__(1024) void k_fdm_back(Fdm f, const float* __restrict__ u,
                                                   const double* __restrict__ r,
                                                   float* __restrict__ z, double* part_z,
                                                   const Scal* s) {
  extern __shared__ float plane[];
  __shared__ double sh[2][16];
  if (s->done) return;
  const int64_t base = (int64_t)blockIdx.x * f.x.n * f.y.n;
  double v[2] = {0.0, 0.0};
  plane_transform(f.x, f.y, u + base, plane, [&](int j, int i, float zv) {
    const int64_t t = base + j * f.x.n + i;
    z[t] = zv;
    v[0] += r[t] * zv;
    v[1] += (double)zv;
  });
#pragma unroll
  for (int q = 0; q < 2; ++q) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v[q] += __shfl_down(v[q], d);
    if ((threadIdx.x & 63) == 0) sh[q][threadIdx.x >> 6] = v[q];
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    double x = 0.0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) x += sh[threadIdx.x][w];
    part_z[2 * blockIdx.x + threadIdx.x] = x;
  }
}

// Iteration k (parity P): beta from the sums of r z and z, p_new = z + beta
// p_old and q = A p_new; per-block sums of p.q into part_pq.
__global__ __launch_bounds__(kB) void k_pcg_q(Grid3 g, double dx, double dy, double dz,
                                              const float* __restrict__ z,
                                              const float* __restrict__ p_old,
                                              float* __restrict__ p_new, double* __restrict__ q,
                                              const double* part_z, double* part_pq, int P,
                                              Scal* s) {
  if (s->done) return;
  double tot[2];
  total_sums<2>(part_z, g.nz, tot);
  const double rz = fmax(tot[0] - s->slot[P].c * tot[1], 0.0);  // (r - c).z
  const double rz_prev = s->slot[P ^ 1].rz;
  if (first_thread()) {
    s->slot[P].rz = rz;
    s->it += 1;
  }
  const float beta = (rz_prev > 0.0 && rz_prev < INFINITY) ? (float)(rz / rz_prev) : 0.0f;
  int i, j, k;
  uint32_t t;
  double v[1] = {0.0};
  if (node_of(g, i, j, k, t)) {
    const uint32_t nxy = (uint32_t)(g.nx * g.ny);
    auto pn = [&](uint32_t kk, uint32_t l) {
      const uint32_t n = kk * nxy + l;
      return fmaf(beta, at(p_old, n), at(z, n));
    };
    double d;
    const double qt = apply_row<double>(g, dx, dy, dz, i, j, k, pn, d);
    const float pt = fmaf(beta, p_old[t], z[t]);
    p_new[t] = pt;
    q[t] = qt;
    v[0] = pt * qt;
  }
  block_sums<1>(v, part_pq);
}

// Iteration k (parity P): alpha from the sums of p.q, x += alpha p, r <- (r -
// c) - alpha q; per-block sums of r and r^2 into part_r (the buffer of parity
// P ^ 1) and of x into part_x.
__global__ __launch_bounds__(kB) void k_pcg_x(Grid3 g, const float* __restrict__ p,
                                              const double* __restrict__ q, float* __restrict__ x,
                                              double* __restrict__ r, const double* part_pq,
                                              double* part_r, double* part_x, int nblocks, int P,
                                              const Scal* s) {
  if (s->done) return;
  double tot[1];
  total_sums<1>(part_pq, nblocks, tot);
  const float alpha = tot[0] > 0.0 ? (float)(s->slot[P].rz / tot[0]) : 0.0f;
  const double c = s->slot[P].c;
  int i, j, k;
  uint32_t t;
  double v[2] = {0.0, 0.0}, vx[1] = {0.0};
  if (node_of(g, i, j, k, t)) {
    const float xt = fmaf(alpha, p[t], x[t]);
    x[t] = xt;
    const double rt = fma(-(double)alpha, q[t], r[t] - c);
    r[t] = rt;
    v[0] = rt;
    v[1] = rt * rt;
    vx[0] = (double)xt;
  }
  block_sums<2>(v, part_r);
  block_sums<1>(vx, part_x);
}

// Start from the last solution x: bp = b - mean(b), r = bp - A x; per-block
// sums of r and r^2 into part_r, of bp.bp and of x.
__global__ __launch_bounds__(kB) void k_pcg_start(Grid3 g, double dx, double dy, double dz,
                                                  const float* __restrict__ b,
                                                  const float* __restrict__ x,
                                                  double* __restrict__ r, double* part_r,
                                                  double* part_b, double* part_x, const Scal* s) {
  int i, j, k;
  uint32_t t;
  double v[2] = {0.0, 0.0}, vb[1] = {0.0}, vx[1] = {0.0};
  if (node_of(g, i, j, k, t)) {
    double d;
    const double ax =
        apply_row<double>(g, dx, dy, dz, i, j, k, MeshVec{x, (uint32_t)(g.nx * g.ny)}, d);
    const double bp = (double)b[t] - s->mean_b;
    const double rt = bp - ax;
    r[t] = rt;
    v[0] = rt;
    v[1] = rt * rt;
    vb[0] = bp * bp;
    vx[0] = (double)x[t];
  }
  block_sums<2>(v, part_r);
  block_sums<1, 0>(vb, part_b);
  block_sums<1, 1>(vx, part_x);
}

__global__ __launch_bounds__(kB) void k_pcg_started(const double* part_r, const double* part_b,
                                                    int nblocks, int64_t n, double tol2, Scal* s) {
  double tot[2], tb[1];
  total_sums<2>(part_r, nblocks, tot);
  total_sums<1>(part_b, nblocks, tb);
  if (threadIdx.x == 0) {
    const double c = tot[0] / (double)n, rr = fmax(tot[1] - (double)n * c * c, 0.0);
    s->tol2 = tol2;
    s->bb = tb[0];
    s->rr = rr;
    s->it = 0;
    s->slot[1].rz = INFINITY;  // beta = 0 in the first iteration
    s->done = (tb[0] == 0.0 || rr <= tol2 * tb[0]) ? 1 : 0;
  }
}

// r.r of the last iterate, where the launches enqueued so far did not
// converge.
__global__ __launch_bounds__(kB) void k_pcg_final(const double* part_r, int nblocks, int64_t n,
                                                  Scal* s) {
  if (s->done) return;
  double tot[2];
  total_sums<2>(part_r, nblocks, tot);
  if (threadIdx.x == 0) {
    const double c = tot[0] / (double)n, rr = fmax(tot[1] - (double)n * c * c, 0.0);
    s->rr = rr;
    if (rr <= s->tol2 * s->bb) s->done = 1;
  }
}

// Once converged (or `last`): x -= mean(x); x = 0 where b = 0.
__global__ __launch_bounds__(kB) void k_pcg_shift(Grid3 g, float* __restrict__ x,
                                                  const double* part_x, int nblocks, int last,
                                                  const Scal* s) {
  if (!s->done && !last) return;
  double tot[1];
  total_sums<1>(part_x, nblocks, tot);
  const float mean = (float)(tot[0] / (double)g.n);
  int i, j, k;
  uint32_t t;
  if (node_of(g, i, j, k, t)) x[t] = s->bb == 0.0 ? 0.0f : x[t] - mean;
}

// r.r of the last iterate when the iteration limit stopped the solve.
__global__ __launch_bounds__(kB) void k_cg_final(const double* part_r, int nblocks, int64_t n,
                                                 Scal* s) {
  if (s->done) return;
  double tot[4];
  total_sums<4>(part_r, nblocks, tot);
  if (threadIdx.x == 0) s->rr = project(tot, n, s->sd).rr;
}

// x -= mean(x): the per-block sums, the mean, the subtraction.
__global__ __launch_bounds__(kB) void k_emg_sum(Grid3 g, const float* __restrict__ x,
                                                double* partials) {
  int i, j, k;
  uint32_t t;
  double v[1] = {node_of(g, i, j, k, t) ? (double)x[t] : 0.0};
  block_sums<1>(v, partials);
}

__global__ __launch_bounds__(kB) void k_emg_shift(Grid3 g, float* __restrict__ x, const Scal* s) {
  int i, j, k;
  uint32_t t;
  if (node_of(g, i, j, k, t)) x[t] -= (float)s->mean_b;
}

int efail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  return fib::set_error(code, buf);
}

#define EHIP(expr)                                                                    \
  do {                                                                                \
    hipError_t e_ = (expr);                                                           \
    if (e_ != hipSuccess) return efail(FIB_EHIP, "%s: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

}  // namespace

struct fib_emg {
  fib_t* ctx = nullptr;
  fib_emg_params p{};
  Grid3 g{};
  int32_t n_fib = 0;          // nodes per fiber
  float* d_vec = nullptr;     // b, x, r, 1/diag, p0, p1, q (n each)
  double* d_part = nullptr;   // per-block sums, 9 x blocks
  Scal* d_s = nullptr;
  Scal* h_s = nullptr;        // pinned copy of the scalars
  dim3 grid;                  // (blocks per layer, layers)
  int nblocks = 0;
  float* b() const { return d_vec; }
  float* x() const { return d_vec + g.n; }
  float* r() const { return d_vec + 2 * g.n; }
  float* invd() const { return d_vec + 3 * g.n; }
  float* pb(int i) const { return d_vec + (4 + i) * g.n; }
  float* q() const { return d_vec + 6 * g.n; }
  double* part_r(int par) const { return d_part + (size_t)par * 4 * nblocks; }
  double* part_pq() const { return d_part + (size_t)8 * nblocks; }
  // the preconditioned solve: transforms of the axes in one array, its vectors
  // (b, x, u, z, p0, p1, then r and q in FP64), and its sums (r in two buffers,
  // p.q, x, b.b, then r.z and z by layer)
  bool fdm = false;
  Fdm f{};
  float* d_axes = nullptr;
  float* u() const { return d_vec + 2 * g.n; }
  float* z() const { return d_vec + 3 * g.n; }
  double* r64() const { return reinterpret_cast<double*>(d_vec + 6 * g.n); }
  double* q64() const { return reinterpret_cast<double*>(d_vec + 8 * g.n); }
  double* pcg_r(int par) const { return d_part + (size_t)par * 2 * nblocks; }
  double* pcg_pq() const { return d_part + (size_t)4 * nblocks; }
  double* pcg_x() const { return d_part + (size_t)5 * nblocks; }
  double* pcg_b() const { return d_part + (size_t)6 * nblocks; }
  double* pcg_z() const { return d_part + (size_t)7 * nblocks; }
};

namespace {

// Sets up the axes of the preconditioned solve.
int fdm_setup(fib_emg* e, hipStream_t st) {
  Axis* ax[3] = {&e->f.x, &e->f.y, &e->f.z};
  const int n[3] = {e->g.nx, e->g.ny, e->g.nz};
  const double h[3] = {e->p.hx, e->p.hy, (double)e->g.hz};
  size_t total = 0;
  for (int a = 0; a < 3; ++a) {
    const size_t np = (size_t)(n[a] + 15) / 16 * 16;
    total += np * np + 2 * np;
  }
  if (hipMalloc(&e->d_axes, sizeof(float) * total) != hipSuccess)
    return efail(FIB_ENOMEM, "device allocation failed");
  float* at = e->d_axes;
  for (int a = 0; a < 3; ++a) {
    const int np = (n[a] + 15) / 16 * 16;
    float2* km = reinterpret_cast<float2*>(at + (size_t)np * np);
    *ax[a] = Axis{n[a], np, at, km};
    hipLaunchKernelGGL(k_fdm_axis, dim3((unsigned)(((size_t)np * np + kB - 1) / kB)), dim3(kB), 0,
                       st, n[a], np, h[a], at, km);
    at += (size_t)np * np + 2 * np;
  }
  e->f.dx = e->f.dy = (float)e->p.sigma_et;
  e->f.dz = (float)(e->p.sigma_el + e->p.sigma_i);
  EHIP(hipGetLastError());
  return FIB_OK;
}

// fib_emg_solve with the preconditioner k_fdm_*.
int fdm_solve(fib_emg* e, const fib::CtxView& v, double tol, int32_t max_iter) {
  hipStream_t st = v.stream;
  const Grid3 g = e->g;
  const Fdm f = e->f;
  const dim3 grid = e->grid, block(kB), one(1);
  const int nb = e->nblocks, cols = g.nx * g.ny;
  const double dx = e->p.sigma_et, dy = e->p.sigma_et, dz = e->p.sigma_el + e->p.sigma_i;
  // a wave per 16 x 16 tile of a layer (at least the block total_sums wants)
  // and per 16 layers of a panel
  const int tiles = (f.x.np >> 4) * (f.y.np >> 4);
  const dim3 bxy((unsigned)std::min(1024, std::max(kB, 64 * tiles)));
  const dim3 bz((unsigned)std::min(1024, 64 * (f.z.np >> 4)));
  const size_t lds_xy = sizeof(float) * f.y.np * (f.x.np + 1);
  const size_t panel = sizeof(float) * f.z.np * 17;
  const int two = 2 * panel <= 128 * 1024;
  hipLaunchKernelGGL(k_emg_rhs, grid, block, 0, st, g, v.d_state, e->n_fib, e->p.stride,
                     e->p.sigma_i, e->b(), e->d_part);
  hipLaunchKernelGGL(k_emg_mean, one, block, 0, st, e->d_part, nb, g.n, e->d_s);
  hipLaunchKernelGGL(k_pcg_start, grid, block, 0, st, g, dx, dy, dz, e->b(), e->x(), e->r64(),
                     e->pcg_r(0), e->pcg_b(), e->pcg_x(), e->d_s);
  hipLaunchKernelGGL(k_pcg_started, one, block, 0, st, e->pcg_r(0), e->pcg_b(), nb, g.n,
                     tol * tol, e->d_s);
  // Two iterations reach 1e-8 and more on the meshes measured (2 x 2 x 3 to 37
  // x 37 x 149, 3 x 2 x 1481), so that many are enqueued before the host
  // looks, then one at a time, and half as many as were taken once it is clear
  // that more are needed (a look costs about an iteration: 2000 one by one
  // took 110 ms); launches past convergence return at once.
  int32_t launched = 0;
  for (;;) {
    const int batch = launched == 0 ? 2 : std::min(std::max(launched / 2 - 1, 1), 32);
    const int n_it = std::min(batch, max_iter - launched);
    for (int b = 0; b < n_it; ++b) {
      const int P = (launched + b) & 1;
      hipLaunchKernelGGL(k_fdm_xy, dim3((unsigned)g.nz), bxy, lds_xy, st, f, e->r64(), e->u(),
                         e->pcg_r(P), nb, g.n, P, e->d_s);
      hipLaunchKernelGGL(k_fdm_z, dim3((unsigned)((cols + 15) / 16)), bz,
                         two ? 2 * panel : panel, st, f, e->u(), cols, two, e->d_s);
      hipLaunchKernelGGL(k_fdm_back, dim3((unsigned)g.nz), bxy, lds_xy, st, f, e->u(), e->r64(),
                         e->z(), e->pcg_z(), e->d_s);
      hipLaunchKernelGGL(k_pcg_q, grid, block, 0, st, g, dx, dy, dz, e->z(), e->pb(P),
                         e->pb(P ^ 1), e->q64(), e->pcg_z(), e->pcg_pq(), P, e->d_s);
      hipLaunchKernelGGL(k_pcg_x, grid, block, 0, st, g, e->pb(P ^ 1), e->q64(), e->x(), e->r64(),
                         e->pcg_pq(), e->pcg_r(P ^ 1), e->pcg_x(), nb, P, e->d_s);
    }
    launched += n_it;
    const int last = launched >= max_iter ? 1 : 0;
    hipLaunchKernelGGL(k_pcg_final, one, block, 0, st, e->pcg_r(launched & 1), nb, g.n, e->d_s);
    hipLaunchKernelGGL(k_pcg_shift, grid, block, 0, st, g, e->x(), e->pcg_x(), nb, last, e->d_s);
    EHIP(hipGetLastError());
    EHIP(hipMemcpyAsync(e->h_s, e->d_s, sizeof(Scal), hipMemcpyDeviceToHost, st));
    EHIP(hipStreamSynchronize(st));
    if (e->h_s->done || last) return FIB_OK;
    if (std::isnan(e->h_s->bb)) {
      // V_m is not finite: phi_e is NaN, and every further iteration leaves it
      // so
      e->h_s->it = max_iter;
      return FIB_OK;
    }
  }
}

}  // namespace

extern "C" {

int fib_emg_create(fib_t* ctx, const fib_emg_params* p, fib_emg_t** out) {
  if (!out) return efail(FIB_EINVAL, "null output pointer");
  *out = nullptr;
  if (!ctx || !p) return efail(FIB_EINVAL, "null argument");
  const fib::CtxView v = fib::ctx_view(ctx);
  if (p->nx < 2 || p->ny < 2 || p->stride < 1)
    return efail(FIB_EINVAL, "nx, ny must be >= 2 and the stride >= 1");
  auto pos = [](double x) { return std::isfinite(x) && x > 0.0; };
  if (!pos(p->hx) || !pos(p->hy) || !pos(p->sigma_i) || !pos(p->sigma_el) || !pos(p->sigma_et))
    return efail(FIB_EINVAL, "spacings and conductivities must be > 0");
  if ((int64_t)p->nx * p->ny != v.n_fibers)
    return efail(FIB_EINVAL, "%d x %d fibers expected, the context has %d", p->nx, p->ny,
                 v.n_fibers);
  const int32_t n = v.n_nodes[0];
  for (int32_t f = 1; f < v.n_fibers; ++f)
    if (v.n_nodes[f] != n) return efail(FIB_EINVAL, "fibers of unequal length");
  if (n < 2 || (n - 1) % p->stride != 0)
    return efail(FIB_EINVAL, "fiber length %d: (n - 1) must be a positive multiple of %d", n,
                 p->stride);
  // the kernels address the fiber state and the mesh vectors with 32-bit
  // byte offsets
  if ((int64_t)v.n_fibers * n > (int64_t(1) << 30))
    return efail(FIB_EUNSUPPORTED, "EMG bundles hold at most 2^30 fiber nodes");
  fib_emg* e = new (std::nothrow) fib_emg();
  if (!e) return efail(FIB_ENOMEM, "host allocation failed");
  e->ctx = ctx;
  e->p = *p;
  e->n_fib = n;
  e->g.nx = p->nx;
  e->g.ny = p->ny;
  e->g.nz = (n - 1) / p->stride + 1;
  e->g.hx = (float)p->hx;
  e->g.hy = (float)p->hy;
  e->g.hz = (float)(p->stride * v.h);
  e->g.h64[0] = p->hx;
  e->g.h64[1] = p->hy;
  e->g.h64[2] = p->stride * v.h;
  e->g.n = (int64_t)e->g.nx * e->g.ny * e->g.nz;
  e->grid = dim3((unsigned)((e->g.nx * e->g.ny + kB - 1) / kB), (unsigned)e->g.nz);
  e->nblocks = (int)(e->grid.x * e->grid.y);
  // The transforms hold a layer, and a panel of every layer, in LDS; bundles
  // beyond that take the diagonal preconditioner (230 iterations instead of
  // two at 37 x 37 x 149 nodes, and growing with the layers).
  e->fdm = p->nx <= kFdmPlane && p->ny <= kFdmPlane && e->g.nz <= kFdmLayers;
  const size_t nv = (size_t)e->g.n * (e->fdm ? 10 : 7);
  if (hipMalloc(&e->d_vec, sizeof(float) * nv) != hipSuccess ||
      hipMalloc(&e->d_part, sizeof(double) * 9 * e->nblocks) != hipSuccess ||
      hipMalloc(&e->d_s, sizeof(Scal)) != hipSuccess ||
      hipHostMalloc(&e->h_s, sizeof(Scal)) != hipSuccess) {
    fib_emg_destroy(e);
    return efail(FIB_ENOMEM, "device allocation failed");
  }
  // zeros (x = 0 is the first solve's start), then 1/diag(A) and its sum,
  // all on the context's stream
  hipStream_t st = v.stream;
  bool ok = hipMemsetAsync(e->d_vec, 0, sizeof(float) * nv, st) == hipSuccess &&
            hipMemsetAsync(e->d_s, 0, sizeof(Scal), st) == hipSuccess;
  if (ok && e->fdm) {
    if (int rc = fdm_setup(e, st)) {
      fib_emg_destroy(e);
      return rc;
    }
    ok = hipStreamSynchronize(st) == hipSuccess;
  } else if (ok) {
    hipLaunchKernelGGL(k_emg_invd, e->grid, dim3(kB), 0, st, e->g, (float)p->sigma_et,
                       (float)p->sigma_et, (float)(p->sigma_el + p->sigma_i), e->invd(),
                       e->d_part);
    hipLaunchKernelGGL(k_emg_sd, dim3(1), dim3(kB), 0, st, e->d_part, e->nblocks, e->d_s);
    ok = hipGetLastError() == hipSuccess && hipStreamSynchronize(st) == hipSuccess;
  }
  if (!ok) {
    fib_emg_destroy(e);
    return efail(FIB_EHIP, "device initialisation failed");
  }
  *out = e;
  return FIB_OK;
}

void fib_emg_destroy(fib_emg_t* e) {
  if (!e) return;
  (void)hipFree(e->d_vec);
  (void)hipFree(e->d_part);
  (void)hipFree(e->d_axes);
  (void)hipFree(e->d_s);
  if (e->h_s) (void)hipHostFree(e->h_s);
  delete e;
}

int fib_emg_dims(const fib_emg_t* e, int32_t* nx, int32_t* ny, int32_t* nz) {
  if (!e) return efail(FIB_EINVAL, "null EMG handle");
  if (nx) *nx = e->g.nx;
  if (ny) *ny = e->g.ny;
  if (nz) *nz = e->g.nz;
  return FIB_OK;
}

int fib_emg_solve(fib_emg_t* e, double tol, int32_t max_iter, int32_t* iters, double* rel_res) {
  if (!e) return efail(FIB_EINVAL, "null EMG handle");
  if (!(std::isfinite(tol) && tol > 0.0) || max_iter < 0)
    return efail(FIB_EINVAL, "tol must be > 0 and max_iter >= 0");
  const fib::CtxView v = fib::ctx_view(e->ctx);
  if (!v.state_ready) return efail(FIB_ESTATE, "state not initialized");
  if (e->fdm) {
    if (int rc = fdm_solve(e, v, tol, max_iter)) return rc;
    if (iters) *iters = e->h_s->it;
    if (rel_res) *rel_res = e->h_s->bb > 0.0 ? std::sqrt(e->h_s->rr / e->h_s->bb) : 0.0;
    return FIB_OK;
  }
  hipStream_t st = v.stream;
  const Grid3 g = e->g;
  const float dx = (float)e->p.sigma_et, dy = (float)e->p.sigma_et,
              dz = (float)(e->p.sigma_el + e->p.sigma_i);
  const dim3 grid = e->grid, block(kB), one(1);
  const int nb = e->nblocks;
  // the tolerance; the host bounds the iterations
  e->h_s->tol2 = tol * tol;
  EHIP(hipMemcpyAsync(&e->d_s->tol2, &e->h_s->tol2, sizeof(double), hipMemcpyHostToDevice, st));
  hipLaunchKernelGGL(k_emg_rhs, grid, block, 0, st, g, v.d_state, e->n_fib, e->p.stride,
                     e->p.sigma_i, e->b(), e->d_part);
  hipLaunchKernelGGL(k_emg_mean, one, block, 0, st, e->d_part, nb, g.n, e->d_s);
  hipLaunchKernelGGL(k_emg_start, grid, block, 0, st, g, dx, dy, dz, e->b(), e->x(),
                     e->invd(), e->r(), e->part_r(0), e->part_pq(), e->d_s);
  hipLaunchKernelGGL(k_emg_started, one, block, 0, st, e->part_r(0), e->part_pq(), nb, g.n,
                     e->d_s);
  EHIP(hipGetLastError());
  // Iterations in batches between host checks.  The first batch is 8; then
  // the residual's mean decay rate over the last batch predicts how many
  // iterations remain, and the next batch is that (+ 25 %, at most 64), so
  // a solve wastes few no-op launches past convergence and few round trips.
  int32_t launched = 0;
  int batch = 8;
  double rr_last = -1.0;
  int32_t it_last = 0;
  for (;;) {
    EHIP(hipMemcpyAsync(e->h_s, e->d_s, sizeof(Scal), hipMemcpyDeviceToHost, st));
    EHIP(hipStreamSynchronize(st));
    if (e->h_s->done || launched >= max_iter) break;
    const double rr = e->h_s->rr, goal = e->h_s->tol2 * e->h_s->bb;
    if (rr_last > 0.0 && rr > 0.0 && rr < rr_last && e->h_s->it > it_last) {
      const double per_it = std::log(rr / rr_last) / (double)(e->h_s->it - it_last);
      const double need = std::log(goal / rr) / per_it;  // > 0: rr > goal here
      batch = (int)std::min(64.0, std::max(2.0, std::ceil(1.25 * need) + 1.0));
    } else if (rr_last > 0.0) {
      batch = std::min(2 * batch, 64);
    }
    rr_last = rr;
    it_last = e->h_s->it;
    const int n_it = std::min(batch, max_iter - launched);
    for (int b = 0; b < n_it; ++b) {
      const int P = (launched + b) & 1;
      hipLaunchKernelGGL(k_cg_q, grid, block, 0, st, g, dx, dy, dz, e->r(), e->invd(),
                         e->pb(P), e->pb(P ^ 1), e->q(), e->part_r(P), e->part_pq(), nb, P,
                         e->d_s);
      hipLaunchKernelGGL(k_cg_x, grid, block, 0, st, g, e->pb(P ^ 1), e->q(), e->invd(),
                         e->x(), e->r(), e->part_pq(), e->part_r(P ^ 1), nb, P, e->d_s);
    }
    EHIP(hipGetLastError());
    launched += n_it;
  }
  if (!e->h_s->done && launched > 0) {
    // stopped by the limit: the residual of the last iterate
    hipLaunchKernelGGL(k_cg_final, one, block, 0, st, e->part_r(launched & 1), nb, g.n, e->d_s);
    EHIP(hipGetLastError());
    EHIP(hipMemcpyAsync(e->h_s, e->d_s, sizeof(Scal), hipMemcpyDeviceToHost, st));
    EHIP(hipStreamSynchronize(st));
  }
  const int32_t done_it = e->h_s->it;
  if (e->h_s->bb == 0.0) {
    // b = 0: phi_e is a constant, zero after the projection
    EHIP(hipMemsetAsync(e->x(), 0, sizeof(float) * g.n, st));
  } else {
    hipLaunchKernelGGL(k_emg_sum, grid, block, 0, st, g, e->x(), e->d_part);
    hipLaunchKernelGGL(k_emg_mean, one, block, 0, st, e->d_part, nb, g.n, e->d_s);
    hipLaunchKernelGGL(k_emg_shift, grid, block, 0, st, g, e->x(), e->d_s);
    EHIP(hipGetLastError());
  }
  EHIP(hipStreamSynchronize(st));
  if (iters) *iters = done_it;
  if (rel_res) *rel_res = e->h_s->bb > 0.0 ? std::sqrt(e->h_s->rr / e->h_s->bb) : 0.0;
  return FIB_OK;
}

int fib_emg_get_phi(fib_emg_t* e, double* phi, int64_t n) {
  if (!e) return efail(FIB_EINVAL, "null EMG handle");
  if (n != e->g.n || !phi) return efail(FIB_EINVAL, "expected %lld values", (long long)e->g.n);
  std::vector<float> h(n);
  EHIP(hipStreamSynchronize(fib::ctx_view(e->ctx).stream));
  EHIP(hipMemcpy(h.data(), e->x(), sizeof(float) * n, hipMemcpyDeviceToHost));
  for (int64_t i = 0; i < n; ++i) phi[i] = h[i];
  return FIB_OK;
}

int fib_emg_get_rhs(fib_emg_t* e, double* rhs, int64_t n) {
  if (!e) return efail(FIB_EINVAL, "null EMG handle");
  if (n != e->g.n || !rhs) return efail(FIB_EINVAL, "expected %lld values", (long long)e->g.n);
  std::vector<float> h(n);
  EHIP(hipStreamSynchronize(fib::ctx_view(e->ctx).stream));
  EHIP(hipMemcpy(h.data(), e->b(), sizeof(float) * n, hipMemcpyDeviceToHost));
  for (int64_t i = 0; i < n; ++i) rhs[i] = h[i];
  return FIB_OK;
}

}  // extern "C"
