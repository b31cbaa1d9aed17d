// The vertex reparameterisation of the mesh optimiser: solves
// (I + lambda L) x = b for the three coordinate columns, L the combinatorial
// Laplacian D - A of the mesh's edge graph, by Chebyshev iteration on the
// device.  The matrix's eigenvalues lie in [1, 1 + lambda m], m = the largest
// d_v + (mean degree of v's neighbours) over the vertices v (an upper bound of
// L's largest eigenvalue, Merris 1998; never above the largest d_i + d_j over
// the edges), and on a known interval the Chebyshev recurrence's scalars are
// fixed numbers, computed on the host: an iteration takes no inner product, so
// it is one kernel, where conjugate gradients need two with a global sum each.
// A step runs on the iterates alone, x_{k+1} = x_k + c1 (x_k - x_{k-1}) + c2 (b -
// A x_k): it reads x_k, x_{k-1} and b and writes x_{k+1} over x_{k-1}, 20 MB at
// 155,992 vertices, where carrying the residual and the correction (x += d, r -= A d,
// d' = c1 d + c2 r) moves 30 (6.1 against 7.7 us a step; with the correction kept
// but the residual taken afresh 7.2).  But the recurrence amplifies the rounding of
// x in its residual by up to sqrt(condition): on a star with eigenvalues up to 4e5
// it stalled at 3e-8.  So from the condition number at which that could come near
// the tolerance the residual is carried.
//
// After k steps the residual is p_k(A) r_0 with |p_k| <= 1 / T_k(sigma) on the
// interval, so the step at which that bound meets the tolerance is known in
// advance, and the residual's norm (summed in a fixed order, read back) is looked
// at every CHECK steps from shortly before it, not from the start.  The solve is
// deterministic.
#include <math.h>

#include "dt_internal.h"

namespace {

constexpr int ST = 256;          // threads per block
constexpr int WAVES = ST / 64;
constexpr int CHECK = 16;        // steps between residual read-backs, once they start

struct SmoothWs {
  double* r;        // [nv][3] the carried residual; else the other iterate (even steps write the caller's x)
  double* d[2];     // [nv][3] carried: corrections, iteration k reads d[k & 1] and writes d[(k + 1) & 1]
  double* part;     // [2][blocks][3] partial b . b and r . r
  double* sums;     // [8]: b . b, r . r per column; [6] the bound m
  // in the corrections' room until a carried recurrence takes it:
  int4* nbr;        // [nv][2] the first NBR neighbours of each vertex (itself where there are fewer)
  int* deg;         // [nv] degrees
  double* bmax;     // [blocks] largest eigenvalue bound of the block's vertices
};

constexpr int NBR = 8;
constexpr unsigned DIES = 8;

size_t smooth_layout(int32_t nv, SmoothWs* w, char* base) {
  size_t o = 0;
  auto take = [&](size_t bytes) {
    size_t at = o;
    o = dt_align(o + bytes);
    return base ? (double*)(base + at) : nullptr;
  };
  SmoothWs t;
  t.r = take(3 * (size_t)nv * sizeof(double));
  t.d[0] = take(3 * (size_t)nv * sizeof(double));
  t.d[1] = take(3 * (size_t)nv * sizeof(double));
  const size_t nb = dt_blocks(nv, ST);
  t.part = take(6 * nb * sizeof(double));
  t.sums = take(8 * sizeof(double));
  // 36 bytes a vertex and 8 a block, of the 48 a vertex that the corrections hold
  t.nbr = (int4*)t.d[0];
  t.deg = base ? (int*)(t.nbr + 2 * (size_t)nv) : nullptr;
  t.bmax = base ? (double*)(t.deg + 2 * (((size_t)nv + 1) / 2)) : nullptr;
  if (w) *w = t;
  return o;
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int m = 32; m > 0; m >>= 1) v += __shfl_xor(v, m, 64);
  return v;
}

// the block's sums of v[0..2] over its threads, in a fixed order
__device__ __forceinline__ void block_sum3(const double v[3], double out[3]) {
  __shared__ double sh[3][WAVES];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const double s = wave_sum(v[c]);
    if (lane == 0) sh[c][wv] = s;
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < WAVES; ++k) s += sh[c][k];
    out[c] = s;
  }
  __syncthreads();
}

// this block's sums of v[0..2] into part[blockIdx]
__device__ __forceinline__ void block_partial(const double v[3], double* part) {
  double s[3];
  block_sum3(v, s);
  if (threadIdx.x == 0)
    for (int c = 0; c < 3; ++c) part[3 * blockIdx.x + c] = s[c];
}

struct D3 {
  double x, y, z;
};
__device__ __forceinline__ D3 load_d3(const double* p, int64_t i) { return ((const D3*)p)[i]; }
__device__ __forceinline__ double comp(const D3& v, int c) { return c == 0 ? v.x : (c == 1 ? v.y : v.z); }

// the first NBR neighbours of vertex i (itself where there are fewer); its degree
__device__ __forceinline__ int first_neighbours(const int32_t* off, const int32_t* adj, int i, int j[NBR]) {
  const int a = off[i], deg = off[i + 1] - a;
#pragma unroll
  for (int k = 0; k < NBR; ++k) j[k] = k < deg ? adj[a + k] : i;
  return deg;
}

// y = (I + lambda L) v at vertex i, (1 + lambda deg) v_i - lambda sum_j v_j, and
// v_i.  TABLE: a vertex's first NBR neighbours come from the table that the
// solve's first kernel makes of the adjacency, so a step waits for one table read
// and one round of value reads; else (the carried recurrence has taken the
// table's room) from the lists, all their indices at once.  Walking the list
// index by index, each with its value, was most of a step's 10.9 us.
template <bool TABLE>
__device__ __forceinline__ void apply_row(const int32_t* off, const int32_t* adj, const SmoothWs& w, int i,
                                          double lambda, const double* v, D3& vi, double y[3]) {
  int deg, j[NBR];
  vi = load_d3(v, i);
  if constexpr (TABLE) {
    deg = w.deg[i];
    const int4 j0 = w.nbr[2 * (size_t)i], j1 = w.nbr[2 * (size_t)i + 1];
    j[0] = j0.x, j[1] = j0.y, j[2] = j0.z, j[3] = j0.w;
    j[4] = j1.x, j[5] = j1.y, j[6] = j1.z, j[7] = j1.w;
  } else {
    deg = first_neighbours(off, adj, i, j);
  }
  D3 n[NBR];
#pragma unroll
  for (int k = 0; k < NBR; ++k) n[k] = load_d3(v, j[k]);
  double s0 = 0.0, s1 = 0.0, s2 = 0.0;
#pragma unroll
  for (int k = 0; k < NBR; ++k) {
    s0 += k < deg ? n[k].x : 0.0;
    s1 += k < deg ? n[k].y : 0.0;
    s2 += k < deg ? n[k].z : 0.0;
  }
  if (deg > NBR) {
    const int a = off[i];
    for (int k = a + NBR; k < a + deg; ++k) {
      const D3 q = load_d3(v, adj[k]);
      s0 += q.x;
      s1 += q.y;
      s2 += q.z;
    }
  }
  const double dg = 1.0 + lambda * (double)deg;
  y[0] = dg * vi.x - lambda * s0;
  y[1] = dg * vi.y - lambda * s1;
  y[2] = dg * vi.z - lambda * s2;
}

// the neighbour table
__global__ void __launch_bounds__(ST) k_sm_table(const int32_t* off, const int32_t* adj, int nv, SmoothWs w) {
  const int i = blockIdx.x * ST + threadIdx.x;
  if (i >= nv) return;
  int j[NBR];
  w.deg[i] = first_neighbours(off, adj, i, j);
  w.nbr[2 * (size_t)i] = make_int4(j[0], j[1], j[2], j[3]);
  w.nbr[2 * (size_t)i + 1] = make_int4(j[4], j[5], j[6], j[7]);
}

// r = b - A x; partials of b . b (part[0 .. nb)) and r . r
// (part[nb .. 2 nb)), and the largest eigenvalue bound of the block's vertices
__global__ void __launch_bounds__(ST) k_sm_init(const int32_t* off, const int32_t* adj, int nv, double lambda,
                                                const double* b, const double* x, SmoothWs w) {
  const int i = blockIdx.x * ST + threadIdx.x;
  double bb[3] = {0.0, 0.0, 0.0}, rr[3] = {0.0, 0.0, 0.0}, m = 0.0;
  if (i < nv) {
    double ax[3];
    D3 xi;
    apply_row<true>(off, adj, w, i, lambda, x, xi, ax);
    const D3 bi = load_d3(b, i);
    const D3 r = {bi.x - ax[0], bi.y - ax[1], bi.z - ax[2]};
    ((D3*)w.r)[i] = r;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      bb[c] = comp(bi, c) * comp(bi, c);
      rr[c] = comp(r, c) * comp(r, c);
    }
    const int a = off[i], e = off[i + 1];
    int sum = 0;
    for (int k = a; k < e; ++k) sum += w.deg[adj[k]];
    // rounded up: the interval must not be too short
    m = e > a ? ((double)(e - a) + (double)sum / (double)(e - a)) * (1.0 + 1e-14) : 0.0;
  }
  block_partial(rr, w.part + 3 * gridDim.x);
  block_partial(bb, w.part);
  __shared__ double sh[WAVES];
  for (int s = 32; s > 0; s >>= 1) m = fmax(m, __shfl_xor(m, s, 64));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 0; k < WAVES; ++k) m = fmax(m, sh[k]);
    w.bmax[blockIdx.x] = m;
  }
}

// partials of r . r (part[nb .. 2 nb)), r the carried residual or (x given) b - A x
__global__ void __launch_bounds__(ST) k_sm_norm(const int32_t* off, const int32_t* adj, int nv, double lambda,
                                                const double* b, const double* x, SmoothWs w) {
  const int i = blockIdx.x * ST + threadIdx.x;
  double rr[3] = {0.0, 0.0, 0.0};
  if (i < nv) {
    D3 r;
    if (x) {
      double ax[3];
      D3 xi;
      apply_row<true>(off, adj, w, i, lambda, x, xi, ax);
      const D3 bi = load_d3(b, i);
      r = {bi.x - ax[0], bi.y - ax[1], bi.z - ax[2]};
    } else {
      r = load_d3(w.r, i);
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) rr[c] = comp(r, c) * comp(r, c);
  }
  block_partial(rr, w.part + 3 * gridDim.x);
}

// sums[0..3) = sum of part[0 .. nb) (with both), sums[3..6) = sum of
// part[nb .. 2 nb), in block order; with both, sums[6] = the largest bmax
__global__ void __launch_bounds__(ST) k_sm_sums(int nb, int both, SmoothWs w) {
  for (int h = both ? 0 : 1; h < 2; ++h) {
    double a[3] = {0.0, 0.0, 0.0};
    const double* part = w.part + 3 * (size_t)nb * h;
    for (int k = threadIdx.x; k < nb; k += ST)
      for (int c = 0; c < 3; ++c) a[c] += part[3 * k + c];
    double s[3];
    block_sum3(a, s);
    if (threadIdx.x == 0)
      for (int c = 0; c < 3; ++c) w.sums[3 * h + c] = s[c];
  }
  if (both) {
    __shared__ double sh[WAVES];
    double m = 0.0;
    for (int k = threadIdx.x; k < nb; k += ST) m = fmax(m, w.bmax[k]);
    for (int s = 32; s > 0; s >>= 1) m = fmax(m, __shfl_xor(m, s, 64));
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int k = 0; k < WAVES; ++k) m = fmax(m, sh[k]);
      w.sums[6] = m;
    }
  }
}

// Consecutive workgroups go to the chip's dies in turn: die k takes the k-th
// stretch of the vertices, so most neighbours' values lie in its own L2 (7.1 ->
// 6.1 us a step).
__device__ __forceinline__ int step_vertex() {
  return (int)((blockIdx.x % DIES) * (gridDim.x / DIES) + blockIdx.x / DIES) * ST + (int)threadIdx.x;
}

// One Chebyshev step on the iterates: prev = x + c1 (x - prev) + c2 (b - A x).
// first: prev holds nothing yet (c1 = 0).  Bound by latency and launch: 6.1 us a
// step at 155,992 vertices (4 us for its 20 MB at the rate of a copy).
__global__ void __launch_bounds__(ST) k_sm_step(const int32_t* off, const int32_t* adj, int nv, double lambda,
                                                int first, const double* b, const double* x, double* prev,
                                                double c1, double c2, SmoothWs w) {
  const int i = step_vertex();
  if (i >= nv) return;
  const D3 bi = load_d3(b, i);
  D3 p = {0.0, 0.0, 0.0};
  if (!first) p = load_d3(prev, i);
  double ax[3];
  D3 xi;
  apply_row<true>(off, adj, w, i, lambda, x, xi, ax);
  if (first) p = xi;
  ((D3*)prev)[i] = {xi.x + c1 * (xi.x - p.x) + c2 * (bi.x - ax[0]), xi.y + c1 * (xi.y - p.y) + c2 * (bi.y - ax[1]),
                    xi.z + c1 * (xi.z - p.z) + c2 * (bi.z - ax[2])};
}

// The step with the residual carried: x += d, r -= A d, dn = c1 d + c2 r (the new
// r).  first: d holds a copy of r (over the table) and the correction is r / theta.
__global__ void __launch_bounds__(ST) k_sm_step_carry(const int32_t* off, const int32_t* adj, int nv, double lambda,
                                                      int first, double inv_theta, const double* d, double* dn,
                                                      double c1, double c2, double* x, SmoothWs w) {
  const int i = step_vertex();
  if (i >= nv) return;
  const double sc = first ? inv_theta : 1.0;
  const D3 xi = load_d3(x, i), ri = load_d3(w.r, i);
  double ad[3];
  D3 di;
  apply_row<false>(off, adj, w, i, lambda, d, di, ad);
  const D3 dk = {sc * di.x, sc * di.y, sc * di.z};
  ((D3*)x)[i] = {xi.x + dk.x, xi.y + dk.y, xi.z + dk.z};
  const D3 r = {ri.x - sc * ad[0], ri.y - sc * ad[1], ri.z - sc * ad[2]};
  ((D3*)w.r)[i] = r;
  ((D3*)dn)[i] = {c1 * dk.x + c2 * r.x, c1 * dk.y + c2 * r.y, c1 * dk.z + c2 * r.z};
}

__global__ void __launch_bounds__(ST) k_sm_copy(double* dst, const double* src, int64_t n) {
  const int64_t i = blockIdx.x * (int64_t)ST + threadIdx.x;
  if (i < n) dst[i] = src[i];
}

}  // namespace

extern "C" dt_status dt_smooth_bytes(int32_t nv, size_t* ws_bytes) {
  DT_REQUIRE(ws_bytes, "dt_smooth_bytes: ws_bytes is NULL");
  DT_REQUIRE(nv >= 1 && nv < (1 << 28), "dt_smooth_bytes: nv must be in [1, 2^28) (got %d)", nv);
  *ws_bytes = smooth_layout(nv, nullptr, nullptr);
  return DT_OK;
}

extern "C" dt_status dt_smooth_solve(const int32_t* adj_off, const int32_t* adj, int32_t nv, double lambda,
                                     const double* b, double* x, double tol, int32_t max_iters,
                                     int32_t* iters_out, double* resid_out, void* ws, size_t ws_bytes,
                                     void* stream) {
  DT_REQUIRE(adj_off && adj && b && x && ws, "dt_smooth_solve: a required pointer is NULL");
  DT_REQUIRE(nv >= 1 && nv < (1 << 28), "dt_smooth_solve: nv must be in [1, 2^28) (got %d)", nv);
  DT_REQUIRE(lambda >= 0.0 && tol > 0.0 && max_iters >= 1,
             "dt_smooth_solve: needs lambda >= 0, tol > 0, max_iters >= 1");
  const size_t need = smooth_layout(nv, nullptr, nullptr);
  if (ws_bytes < need) {
    dt_set_error("dt_smooth_solve: workspace has %zu bytes, needs %zu", ws_bytes, need);
    return DT_ERR_WORKSPACE_TOO_SMALL;
  }
  SmoothWs w;
  smooth_layout(nv, &w, (char*)ws);
  hipStream_t s = (hipStream_t)stream;
  const int nb = (int)dt_blocks(nv, ST);
  hipLaunchKernelGGL(k_sm_table, dim3(nb), dim3(ST), 0, s, adj_off, adj, nv, w);
  hipLaunchKernelGGL(k_sm_init, dim3(nb), dim3(ST), 0, s, adj_off, adj, nv, lambda, b, x, w);
  hipLaunchKernelGGL(k_sm_sums, dim3(1), dim3(ST), 0, s, nb, 1, w);
  DT_CHECK_LAUNCH();
  double sums[7];
  DT_CHECK_HIP(hipMemcpyAsync(sums, w.sums, sizeof(sums), hipMemcpyDeviceToHost, s));
  DT_CHECK_HIP(hipStreamSynchronize(s));
  // eigenvalues in [1, 1 + lambda m]
  const double lo = 1.0, hi = 1.0 + lambda * sums[6];
  const double theta = 0.5 * (hi + lo), delta = 0.5 * (hi - lo);
  double b2[3], lim[3];
  for (int c = 0; c < 3; ++c) {
    b2[c] = sums[c] > 1e-300 ? sums[c] : 1e-300;
    lim[c] = tol * tol * b2[c];
  }
  auto within_tol = [&](const double* rr, double& worst) {
    bool ok = true;
    worst = 0.0;
    for (int c = 0; c < 3; ++c) {
      ok = ok && rr[c] <= lim[c];
      worst = fmax(worst, rr[c] / b2[c]);
    }
    return ok;
  };
  double worst = 0.0;
  bool done = within_tol(sums + 3, worst);
  int it = 0;
  // rho_0 = delta / theta, rho_{k+1} = 1 / (2 sigma - rho_k), sigma = theta / delta;
  // d_{k+1} = rho_{k+1} rho_k d_k + (2 rho_{k+1} / delta) r_{k+1} (a matrix with
  // one eigenvalue, delta = 0, is solved by the first step alone)
  const bool single = delta <= 1e-12 * theta;
  const double sigma = single ? 0.0 : theta / delta;
  double rho = single ? 0.0 : delta / theta;
  // the first look: the last multiple of CHECK a little before the step whose
  // bound 1 / T_k(sigma) takes the residual to the tolerance
  int first_look = CHECK;
  if (!single && !done) {
    const double need = acosh(fmax(sqrt(worst) / tol, 1.0)) / acosh(sigma);
    const double at = fmin(need - 0.5 * CHECK, (double)max_iters);
    if (at > CHECK) first_look = (int)(at / CHECK) * CHECK;
  }
  // on the iterates while the amplified rounding, some condition^(3/2) u (3e-8 at
  // 4e5 is once that), stays a factor of 32 below the tolerance
  // (carried also where x shares memory with b, which only the first kernel reads
  // then: each step on the iterates reads b anew)
  const bool shared = (const char*)b < (const char*)(x + 3 * (size_t)nv) &&
                      (const char*)x < (const char*)(b + 3 * (size_t)nv);
  const bool carry = shared || 32.0 * hi * sqrt(hi) * 1.1102230246251565e-16 > tol;
  const unsigned grid = (unsigned)(nb + DIES - 1) / DIES * DIES;
  double* const xs[2] = {x, w.r};  // not carried: step it reads xs[(it - 1) & 1] and writes xs[it & 1]
  double d1 = 0.0, d2 = 1.0 / theta;  // not carried: this step's c1, c2
  const dim3 all3(dt_blocks(3 * (int64_t)nv, ST));
  if (carry && !done) hipLaunchKernelGGL(k_sm_copy, all3, dim3(ST), 0, s, w.d[0], w.r, 3 * (int64_t)nv);
  while (!done && it < max_iters) {
    double c1 = 0.0, c2 = 0.0;  // carried: the next correction's; else the next step's
    if (!single) {
      const double rn = 1.0 / (2.0 * sigma - rho);
      c1 = rn * rho;
      c2 = 2.0 * rn / delta;
      rho = rn;
    }
    ++it;
    if (carry)
      hipLaunchKernelGGL(k_sm_step_carry, dim3(grid), dim3(ST), 0, s, adj_off, adj, nv, lambda, (int)(it == 1),
                         1.0 / theta, w.d[(it - 1) & 1], w.d[it & 1], c1, c2, x, w);
    else
      hipLaunchKernelGGL(k_sm_step, dim3(grid), dim3(ST), 0, s, adj_off, adj, nv, lambda, (int)(it == 1), b,
                         xs[(it - 1) & 1], xs[it & 1], d1, d2, w);
    d1 = c1;
    d2 = c2;
    if ((it % CHECK == 0 && it >= first_look) || it == max_iters || single) {
      hipLaunchKernelGGL(k_sm_norm, dim3(nb), dim3(ST), 0, s, adj_off, adj, nv, lambda, b,
                         carry ? nullptr : xs[it & 1], w);
      hipLaunchKernelGGL(k_sm_sums, dim3(1), dim3(ST), 0, s, nb, 0, w);
      DT_CHECK_LAUNCH();
      DT_CHECK_HIP(hipMemcpyAsync(sums + 3, w.sums + 3, 3 * sizeof(double), hipMemcpyDeviceToHost, s));
      DT_CHECK_HIP(hipStreamSynchronize(s));
      done = within_tol(sums + 3, worst);
    }
  }
  if (!carry && (it & 1))  // the last iterate lies in the workspace
    hipLaunchKernelGGL(k_sm_copy, all3, dim3(ST), 0, s, x, w.r, 3 * (int64_t)nv);
  DT_CHECK_LAUNCH();
  if (iters_out) *iters_out = it;
  if (resid_out) *resid_out = sqrt(worst);
  if (!done) {
    dt_set_error("dt_smooth_solve: relative residual %.3e above %.1e after %d iterations", sqrt(worst), tol,
                 it);
    return DT_ERR_NOT_CONVERGED;
  }
  return DT_OK;
}
