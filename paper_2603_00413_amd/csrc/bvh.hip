// Scene build on the device: unit face normals, vertex normals (paper Eq. 13),
// and a linear BVH over the triangles (Morton order, binary radix tree,
// bottom-up box fit).  Everything here is deterministic: integer atomics
// only count, FP32 sums run in a fixed order.
#include <stdarg.h>
#include <stdio.h>

#include <mutex>

#include "dt_internal.h"

namespace {

constexpr int SCAN_NB = 256;  // blocks (= partial sums) of the chunked device scan
constexpr int TILE_PASSES = 8;  // treelet restructuring passes inside the tiles
constexpr int TOP_PASSES = 2;   // and over the nodes that span tiles
constexpr int SCAN_T = 256;

// ------------------------------------------------------------------ block scans
template <class T>
__device__ T block_incl_scan(T v, T* sh) {
  const int t = threadIdx.x;
  sh[t] = v;
  __syncthreads();
  for (int off = 1; off < (int)blockDim.x; off <<= 1) {
    T x = t >= off ? sh[t - off] : T(0);
    __syncthreads();
    sh[t] += x;
    __syncthreads();
  }
  return sh[t];
}

template <class T>
__global__ void k_scan_reduce(const T* in, int32_t n, int32_t chunk, T* part) {
  __shared__ T sh[SCAN_T];
  int64_t lo = (int64_t)blockIdx.x * chunk;
  int64_t hi = lo + chunk < n ? lo + chunk : n;
  T s = 0;
  for (int64_t i = lo + threadIdx.x; i < hi; i += blockDim.x) s += in[i];
  T tot = block_incl_scan(s, sh);
  if (threadIdx.x == blockDim.x - 1) part[blockIdx.x] = tot;
}

// exclusive scan of part[0..nb) in place; part[nb] = total, also to *total
template <class T>
__global__ void k_scan_partials(T* part, int nb, T* total) {
  __shared__ T sh[SCAN_NB];
  int t = threadIdx.x;
  T v = t < nb ? part[t] : 0;
  T inc = block_incl_scan(v, sh);
  __syncthreads();
  if (t < nb) part[t] = inc - v;
  if (t == (int)blockDim.x - 1) {
    part[nb] = inc;
    if (total) *total = inc;
  }
}

template <class T>
__global__ void k_scan_apply(const T* in, T* out, int32_t n, int32_t chunk, const T* part) {
  __shared__ T sh[SCAN_T];
  int64_t lo = (int64_t)blockIdx.x * chunk;
  int64_t hi = lo + chunk < n ? lo + chunk : n;
  T carry = part[blockIdx.x];
  for (int64_t base = lo; base < hi; base += blockDim.x) {
    int64_t i = base + threadIdx.x;
    T v = i < hi ? in[i] : 0;
    T inc = block_incl_scan(v, sh);
    T tot = sh[blockDim.x - 1];
    if (i < hi) out[i] = carry + inc - v;
    carry += tot;
    __syncthreads();
  }
}

// the whole scan in one block, SCAN_ONE elements a step: a launch costs about as
// much as two steps (2.4 us each), so up to SCAN_ONE_MAX elements it beats the
// three kernels above (10 us)
constexpr int SCAN_ONE_T = 1024;
constexpr int SCAN_ONE = 4 * SCAN_ONE_T;
constexpr int SCAN_ONE_MAX = 2 * SCAN_ONE;
template <class T>
__global__ void __launch_bounds__(SCAN_ONE_T) k_scan_one(const T* in, T* out, int32_t n, T* part, T* total) {
  __shared__ T wsum[SCAN_ONE_T / 64];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  T carry = 0;
  for (int base = 0; base < n; base += SCAN_ONE) {
    const int i = base + 4 * t;
    T v[4], s = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v[k] = i + k < n ? in[i + k] : (T)0;
      s += v[k];
    }
    T inc = s;
#pragma unroll
    for (int st = 1; st < 64; st <<= 1) {
      const T up = __shfl_up(inc, st);
      if (lane >= st) inc += up;
    }
    if (lane == 63) wsum[wv] = inc;
    __syncthreads();
    T before = carry, all = 0;
#pragma unroll
    for (int k = 0; k < SCAN_ONE_T / 64; ++k) {
      const T w = wsum[k];
      before += k < wv ? w : (T)0;
      all += w;
    }
    T run = before + inc - s;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (i + k < n) out[i + k] = run;
      run += v[k];
    }
    carry += all;
    __syncthreads();
  }
  if (t == 0) {
    part[SCAN_NB] = carry;
    if (total) *total = carry;
  }
}

// ------------------------------------------------------------------ normals
__device__ __forceinline__ bool face_ok(const int32_t* F, int f, int32_t nv) {
  int a = F[3 * f], b = F[3 * f + 1], c = F[3 * f + 2];
  return a >= 0 && a < nv && b >= 0 && b < nv && c >= 0 && c < nv;
}

// header, and the vertices' face counts cleared
__global__ void k_build_init(BvhHeader* hdr, int32_t nv, int32_t nf, int32_t* cnt) {
  const int v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v < nv) cnt[v] = 0;
  if (v == 0) {
    hdr->nv = nv;
    hdr->nf = nf;
    hdr->depth = nf == 1 ? 1 : 0;  // larger trees: k_wide_roots
    hdr->pad0 = 0;
  }
}

// Unit face normals, and the vertices' incident faces counted: corner k of
// face f is its vertex's rank[3 f + k]-th, in the order the atomics arrive
// (k_vnormals sorts the lists)
__global__ void k_faces(const float* V, const int32_t* F, int32_t nf, int32_t nv, float4* fn, int32_t* cnt,
                        int32_t* rank) {
  int f = blockIdx.x * blockDim.x + threadIdx.x;
  if (f >= nf) return;
  if (!face_ok(F, f, nv)) {
    fn[f] = make_float4(0.f, 0.f, 0.f, 0.f);
    return;
  }
  const int i0 = F[3 * f], i1 = F[3 * f + 1], i2 = F[3 * f + 2];
  rank[3 * (size_t)f] = atomicAdd(&cnt[i0], 1);
  rank[3 * (size_t)f + 1] = atomicAdd(&cnt[i1], 1);
  rank[3 * (size_t)f + 2] = atomicAdd(&cnt[i2], 1);
  v3 a = load3(V + 3 * i0), b = load3(V + 3 * i1), c = load3(V + 3 * i2);
  v3 n = cross(b - a, c - a);
  float l2 = dot(n, n);
  if (l2 > 0.0f) {
    v3 u = n * (1.0f / sqrtf(l2));
    fn[f] = make_float4(u.x, u.y, u.z, 1.0f);
  } else {
    fn[f] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
}

__global__ void k_vfill(const int32_t* F, int32_t nf, int32_t nv, const int32_t* off,
                        const int32_t* rank, int32_t* idx) {
  int f = blockIdx.x * blockDim.x + threadIdx.x;
  if (f >= nf || !face_ok(F, f, nv)) return;
  for (int k = 0; k < 3; ++k) idx[off[F[3 * f + k]] + rank[3 * (size_t)f + k]] = f;
}

// Each vertex's face list in ascending face order (fixed summation order), and
// Eq. 13: one third of the sum of the unit normals of the incident faces, in that
// order (not renormalised: the shading normal normalises the barycentric blend
// of Eq. 12 instead)
__global__ void k_vnormals(const int32_t* off, int32_t* idx, const float4* fn, int32_t nv, float4* vn) {
  int v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= nv) return;
  const int lo = off[v], hi = off[v + 1];
  for (int i = lo + 1; i < hi; ++i) {
    int x = idx[i];
    int j = i - 1;
    while (j >= lo && idx[j] > x) {
      idx[j + 1] = idx[j];
      --j;
    }
    idx[j + 1] = x;
  }
  v3 s = mk3(0.f, 0.f, 0.f);
  for (int i = lo; i < hi; ++i) s += xyz(fn[idx[i]]);
  v3 n = s * (1.0f / 3.0f);
  vn[v] = make_float4(n.x, n.y, n.z, 0.0f);
}

// ------------------------------------------------------------------ Morton codes
constexpr int NBB = 256;  // blocks of the bounds reduction

__device__ __forceinline__ int vclamp(int i, int nv) { return i < 0 ? 0 : (i >= nv ? nv - 1 : i); }

__device__ __forceinline__ v3 centroid(const float* V, const int32_t* F, int f, int nv) {
  v3 a = load3(V + 3 * vclamp(F[3 * f], nv)), b = load3(V + 3 * vclamp(F[3 * f + 1], nv));
  v3 c = load3(V + 3 * vclamp(F[3 * f + 2], nv));
  return (a + b + c) * (1.0f / 3.0f);
}

__global__ void k_bounds(const float* V, const int32_t* F, int32_t nf, int32_t nv, float* part) {
  __shared__ float sh[6][256];
  float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  for (int f = blockIdx.x * blockDim.x + threadIdx.x; f < nf; f += gridDim.x * blockDim.x) {
    v3 c = centroid(V, F, f, nv);
    lo[0] = fminf(lo[0], c.x);
    lo[1] = fminf(lo[1], c.y);
    lo[2] = fminf(lo[2], c.z);
    hi[0] = fmaxf(hi[0], c.x);
    hi[1] = fmaxf(hi[1], c.y);
    hi[2] = fmaxf(hi[2], c.z);
  }
  int t = threadIdx.x;
  for (int k = 0; k < 3; ++k) {
    sh[k][t] = lo[k];
    sh[3 + k][t] = hi[k];
  }
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if (t < s)
      for (int k = 0; k < 3; ++k) {
        sh[k][t] = fminf(sh[k][t], sh[k][t + s]);
        sh[3 + k][t] = fmaxf(sh[3 + k][t], sh[3 + k][t + s]);
      }
    __syncthreads();
  }
  if (t < 6) part[blockIdx.x * 6 + t] = sh[t][0];
}

__device__ __forceinline__ uint64_t spread21(uint32_t v) {
  uint64_t x = v & 0x1fffffu;
  x = (x | x << 32) & 0x1f00000000ffffull;
  x = (x | x << 16) & 0x1f0000ff0000ffull;
  x = (x | x << 8) & 0x100f00f00f00f00full;
  x = (x | x << 4) & 0x10c30c30c30c30c3ull;
  x = (x | x << 2) & 0x1249249249249249ull;
  return x;
}

__device__ __forceinline__ uint32_t quant21(float c, float lo, float ext) {
  if (!(ext > 0.0f)) return 0u;
  float q = (c - lo) / ext * 2097152.0f;
  q = fminf(fmaxf(q, 0.0f), 2097151.0f);
  return (uint32_t)q;
}

// keys: 63-bit Morton codes of the centroids (21 bits per axis) shifted right
// by `drop` bits (31 keeps the top 32, about 11 bits per axis).  Every block
// reduces k_bounds' partials to the scene bounds for itself; block 0 also
// writes them to the header.
template <class K>
__global__ void __launch_bounds__(NBB) k_morton(const float* V, const int32_t* F, int32_t nf, int32_t nv, int drop,
                                                const float* part, BvhHeader* hdr, K* keys, int32_t* vals) {
  __shared__ float sh[NBB / 64][6];
  const int t = threadIdx.x;
  float bb[6];
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    float x = part[t * 6 + k];
#pragma unroll
    for (int st = 32; st > 0; st >>= 1) {
      const float y = __shfl_xor(x, st);
      x = k < 3 ? fminf(x, y) : fmaxf(x, y);
    }
    if ((t & 63) == 0) sh[t >> 6][k] = x;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    bb[k] = sh[0][k];
#pragma unroll
    for (int w = 1; w < NBB / 64; ++w) bb[k] = k < 3 ? fminf(bb[k], sh[w][k]) : fmaxf(bb[k], sh[w][k]);
  }
  if (blockIdx.x == 0 && t == 0)
    for (int k = 0; k < 3; ++k) {
      hdr->lo[k] = bb[k];
      hdr->hi[k] = bb[3 + k];
    }
  const int f = blockIdx.x * NBB + t;
  if (f >= nf) return;
  v3 c = centroid(V, F, f, nv);
  uint32_t qx = quant21(c.x, bb[0], bb[3] - bb[0]);
  uint32_t qy = quant21(c.y, bb[1], bb[4] - bb[1]);
  uint32_t qz = quant21(c.z, bb[2], bb[5] - bb[2]);
  keys[f] = (K)(((spread21(qx) << 2) | (spread21(qy) << 1) | spread21(qz)) >> drop);
  vals[f] = f;
}

// ------------------------------------------------------------------ stable LSD radix sort
constexpr int RS_T = 256;
constexpr int RS_ITEMS = 8;  // keys per thread of the tile; 4 for short sorts (sort_and_link)
// SELF (short sorts): the histogram is [tile][digit] and each scatter block adds
// up the few tiles' columns itself; otherwise it is [digit][tile], scanned in
// place between the two kernels.
constexpr int RS_WAVES = RS_T / 64;

template <class K, int ITEMS, bool SELF>
__global__ void k_rs_hist(const K* keys, int32_t n, int shift, int32_t* hist, int ntiles) {
  __shared__ uint32_t h[256];
  for (int i = threadIdx.x; i < 256; i += blockDim.x) h[i] = 0;
  __syncthreads();
  int64_t base = (int64_t)blockIdx.x * (RS_T * ITEMS);
  for (int j = 0; j < ITEMS; ++j) {
    int64_t i = base + (int64_t)j * RS_T + threadIdx.x;
    if (i < n) atomicAdd(&h[(uint32_t)(keys[i] >> shift) & 255u], 1u);
  }
  __syncthreads();
  for (int dg = threadIdx.x; dg < 256; dg += blockDim.x)
    hist[SELF ? (size_t)blockIdx.x * 256 + dg : (size_t)dg * ntiles + blockIdx.x] = (int32_t)h[dg];
}

// lanes of the wave holding the same 8-bit digit (restricted to valid lanes)
__device__ __forceinline__ uint64_t digit_peers(uint32_t dg, bool valid) {
  uint64_t m = __ballot(valid);
  for (int b = 0; b < 8; ++b) {
    bool bit = (dg >> b) & 1u;
    uint64_t bb = __ballot(bit);
    m &= bit ? bb : ~bb;
  }
  return m;
}

// Each wave owns ITEMS * 64 consecutive keys of the tile; ranks are stable.
template <class K, int ITEMS, bool SELF>
__global__ void k_rs_scatter(const K* kin, const int32_t* vin, K* kout,
                             int32_t* vout, int32_t n, int shift, const int32_t* offs, int ntiles) {
  __shared__ uint32_t cnt[RS_WAVES][256];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int i = threadIdx.x; i < RS_WAVES * 256; i += blockDim.x) (&cnt[0][0])[i] = 0;
  __syncthreads();
  const int64_t wbase = (int64_t)blockIdx.x * (RS_T * ITEMS) + (int64_t)w * (ITEMS * 64);
  const uint64_t lt = (1ull << lane) - 1ull;
  for (int s = 0; s < ITEMS; ++s) {
    int64_t i = wbase + s * 64 + lane;
    bool valid = i < n;
    uint32_t dg = valid ? ((uint32_t)(kin[i] >> shift) & 255u) : 0u;
    uint64_t peers = digit_peers(dg, valid);
    if (valid && (peers & lt) == 0) cnt[w][dg] += (uint32_t)__popcll(peers);
  }
  __syncthreads();
  {
    static_assert(RS_T == 256, "a thread per digit");
    const int dg = threadIdx.x;
    uint32_t run = 0;
    if constexpr (SELF) {
      // keys of smaller digits anywhere, and of this one in earlier tiles
      uint32_t all = 0;
#pragma unroll 8
      for (int k = 0; k < ntiles; ++k) {
        const uint32_t c = (uint32_t)offs[(size_t)k * 256 + dg];
        all += c;
        run += k < (int)blockIdx.x ? c : 0u;
      }
      __shared__ uint32_t wsum[RS_WAVES];
      uint32_t inc = all;
#pragma unroll
      for (int st = 1; st < 64; st <<= 1) {
        const uint32_t up = __shfl_up(inc, st);
        if (lane >= st) inc += up;
      }
      if (lane == 63) wsum[w] = inc;
      __syncthreads();
      run += inc - all;
      for (int k = 0; k < w; ++k) run += wsum[k];
    } else {
      run = (uint32_t)offs[(size_t)dg * ntiles + blockIdx.x];
    }
    for (int ww = 0; ww < RS_WAVES; ++ww) {
      uint32_t c = cnt[ww][dg];
      cnt[ww][dg] = run;
      run += c;
    }
  }
  __syncthreads();
  for (int s = 0; s < ITEMS; ++s) {
    int64_t i = wbase + s * 64 + lane;
    bool valid = i < n;
    K k = valid ? kin[i] : (K)0;
    int32_t val = valid ? vin[i] : 0;
    uint32_t dg = (uint32_t)(k >> shift) & 255u;
    uint64_t peers = digit_peers(dg, valid);
    uint32_t pos = cnt[w][dg] + (uint32_t)__popcll(peers & lt);
    __builtin_amdgcn_wave_barrier();
    if (valid) {
      kout[pos] = k;
      vout[pos] = val;
      if ((peers & lt) == 0) cnt[w][dg] += (uint32_t)__popcll(peers);
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// ------------------------------------------------------------------ binary radix tree
__device__ __forceinline__ int key_clz(uint32_t x) { return __clz((int)x); }
__device__ __forceinline__ int key_clz(uint64_t x) { return __clzll((long long)x); }

template <class K>
__device__ __forceinline__ int kdelta(const K* k, int n, int i, int j) {
  if (j < 0 || j >= n) return -1;
  K a = k[i], b = k[j];
  if (a == b) return 8 * (int)sizeof(K) + __clz((uint32_t)(i ^ j));
  return key_clz((K)(a ^ b));
}

// Node i covers the sorted triangles between i and its other end.  topo[i]:
// children, parent, other end.  Also clears the node's arrival counter (k_tile)
// and cut membership (k_cut).
template <class K>
__global__ void k_karras(const K* keys, int n, int4* topo, int32_t* leaf_parent, int32_t* arrive, int32_t* member) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n - 1) return;
  arrive[i] = 0;
  member[i] = 0;
  int dl = kdelta(keys, n, i, i - 1), dr = kdelta(keys, n, i, i + 1);
  int d = dr > dl ? 1 : -1;
  int dmin = d > 0 ? dl : dr;
  int lmax = 2;
  while (kdelta(keys, n, i, i + lmax * d) > dmin) lmax <<= 1;
  int l = 0;
  for (int t = lmax >> 1; t >= 1; t >>= 1)
    if (kdelta(keys, n, i, i + (l + t) * d) > dmin) l += t;
  int j = i + l * d;
  int dnode = kdelta(keys, n, i, j);
  int s = 0, t = l;
  do {
    t = (t + 1) >> 1;
    if (kdelta(keys, n, i, i + (s + t) * d) > dnode) s += t;
  } while (t > 1);
  int gamma = i + s * d + (d < 0 ? -1 : 0);
  int lo = i < j ? i : j, hi = i < j ? j : i;
  int* nd = (int*)&topo[i];
  if (lo == gamma) {
    nd[0] = (int)((uint32_t)gamma | DT_LEAF_BIT);
    leaf_parent[gamma] = i;
  } else {
    nd[0] = gamma;
    ((int*)&topo[gamma])[2] = i;
  }
  if (hi == gamma + 1) {
    nd[1] = (int)((uint32_t)(gamma + 1) | DT_LEAF_BIT);
    leaf_parent[gamma + 1] = i;
  } else {
    nd[1] = gamma + 1;
    ((int*)&topo[gamma + 1])[2] = i;
  }
  nd[3] = j;
  if (i == 0) nd[2] = -1;
}

__device__ __forceinline__ v3 vmin(v3 a, v3 b) { return {fminf(a.x, b.x), fminf(a.y, b.y), fminf(a.z, b.z)}; }
__device__ __forceinline__ v3 vmax(v3 a, v3 b) { return {fmaxf(a.x, b.x), fmaxf(a.y, b.y), fmaxf(a.z, b.z)}; }

// Order-preserving map of floats to ints.
__device__ __forceinline__ int fenc(float f) {
  int i = __float_as_int(f);
  return i >= 0 ? i : i ^ 0x7FFFFFFF;
}

// ------------------------------------------------------------------ treelet restructuring
// The Morton-order tree groups triangles by space-filling-curve position, not
// by how much box surface the grouping costs, and the excess sits in the lower
// levels.  Each pass takes the nodes X at one depth parity as roots of
// disjoint two-level treelets: X, its internal children, and as treelet leaves
// the grandchildren (or a child that is itself a triangle), 3 or 4 of them.
// Among all binary trees over those leaves it keeps the one whose inner nodes
// have the least total surface area (the root's box, and every box below the
// treelet leaves, are unchanged), reusing X and its internal children as the
// inner nodes.  Treelets of one pass share no inner node, and a thread writes
// only its own inner nodes, the child fields of X (not X's parent link) and
// the parent links of its treelet leaves, so the threads of a pass are
// independent.  Alternating parities over passes lets changes travel.
struct TBox {
  v3 lo, hi;
};
__device__ __forceinline__ TBox tunion(const TBox& a, const TBox& b) {
  return {vmin(a.lo, b.lo), vmax(a.hi, b.hi)};
}
__device__ __forceinline__ float tarea(const TBox& b) {
  v3 e = vmax(b.hi - b.lo, mk3(0.f, 0.f, 0.f));
  return 2.f * (e.x * e.y + e.y * e.z + e.z * e.x);
}
__device__ __forceinline__ TBox read_box(const float* p) {
  return {mk3(p[0], p[1], p[2]), mk3(p[3], p[4], p[5])};
}
__device__ __forceinline__ void write_box(float* p, const TBox& b) {
  p[0] = b.lo.x;
  p[1] = b.lo.y;
  p[2] = b.lo.z;
  p[3] = b.hi.x;
  p[4] = b.hi.y;
  p[5] = b.hi.z;
}
__device__ __forceinline__ TBox get_box(const BvhNode& n, int slot) { return read_box((const float*)&n + slot * 6); }

// nodes in device memory, as treelet_root sees them: child references, the two
// child boxes (12 floats), and the parent link
struct GlobalNodes {
  BvhNode* n;
  __device__ __forceinline__ int* kids(int i) const { return (int*)&n[i].d; }
  __device__ __forceinline__ float* boxes(int i) const { return (float*)&n[i]; }
  __device__ __forceinline__ void set_up(int i, int parent) const { ((int*)&n[i].d)[2] = parent; }
};

template <class N>
__device__ __forceinline__ void set_node(const N& A, int i, int c0, const TBox& b0, int c1, const TBox& b1) {
  write_box(A.boxes(i), b0);
  write_box(A.boxes(i) + 6, b1);
  A.kids(i)[0] = c0;
  A.kids(i)[1] = c1;
}

template <class N>
__device__ __forceinline__ void set_parent(const N& A, int ref, int parent) {
  if (!((uint32_t)ref & DT_LEAF_BIT)) A.set_up(ref, parent);  // triangles keep no link
}

template <class N>
__device__ __forceinline__ void treelet_root(const N& A, int X) {
  const int k0 = A.kids(X)[0], k1 = A.kids(X)[1];
  const bool leaf0 = ((uint32_t)k0 & DT_LEAF_BIT) != 0u, leaf1 = ((uint32_t)k1 & DT_LEAF_BIT) != 0u;
  if (leaf0 && leaf1) return;
  // candidate topologies, costs = summed areas of the inner nodes below X
  if (leaf0 || leaf1) {
    // three leaves, P1's two and X's own: ((a b) c), the pair with the least box area
    const int P1 = leaf0 ? k1 : k0, r2 = leaf0 ? k0 : k1;
    const int r0 = A.kids(P1)[0], r1 = A.kids(P1)[1];
    const TBox b0 = read_box(A.boxes(P1)), b1 = read_box(A.boxes(P1) + 6);
    const TBox b2 = read_box(A.boxes(X) + (leaf0 ? 0 : 6));
    const float c01 = tarea(tunion(b0, b1)), c02 = tarea(tunion(b0, b2)), c12 = tarea(tunion(b1, b2));
    if (!(c02 < c01) && !(c12 < c01)) return;  // already the best
    const bool with0 = !(c12 < c02);           // the pair is (0 2), else (1 2)
    const int rp = with0 ? r0 : r1, rs = with0 ? r1 : r0;
    const TBox bp = with0 ? b0 : b1, bs = with0 ? b1 : b0;
    set_node(A, P1, rp, bp, r2, b2);
    set_node(A, X, P1, tunion(bp, b2), rs, bs);
    set_parent(A, rs, X);
    set_parent(A, r2, P1);
    return;
  }
  // four leaves: 3 balanced trees ((a b)(c d)) and 12 chains (((a b) c) d)
  uint32_t code;  // a | b << 2 | c << 4 | d << 6 | chain << 8
  {
    const TBox box[4] = {read_box(A.boxes(k0)), read_box(A.boxes(k0) + 6), read_box(A.boxes(k1)),
                         read_box(A.boxes(k1) + 6)};
    float pa[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = i + 1; j < 4; ++j) pa[i][j] = tarea(tunion(box[i], box[j]));
    constexpr auto pack = [](int a, int b, int c, int d, int chain) -> uint32_t {
      return (uint32_t)(a | (b << 2) | (c << 4) | (d << 6) | (chain << 8));
    };
    // the current tree is balanced with pairs (0 1)(2 3)
    float best = pa[0][1] + pa[2][3];
    code = pack(0, 1, 2, 3, 0);
    auto offer = [&](float cost, uint32_t c) {
      if (cost < best) {
        best = cost;
        code = c;
      }
    };
    offer(pa[0][2] + pa[1][3], pack(0, 2, 1, 3, 0));
    offer(pa[0][3] + pa[1][2], pack(0, 3, 1, 2, 0));
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = i + 1; j < 4; ++j)
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (k != i && k != j)
            offer(pa[i][j] + tarea(tunion(tunion(box[i], box[j]), box[k])), pack(i, j, k, 6 - i - j - k, 1));
    if (code == pack(0, 1, 2, 3, 0)) return;  // already the best
  }
  // the chosen order's leaves, read again where they lie (indexing the arrays
  // above would put them in scratch memory)
  int r[4];
  TBox b[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int k = (int)((code >> (2 * q)) & 3u), in = k < 2 ? k0 : k1;
    r[q] = A.kids(in)[k & 1];
    b[q] = read_box(A.boxes(in) + 6 * (k & 1));
  }
  const TBox ab = tunion(b[0], b[1]);
  if (code < 256u) {
    const TBox cd = tunion(b[2], b[3]);
    set_node(A, k0, r[0], b[0], r[1], b[1]);
    set_node(A, k1, r[2], b[2], r[3], b[3]);
    set_node(A, X, k0, ab, k1, cd);
    set_parent(A, r[0], k0);
    set_parent(A, r[1], k0);
    set_parent(A, r[2], k1);
    set_parent(A, r[3], k1);
  } else {
    const TBox abc = tunion(ab, b[2]);
    set_node(A, k1, r[0], b[0], r[1], b[1]);
    set_node(A, k0, k1, ab, r[2], b[2]);
    set_node(A, X, k0, abc, r[3], b[3]);
    A.set_up(k1, k0);
    set_parent(A, r[0], k1);
    set_parent(A, r[1], k1);
    set_parent(A, r[2], k0);
    set_parent(A, r[3], X);
  }
}

// ------------------------------------------------------------------ box fit and treelets, a tile at a time
// A block takes TILE consecutive sorted triangles and every binary node whose
// range lies among them (a "local" node: all but a percent or two).  Their boxes are
// fitted bottom-up and their treelets restructured in LDS, where a step up the
// tree or a pass costs tens of cycles; through device memory the same work was
// one atomic round trip across the chip per level and two launches per pass
// (fit and four passes: 145 us at 102,400 faces, 1.9 ms at 2 M; this kernel with
// k_top_*: 79 and 420 us).  Threads that come out of the tile's local subtrees carry on
// up the nodes that span tiles: a child writes its box into its slot of the
// parent and counts itself in; the second to arrive reads the first one's box and
// goes on.  Both move the boxes with relaxed agent-scope atomics, which are
// coherent across the chip, and a wait for their completion orders them before the
// arrival increment, so no device-wide fence is needed.
constexpr int TILE = 512;  // 32 KB of LDS, one node per thread

struct TileNodes {
  float box[TILE][12];
  int2 kids[TILE];
  int32_t up[TILE];       // parent if it is local too, else -2 - parent
  int32_t arrived[TILE];  // children fitted; -1: not a local node
  uint16_t list[TILE];    // the pass's treelet roots
  int32_t listed[2];      // how many (passes alternate)
};

struct LdsNodes {
  TileNodes* t;
  int base;
  __device__ __forceinline__ int* kids(int i) const { return (int*)&t->kids[i - base]; }
  __device__ __forceinline__ float* boxes(int i) const { return t->box[i - base]; }
  __device__ __forceinline__ void set_up(int i, int parent) const { t->up[i - base] = parent; }
};

// flag[i]: -1 for a local node, else 0 (k_top_parity then overwrites it).
// WAVES per SIMD: a grid of many tiles a CU gains more from a third and fourth
// resident block (8: 64 registers, some spilled) than it loses (2 M faces 449 ->
// 351 us); with a tile or two a CU it only loses (102,400 faces 56 -> 66 us).
constexpr int TILE_CROWD = 512;  // tiles from which 8 waves a SIMD are taken: two per CU
template <int WAVES>
__global__ void __launch_bounds__(TILE, WAVES) k_tile(const float* V, const int32_t* F, int32_t nv, const int32_t* sorted,
                                               int n, const int4* topo, const int32_t* leaf_parent,
                                               BvhNode* nodes, int32_t* arrive, int32_t* flag,
                                               float4* leaves) {
  __shared__ __align__(16) TileNodes T;
  const int n_int = n - 1, base = blockIdx.x * TILE, t = threadIdx.x, i = base + t;
  if (n == 1) {  // no tree: the one leaf (k_wide_write writes them otherwise)
    if (t == 0) {
      const int f = sorted[0];
      const v3 a = load3(V + 3 * vclamp(F[3 * f], nv)), b = load3(V + 3 * vclamp(F[3 * f + 1], nv));
      const v3 c = load3(V + 3 * vclamp(F[3 * f + 2], nv));
      leaves[0] = make_float4(a.x, a.y, a.z, __int_as_float(f));
      leaves[1] = make_float4(b.x, b.y, b.z, 0.f);
      leaves[2] = make_float4(c.x, c.y, c.z, 0.f);
    }
    return;
  }
  auto in_tile = [&](int k) { return (uint32_t)(k - base) < (uint32_t)TILE; };
  // node i is local if its whole range (from i to topo.w) lies in the tile
  const int4 link = i < n_int ? topo[i] : make_int4(0, 0, -1, -1);
  const bool loc = i < n_int && in_tile(link.w);
  T.kids[t] = make_int2(link.x, link.y);
  T.arrived[t] = loc ? 0 : -1;
  if (t < 2) T.listed[t] = 0;
  __syncthreads();
  auto local = [&](int k) { return in_tile(k) && T.arrived[k - base] >= 0; };
  const bool up_local = link.z >= 0 && local(link.z);
  T.up[t] = up_local ? link.z : -2 - link.z;
  // this thread's triangle, and whether its parent is local
  TBox box = {mk3(0.f, 0.f, 0.f), mk3(0.f, 0.f, 0.f)};
  int ref = 0, up = -1;  // up: where the climb goes on, encoded as T.up; -1: nowhere
  if (i < n) {
    const int f = sorted[i];
    const v3 a = load3(V + 3 * vclamp(F[3 * f], nv)), b = load3(V + 3 * vclamp(F[3 * f + 1], nv));
    const v3 c = load3(V + 3 * vclamp(F[3 * f + 2], nv));
    box = {vmin(vmin(a, b), c), vmax(vmax(a, b), c)};
    ref = (int)((uint32_t)i | DT_LEAF_BIT);
    const int p = leaf_parent[i];
    up = local(p) ? p : -2 - p;
  }
  __syncthreads();
  while (up >= 0) {
    const int s = up - base;
    write_box(T.box[s] + (T.kids[s].x == ref ? 0 : 6), box);
    __threadfence_block();
    if (atomicAdd(&T.arrived[s], 1) == 0) {
      up = -1;
      break;
    }
    __threadfence_block();
    box = tunion(read_box(T.box[s]), read_box(T.box[s] + 6));
    ref = up;
    up = T.up[s];
  }
  __syncthreads();
  for (int pass = 0; pass < TILE_PASSES; ++pass) {
    // the treelet roots: local nodes of one parity of the depth below their
    // subtree's root that are not a pair of triangles, about a third of the
    // nodes, listed so that full waves work on them
    int d = 0;
    if (loc)
      for (int k = T.up[t]; k >= 0 && d < TILE; k = T.up[k - base]) ++d;
    const bool act = loc && (d & 1) == (pass & 1) && ((uint32_t)(T.kids[t].x & T.kids[t].y) & DT_LEAF_BIT) == 0u;
    const uint64_t m = __ballot(act);
    int at = 0;
    if ((t & 63) == 0 && m) at = atomicAdd(&T.listed[pass & 1], __popcll(m));
    at = __shfl(at, 0);
    if (act) T.list[at + __popcll(m & ((1ull << (t & 63)) - 1ull))] = (uint16_t)t;
    __syncthreads();
    if (t < T.listed[pass & 1]) treelet_root(LdsNodes{&T, base}, base + (int)T.list[t]);
    if (t == 0) T.listed[1 - (pass & 1)] = 0;
    __syncthreads();
  }
  // local nodes whole; of the others the links (their boxes come from below)
  if (i < n_int) {
    const int z = T.up[t];
    nodes[i].d = make_int4(T.kids[t].x, T.kids[t].y, z >= 0 ? z : -2 - z, link.w);
    flag[i] = loc ? -1 : 0;
  }
  for (int c = t; c < 3 * TILE; c += TILE) {
    const int s = c / 3, part = c - 3 * s;
    if (base + s < n_int && T.arrived[s] >= 0)
      ((float4*)&nodes[base + s])[part] = *(const float4*)(T.box[s] + 4 * part);
  }
  // a binary radix tree over 64-bit keys and 31-bit indices is at most 95 deep
  int p = -2 - up;
  for (int guard = 0; guard < 256 && p >= 0 && p < n_int; ++guard) {
    const int4 at = topo[p];
    const int slot = at.x == ref ? 0 : 1;
    unsigned long long* mine = (unsigned long long*)((float*)&nodes[p] + 6 * slot);
    unsigned long long* other = (unsigned long long*)((float*)&nodes[p] + 6 * (1 - slot));
    const float v[6] = {box.lo.x, box.lo.y, box.lo.z, box.hi.x, box.hi.y, box.hi.z};
#pragma unroll
    for (int k = 0; k < 3; ++k)
      __hip_atomic_store(mine + k, (unsigned long long)__float_as_uint(v[2 * k]) |
                                       ((unsigned long long)__float_as_uint(v[2 * k + 1]) << 32),
                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the box is out before the arrival below
    if (__hip_atomic_fetch_add(&arrive[p], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0) break;
    float w[6];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const unsigned long long x = __hip_atomic_load(other + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      w[2 * k] = __uint_as_float((uint32_t)x);
      w[2 * k + 1] = __uint_as_float((uint32_t)(x >> 32));
    }
    box = tunion(box, read_box(w));
    ref = p;
    p = at.z;
  }
}

// Treelet passes over the nodes that span tiles (flag >= 0), whose treelets
// reach into the local subtrees' tops: the depth parity (root = 0) by a walk to
// the root, then the restructuring of one parity's treelets
__global__ void k_top_parity(int32_t n_int, const BvhNode* nodes, int32_t* flag) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_int || flag[i] < 0) return;
  int dep = 0, p = i;
  while (p > 0 && p < n_int && dep < 4096) {
    p = nodes[p].d.z;
    ++dep;
  }
  flag[i] = dep & 1;
}

__global__ void k_top_treelet(int32_t n_int, BvhNode* nodes, const int32_t* flag, int parity) {
  const int X = blockIdx.x * blockDim.x + threadIdx.x;
  if (X >= n_int || flag[X] != parity) return;
  treelet_root(GlobalNodes{nodes}, X);
}

// Exponent e of the quantization step 2^e of one axis of a node box [lo, hi]:
// 254 steps must span the box (with the origin rounded down to a multiple of
// the step, 255 then reach past hi), and every p + q 2^e, q in [0, 255], must be
// exact in FP32, which holds once 2^(e+22) >= max(|lo|, |hi|).
__device__ __forceinline__ int quant_exponent(float lo, float hi) {
  float m = fmaxf(fabsf(lo), fabsf(hi));
  int e = -126;
  if (m > 0.f) {
    int em = ilogbf(m) + 1 - 22;  // 2^(ilogb + 1) > m
    e = em > e ? em : e;
  }
  float ext = hi - lo;
  if (ext > 0.f) {
    int ee = ilogbf(ext / 254.0f) + 1;  // 2^ee > ext / 254
    e = ee > e ? ee : e;
  }
  // make sure the span fits (the rounded-down origin costs up to one step);
  // p + 255 s is exact, so the comparison is too
  while (e < 127 && floorf(ldexpf(lo, -e)) * ldexpf(1.0f, e) + 255.0f * ldexpf(1.0f, e) < hi) ++e;
  return e;
}

// ------------------------------------------------------------------ 6-wide traversal tree
// Which binary nodes become 6-wide nodes depends on the path from the root
// (a wide node's internal children do), but the children a binary node would
// have as a wide node depend on its own subtree alone.  So k_cut finds every
// binary node's six children at once (its "cut"), and tells each internal one
// from which distance up it belongs to a cut; k_wide_roots then settles by a walk
// to the root which nodes are reached.  A level-by-level pass from the root would
// visit fewer nodes but needs a launch per level.
constexpr int CUT_T = 256;

__device__ __forceinline__ bool better_area(float a, float best) { return !(a <= best); }  // NaN counts as largest

// cut[6 n ..]: node n's children as a wide node, in the order the wide node
// stores them (ascending box centre along `axis`; unused slots DT_NO_CHILD).
// member[c] bit d (1..5): c belongs to the cut of its d-th ancestor; bits 8-9:
// c's own cut's axis.
__global__ void __launch_bounds__(CUT_T) k_cut(int32_t n_int, const BvhNode* nodes, uint32_t* cut, int32_t* member) {
  const int i = blockIdx.x * CUT_T + threadIdx.x;
  if (i >= n_int) return;
  uint32_t c[DT_WIDE];
  TBox b[DT_WIDE];
  int dist[DT_WIDE];
  {
    const BvhNode n = nodes[i];
    c[0] = (uint32_t)n.d.x;
    c[1] = (uint32_t)n.d.y;
    b[0] = get_box(n, 0);
    b[1] = get_box(n, 1);
    dist[0] = dist[1] = 1;
  }
#pragma unroll
  for (int k = 2; k < DT_WIDE; ++k) {
    c[k] = DT_NO_CHILD;
    b[k] = {mk3(0.f, 0.f, 0.f), mk3(0.f, 0.f, 0.f)};
    dist[k] = 0;
  }
  int cnt = 2;
#pragma unroll
  for (int step = 0; step < DT_WIDE - 2; ++step) {
    // the internal child of largest area is replaced by its two children
    int bi = -1, bd = 0;
    uint32_t bc = 0u;
    float best = -1.f;
#pragma unroll
    for (int k = 0; k < step + 2; ++k) {
      if (c[k] & DT_LEAF_BIT) continue;
      const float a = tarea(b[k]);
      if (better_area(a, best)) {
        best = a;
        bi = k;
        bc = c[k];
        bd = dist[k];
      }
    }
    if (bi < 0 || bc >= (uint32_t)n_int) break;
    const BvhNode n = nodes[bc];
    const TBox b0 = get_box(n, 0);
#pragma unroll
    for (int k = 0; k < step + 2; ++k)
      if (k == bi) {
        c[k] = (uint32_t)n.d.x;
        b[k] = b0;
        dist[k] = bd + 1;
      }
    c[step + 2] = (uint32_t)n.d.y;
    b[step + 2] = get_box(n, 1);
    dist[step + 2] = bd + 1;
    cnt = step + 3;
  }
  // the axis the (doubled) box centres spread most along
  v3 mean = mk3(0.f, 0.f, 0.f), sq = mean;
#pragma unroll
  for (int k = 0; k < DT_WIDE; ++k)
    if (k < cnt) {
      const v3 m = b[k].lo + b[k].hi;
      mean += m;
      sq += mk3(m.x * m.x, m.y * m.y, m.z * m.z);
    }
  const float f = 1.f / (float)cnt;
  const v3 var = mk3(sq.x - mean.x * mean.x * f, sq.y - mean.y * mean.y * f, sq.z - mean.z * mean.z * f);
  const int axis = var.x >= var.y ? (var.x >= var.z ? 0 : 2) : (var.y >= var.z ? 1 : 2);
  int key[DT_WIDE];
#pragma unroll
  for (int k = 0; k < DT_WIDE; ++k) key[k] = fenc(comp(b[k].lo, axis) + comp(b[k].hi, axis));
#pragma unroll
  for (int k = 0; k < DT_WIDE; ++k) {
    int rank = k;  // unused slots stay last
    if (k < cnt) {
      rank = 0;
#pragma unroll
      for (int j = 0; j < DT_WIDE; ++j)
        if (j < cnt && j != k) rank += key[j] < key[k] || (key[j] == key[k] && j < k) ? 1 : 0;
      if (!(c[k] & DT_LEAF_BIT) && c[k] < (uint32_t)n_int) atomicOr(&member[c[k]], 1 << dist[k]);
    }
    cut[(size_t)DT_WIDE * i + rank] = c[k];
  }
  if (axis) atomicOr(&member[i], axis << 8);
}

__device__ __forceinline__ int block_max(int v) {
  __shared__ int sh[CUT_T / 64];
  for (int s = 32; s > 0; s >>= 1) v = max(v, __shfl_xor(v, s, 64));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  for (int k = 0; k < CUT_T / 64; ++k) v = max(v, sh[k]);
  return v;
}

// cnt[n] = (internal | leaf << 32) children of the wide node n becomes, 0 where
// it becomes none.  Node n does if it is the root or belongs to the cut of an
// ancestor that does; walking up, bit h of w says "n is one if the ancestor h
// levels above the current one is".  Also the binary tree's height (root = 1).
__global__ void __launch_bounds__(CUT_T) k_wide_roots(int32_t n_int, const BvhNode* nodes, const uint32_t* cut,
                                                      const int32_t* member, unsigned long long* cnt,
                                                      BvhHeader* hdr) {
  const int i = blockIdx.x * CUT_T + threadIdx.x;
  int dep = 0;
  if (i < n_int) {
    uint32_t w = 1u;
    int p = i;
    while (p > 0 && p < n_int && dep < 4096) {
      if (w & 1u) w |= (uint32_t)member[p] & 0x3Eu;
      w >>= 1;
      p = nodes[p].d.z;
      ++dep;
    }
    unsigned long long v = 0ull;
    if (w & 1u) {
      uint32_t ni = 0, nl = 0;
#pragma unroll
      for (int k = 0; k < DT_WIDE; ++k) {
        const uint32_t r = cut[(size_t)DT_WIDE * i + k];
        if (r == DT_NO_CHILD) continue;
        ni += (r & DT_LEAF_BIT) ? 0u : 1u;
        nl += (r & DT_LEAF_BIT) ? 1u : 0u;
      }
      v = (unsigned long long)ni | ((unsigned long long)nl << 32);
    }
    cnt[i] = v;
    dep += 2;  // the deepest internal node has a leaf child one level below it
  }
  dep = block_max(dep);
  if (threadIdx.x == 0) atomicMax(&hdr->depth, dep);
}

// owner[w]: the binary node of wide node w.  The root is wide node 0; the
// internal children of binary node i's wide node are 1 + pre[i] (low) onwards
__global__ void k_wide_owner(int32_t n_int, const uint32_t* cut, const unsigned long long* cnt,
                             const unsigned long long* pre, int32_t* owner, int32_t cap) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_int || cnt[i] == 0ull) return;
  if (i == 0) owner[0] = 0;
  uint32_t at = 1u + (uint32_t)pre[i];
#pragma unroll
  for (int k = 0; k < DT_WIDE; ++k) {
    const uint32_t r = cut[(size_t)DT_WIDE * i + k];
    if (r & DT_LEAF_BIT) continue;  // DT_NO_CHILD has the bit too
    if (at < (uint32_t)cap) owner[at] = (int32_t)r;
    ++at;
  }
}

// Writes wide node w and its leaves: a group of 8 lanes per node, one child
// each (a node per lane leaves most of the chip waiting for one lane's chain
// of child loads).  total: the scan's grand total (low: wide nodes but the
// root).
__global__ void __launch_bounds__(CUT_T) k_wide_write(const float* V, const int32_t* F, int32_t nv, int32_t nf,
                                                      const int32_t* sorted, const BvhNode* nodes,
                                                      const uint32_t* cut, const int32_t* member,
                                                      const unsigned long long* pre,
                                                      const unsigned long long* total, const int32_t* owner,
                                                      WideNode* out, int32_t cap, float4* leaves) {
  const int n_int = nf - 1;
  const uint32_t count = min(1u + (uint32_t)*total, (uint32_t)cap);
  const uint32_t w = (uint32_t)((blockIdx.x * (int64_t)CUT_T + threadIdx.x) >> 3);
  const int sub = threadIdx.x & 7, lane = threadIdx.x & 63;
  const bool live = w < count;
  int n = live ? owner[w] : 0;
  n = n < 0 || n >= n_int ? 0 : n;
  const uint32_t ref = live && sub < DT_WIDE ? cut[(size_t)DT_WIDE * n + sub] : DT_NO_CHILD;
  const bool valid = ref != DT_NO_CHILD;
  const bool is_leaf = valid && (ref & DT_LEAF_BIT) != 0u, is_int = valid && !is_leaf;
  const uint32_t im = (uint32_t)(__ballot(is_int) >> (lane & ~7)) & 0x3Fu;
  const uint32_t lmask = (uint32_t)(__ballot(is_leaf) >> (lane & ~7)) & 0x3Fu;
  const unsigned long long base = live ? pre[n] : 0ull;
  const uint32_t child_base = 1u + (uint32_t)base, leaf_base = (uint32_t)(base >> 32);
  TBox box = {mk3(INFINITY, INFINITY, INFINITY), mk3(-INFINITY, -INFINITY, -INFINITY)};
  if (is_leaf) {
    const uint32_t j = min(ref & ~DT_LEAF_BIT, (uint32_t)(nf - 1));
    const int f = sorted[j];
    const v3 a = load3(V + 3 * vclamp(F[3 * f], nv)), b = load3(V + 3 * vclamp(F[3 * f + 1], nv));
    const v3 c = load3(V + 3 * vclamp(F[3 * f + 2], nv));
    box = {vmin(vmin(a, b), c), vmax(vmax(a, b), c)};
    const size_t q = leaf_base + (uint32_t)__popc(lmask & ((1u << sub) - 1u));
    if (q < (size_t)nf) {
      leaves[3 * q] = make_float4(a.x, a.y, a.z, __int_as_float(f));
      leaves[3 * q + 1] = make_float4(b.x, b.y, b.z, 0.f);
      leaves[3 * q + 2] = make_float4(c.x, c.y, c.z, 0.f);
    }
  } else if (is_int && ref < (uint32_t)n_int) {
    const BvhNode m = nodes[ref];
    box = tunion(get_box(m, 0), get_box(m, 1));
  }
  float org[3];
  uint32_t ebits = 0, qlo[3], qhi[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float lo = comp(box.lo, a), hi = comp(box.hi, a);
    float nlo = lo, nhi = hi;
#pragma unroll
    for (int s = 1; s < 8; s <<= 1) {
      nlo = fminf(nlo, __shfl_xor(nlo, s));
      nhi = fmaxf(nhi, __shfl_xor(nhi, s));
    }
    const int e = quant_exponent(nlo, nhi);
    const float sc = ldexpf(1.0f, e);
    const float p = floorf(ldexpf(nlo, -e)) * sc;  // a multiple of sc, <= nlo
    org[a] = p;
    ebits |= (uint32_t)(uint8_t)(int8_t)e << (8 * a);
    int ql = 255, qh = 0;  // an unused slot's box is inverted: never entered
    if (valid) {
      ql = (int)floorf(ldexpf(lo - p, -e));
      ql = ql < 0 ? 0 : (ql > 255 ? 255 : ql);
      while (ql > 0 && p + (float)ql * sc > lo) --ql;
      qh = (int)ceilf(ldexpf(hi - p, -e));
      qh = qh < 0 ? 0 : (qh > 255 ? 255 : qh);
      while (qh < 255 && p + (float)qh * sc < hi) ++qh;
    }
    qlo[a] = (uint32_t)ql;
    qhi[a] = (uint32_t)qh;
  }
  // the packed step words: children 0-3 one byte each, 4 and 5 with both bounds
  uint32_t lo4[3], hi4[3], q45[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    lo4[a] = sub < 4 ? qlo[a] << (8 * sub) : 0u;
    hi4[a] = sub < 4 ? qhi[a] << (8 * sub) : 0u;
    q45[a] = sub == 4 || sub == 5 ? (qlo[a] << (8 * (sub - 4))) | (qhi[a] << (8 * (sub - 2))) : 0u;
#pragma unroll
    for (int s = 1; s < 8; s <<= 1) {
      lo4[a] |= (uint32_t)__shfl_xor((int)lo4[a], s);
      hi4[a] |= (uint32_t)__shfl_xor((int)hi4[a], s);
      q45[a] |= (uint32_t)__shfl_xor((int)q45[a], s);
    }
  }
  if (!live || sub > 3) return;
  const uint32_t axis = ((uint32_t)member[n] >> 8) & 3u;
  uint4 v = make_uint4(__float_as_uint(org[0]), __float_as_uint(org[1]), __float_as_uint(org[2]),
                       ebits | (im << 24) | (axis << 30));
  if (sub == 1) v = make_uint4((child_base & DT_WIDE_INDEX) | (lmask << 26), leaf_base, lo4[0], hi4[0]);
  if (sub == 2) v = make_uint4(lo4[1], hi4[1], lo4[2], hi4[2]);
  if (sub == 3) v = make_uint4(q45[0], q45[1], q45[2], 0u);
  ((uint4*)(out + w))[sub] = v;
}

__global__ void k_copy_vn(const float4* vn, int32_t nv, float* N) {
  int v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= nv) return;
  float4 a = vn[v];
  N[3 * v] = a.x;
  N[3 * v + 1] = a.y;
  N[3 * v + 2] = a.z;
}

struct BuildWs {
  uint64_t *k0, *k1;
  int32_t *v0, *v1;
  int32_t* hist;
  int32_t* scanp;
  float* bpart;
  int32_t* arrive;
  int* acc;
  int32_t *flag, *member;
  int32_t* vcnt;
};

int rs_tiles(int32_t nf, int items) { return (int)((nf + RS_T * items - 1) / (RS_T * items)); }

size_t carve_build(Carver& c, int32_t nv, int32_t nf, BuildWs* w) {
  int nt = rs_tiles(nf, RS_ITEMS);
  BuildWs x;
  x.k0 = c.take<uint64_t>(nf);
  x.k1 = c.take<uint64_t>(nf);
  x.v0 = c.take<int32_t>(nf);
  x.v1 = c.take<int32_t>(nf);
  x.hist = c.take<int32_t>((size_t)256 * nt);
  x.scanp = c.take<int32_t>(SCAN_NB + 1);
  x.bpart = c.take<float>(NBB * 6);
  x.arrive = c.take<int32_t>(nf > 1 ? nf - 1 : 1);
  x.acc = c.take<int>(6 * (size_t)(nf > 1 ? nf - 1 : 1));
  x.flag = c.take<int32_t>(nf);
  x.member = c.take<int32_t>(nf);
  x.vcnt = c.take<int32_t>(nv);
  c.take<int32_t>(nv);  // spare: the workspace a mesh needs decides what dt_build_bvh_noalloc takes
  if (w) *w = x;
  return c.used();
}

}  // namespace

// ------------------------------------------------------------------ scan
// out[0..n) = exclusive prefix sums of in[0..n); partials[SCAN_NB] = total,
// also to *total if given.  in == out is allowed.
template <class T>
static dt_status scan_exclusive(const T* in, T* out, int32_t n, T* partials, T* total, hipStream_t s) {
  if (n <= 0) return DT_OK;
  if (n <= SCAN_ONE_MAX) {
    hipLaunchKernelGGL(k_scan_one<T>, dim3(1), dim3(SCAN_ONE_T), 0, s, in, out, n, partials, total);
    DT_CHECK_LAUNCH();
    return DT_OK;
  }
  int32_t chunk = (n + SCAN_NB - 1) / SCAN_NB;
  hipLaunchKernelGGL(k_scan_reduce<T>, dim3(SCAN_NB), dim3(SCAN_T), 0, s, in, n, chunk, partials);
  hipLaunchKernelGGL(k_scan_partials<T>, dim3(1), dim3(SCAN_NB), 0, s, partials, SCAN_NB, total);
  hipLaunchKernelGGL(k_scan_apply<T>, dim3(SCAN_NB), dim3(SCAN_T), 0, s, in, out, n, chunk, partials);
  DT_CHECK_LAUNCH();
  return DT_OK;
}

// stable LSD radix sort of (Morton key, face) in passes of 8 bits, then the
// binary radix tree over the sorted keys; *order: the sorted faces
template <class K, int ITEMS>
static dt_status sort_and_link(const float* V, const int32_t* F, int32_t nf, int32_t nv, int drop, const BuildWs& w,
                               int32_t* hist, BvhHeader* hdr, int4* topo, int32_t* lpar, int32_t** order,
                               hipStream_t s) {
  K *ki = (K*)w.k0, *ko = (K*)w.k1;
  int32_t *vi = w.v0, *vo = w.v1;
  const int nt = rs_tiles(nf, ITEMS);
  hipLaunchKernelGGL(k_morton<K>, dim3(dt_blocks(nf, NBB)), dim3(NBB), 0, s, V, F, nf, nv, drop, w.bpart, hdr, ki, vi);
  for (int shift = 0; shift < 8 * (int)sizeof(K); shift += 8) {
    constexpr bool SELF = ITEMS < RS_ITEMS;
    hipLaunchKernelGGL((k_rs_hist<K, ITEMS, SELF>), dim3(nt), dim3(RS_T), 0, s, ki, nf, shift, hist, nt);
    if (!SELF)
      if (dt_status st = scan_exclusive(hist, hist, 256 * nt, w.scanp, (int32_t*)nullptr, s)) return st;
    hipLaunchKernelGGL((k_rs_scatter<K, ITEMS, SELF>), dim3(nt), dim3(RS_T), 0, s, ki, vi, ko, vo, nf, shift, hist, nt);
    DT_CHECK_LAUNCH();
    K* tk = ki;
    ki = ko;
    ko = tk;
    int32_t* tv = vi;
    vi = vo;
    vo = tv;
  }
  if (nf > 1)
    hipLaunchKernelGGL(k_karras<K>, dim3(dt_blocks(nf - 1, 256)), dim3(256), 0, s, ki, nf, topo, lpar, w.arrive,
                       w.member);
  DT_CHECK_LAUNCH();
  *order = vi;
  return DT_OK;
}

// ------------------------------------------------------------------ C ABI
extern "C" dt_status dt_bvh_bytes(int32_t nv, int32_t nf, size_t* bvh_bytes, size_t* ws_bytes) {
  DT_REQUIRE(nv >= 3 && nf >= 1, "dt_bvh_bytes: need nv >= 3 and nf >= 1 (got %d, %d)", nv, nf);
  DT_REQUIRE(nf <= DT_MAX_FACES && nv < (1 << 30), "dt_bvh_bytes: mesh too large (at most 2^26 triangles)");
  DT_REQUIRE(bvh_bytes && ws_bytes, "dt_bvh_bytes: null output pointer");
  *bvh_bytes = bvh_layout(nv, nf).total;
  Carver c(nullptr, 0);
  *ws_bytes = carve_build(c, nv, nf, nullptr);
  return DT_OK;
}

extern "C" dt_status dt_build_bvh(const float* V, int32_t nv, const int32_t* F, int32_t nf,
                                  void* bvh, size_t bvh_bytes, void* ws, size_t ws_bytes,
                                  void* stream) {
  DT_REQUIRE(V && F && bvh && ws, "dt_build_bvh: null pointer argument");
  DT_REQUIRE(nv >= 3 && nf >= 1, "dt_build_bvh: need nv >= 3 and nf >= 1 (got %d, %d)", nv, nf);
  DT_REQUIRE(nf <= DT_MAX_FACES && nv < (1 << 30), "dt_build_bvh: mesh too large (at most 2^26 triangles)");
  BvhLayout L = bvh_layout(nv, nf);
  if (bvh_bytes < L.total) {
    dt_set_error("dt_build_bvh: bvh blob has %zu bytes, needs %zu", bvh_bytes, L.total);
    return DT_ERR_WORKSPACE_TOO_SMALL;
  }
  Carver c(ws, ws_bytes);
  BuildWs w;
  carve_build(c, nv, nf, &w);
  if (c.overflow) {
    dt_set_error("dt_build_bvh: workspace has %zu bytes, needs %zu", ws_bytes, c.used());
    return DT_ERR_WORKSPACE_TOO_SMALL;
  }
  hipStream_t s = (hipStream_t)stream;
  char* b = (char*)bvh;
  BvhHeader* hdr = (BvhHeader*)(b + L.header);
  BvhNode* nodes = (BvhNode*)(b + L.nodes);
  float4* leaves = (float4*)(b + L.leaves);
  float4* vn = (float4*)(b + L.vnormals);
  float4* fn = (float4*)(b + L.fnormals);
  int32_t* off = (int32_t*)(b + L.csr_off);
  int32_t* idx = (int32_t*)(b + L.csr_idx);
  int32_t* lpar = (int32_t*)(b + L.leaf_parent);

  // normals (Eq. 12-13).  The corner ranks sit in the sort's key buffers
  int32_t* rank = (int32_t*)w.k0;
  hipLaunchKernelGGL(k_build_init, dim3(dt_blocks(nv, 256)), dim3(256), 0, s, hdr, nv, nf, w.vcnt);
  hipLaunchKernelGGL(k_faces, dim3(dt_blocks(nf, 256)), dim3(256), 0, s, V, F, nf, nv, fn, w.vcnt, rank);
  if (dt_status st = scan_exclusive(w.vcnt, off, nv, w.scanp, off + nv, s)) return st;
  hipLaunchKernelGGL(k_vfill, dim3(dt_blocks(nf, 256)), dim3(256), 0, s, F, nf, nv, off, rank, idx);
  hipLaunchKernelGGL(k_vnormals, dim3(dt_blocks(nv, 256)), dim3(256), 0, s, off, idx, fn, nv, vn);
  DT_CHECK_LAUNCH();
  // Morton order and the binary tree.  Up to 2^20 triangles the top 32 bits of
  // the code (2,048 cells an axis) order them finely enough (ties fall back to
  // the face index) and halve the sort.  Above, an even mesh's tree has the same
  // node visits with 32 bits and is built sooner (2 M faces 1.57 against 1.86 ms),
  // but one whose detail fills a small part of its box shares cells: with a piece
  // 10^4 units away, two views of 1.2 M faces take 8.1 ms with 32 bits, 1.9 with 63
  hipLaunchKernelGGL(k_bounds, dim3(NBB), dim3(256), 0, s, V, F, nf, nv, w.bpart);
  int32_t* vi = nullptr;
  int4* topo = (int4*)w.acc;
  dt_status st;
  if (nf >= 1024 && nf <= (1 << 17)) {
    // smaller tiles (with eight keys a thread a 102,400-key pass has 50 blocks
    // for 256 CUs) and few enough of them for every block to add up their
    // histograms: a pass 27 -> 17 us.  The histogram, a word per four keys, sits
    // where the links go afterwards
    st = sort_and_link<uint32_t, 4>(V, F, nf, nv, 31, w, (int32_t*)w.acc, hdr, topo, lpar, &vi, s);
  } else if (nf <= (1 << 20)) {
    st = sort_and_link<uint32_t, RS_ITEMS>(V, F, nf, nv, 31, w, w.hist, hdr, topo, lpar, &vi, s);
  } else {
    st = sort_and_link<uint64_t, RS_ITEMS>(V, F, nf, nv, 0, w, w.hist, hdr, topo, lpar, &vi, s);
  }
  if (st != DT_OK) return st;
  // boxes, and treelets restructured
  const unsigned tiles = dt_blocks(nf, TILE);
  if (tiles >= TILE_CROWD)
    hipLaunchKernelGGL(k_tile<8>, dim3(tiles), dim3(TILE), 0, s, V, F, nv, vi, nf, topo, lpar, nodes, w.arrive,
                       w.flag, leaves);
  else
    hipLaunchKernelGGL(k_tile<4>, dim3(tiles), dim3(TILE), 0, s, V, F, nv, vi, nf, topo, lpar, nodes, w.arrive,
                       w.flag, leaves);
  if (nf > TILE) {
    for (int pass = 0; pass < TOP_PASSES; ++pass) {
      hipLaunchKernelGGL(k_top_parity, dim3(dt_blocks(nf - 1, 256)), dim3(256), 0, s, nf - 1, nodes, w.flag);
      hipLaunchKernelGGL(k_top_treelet, dim3(dt_blocks(nf - 1, 256)), dim3(256), 0, s, nf - 1, nodes, w.flag,
                         pass & 1);
    }
  }
  DT_CHECK_LAUNCH();
  // 6-wide traversal tree.  The links, the sort's key buffers and the parity flags
  // are free by now and hold the cuts, the child counts with
  // their prefix sums, and the wide nodes' owners
  if (nf > 1) {
    uint32_t* cut = (uint32_t*)w.acc;
    unsigned long long *cnt = (unsigned long long*)w.k0, *pre = (unsigned long long*)w.k1;
    unsigned long long* part = (unsigned long long*)w.bpart;  // SCAN_NB + 1 sums
    static_assert(NBB * 6 * sizeof(float) >= (SCAN_NB + 1) * sizeof(unsigned long long), "scan partials");
    const int32_t cap = wide_cap(nf);
    const unsigned nb = dt_blocks(nf - 1, CUT_T);
    hipLaunchKernelGGL(k_cut, dim3(nb), dim3(CUT_T), 0, s, nf - 1, nodes, cut, w.member);
    hipLaunchKernelGGL(k_wide_roots, dim3(nb), dim3(CUT_T), 0, s, nf - 1, nodes, cut, w.member, cnt, hdr);
    if (dt_status st = scan_exclusive(cnt, pre, nf - 1, part, (unsigned long long*)nullptr, s)) return st;
    hipLaunchKernelGGL(k_wide_owner, dim3(nb), dim3(CUT_T), 0, s, nf - 1, cut, cnt, pre, w.flag, cap);
    hipLaunchKernelGGL(k_wide_write, dim3(dt_blocks(8 * (int64_t)cap, CUT_T)), dim3(CUT_T), 0, s, V, F, nv, nf, vi,
                       nodes, cut, w.member, pre, part + SCAN_NB, w.flag, (WideNode*)(b + L.wide), cap, leaves);
    DT_CHECK_LAUNCH();
  }
  return DT_OK;
}

// ------------------------------------------------------------------ build without allocation
// Build workspace held by the library itself, for callers that cannot
// allocate device memory.  Every GPU the library runs on holds its own copy
// from module load until the process ends.  In host code `scratch` only names
// the array: its device address is looked up once per device and kept in
// g_scratch_ptr, which is what the kernels are given.
static __device__ __align__(256) unsigned char scratch[DT_BVH_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

dt_status scratch_address(void** out) {
  int dev = -1;
  DT_CHECK_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) {
    dt_set_error("dt_build_bvh_noalloc: device ordinal %d out of range", dev);
    return DT_ERR_UNSUPPORTED;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    // with device `dev` current: this device's copy of the array
    DT_CHECK_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return DT_OK;
}
}  // namespace

extern "C" dt_status dt_build_bvh_noalloc(const float* V, int32_t nv, const int32_t* F, int32_t nf,
                                          void* bvh, size_t bvh_bytes, void* stream) {
  DT_REQUIRE(V && F && bvh, "dt_build_bvh_noalloc: null pointer argument");
  DT_REQUIRE(nv >= 3 && nf >= 1, "dt_build_bvh_noalloc: need nv >= 3 and nf >= 1 (got %d, %d)", nv,
             nf);
  DT_REQUIRE(nf <= DT_MAX_FACES && nv < (1 << 30),
             "dt_build_bvh_noalloc: mesh too large (at most 2^26 triangles)");
  Carver c(nullptr, 0);
  const size_t need = carve_build(c, nv, nf, nullptr);
  if (need > (size_t)DT_BVH_SCRATCH_BYTES) {
    dt_set_error("dt_build_bvh_noalloc: a mesh of %d vertices and %d faces needs %zu bytes of "
                 "build workspace, more than the library's %zu (use dt_build_bvh with a "
                 "caller-owned workspace)", nv, nf, need, (size_t)DT_BVH_SCRATCH_BYTES);
    return DT_ERR_CAPACITY;
  }
  void* ws = nullptr;
  if (dt_status st = scratch_address(&ws)) return st;
  return dt_build_bvh(V, nv, F, nf, bvh, bvh_bytes, ws, (size_t)DT_BVH_SCRATCH_BYTES, stream);
}

extern "C" dt_status dt_bvh_vertex_normals(const void* bvh, int32_t nv, int32_t nf, float* N,
                                           void* stream) {
  DT_REQUIRE(bvh && N, "dt_bvh_vertex_normals: null pointer argument");
  DT_REQUIRE(nv >= 3 && nf >= 1, "dt_bvh_vertex_normals: need nv >= 3 and nf >= 1");
  BvhView v = bvh_view(bvh, nv, nf);
  hipLaunchKernelGGL(k_copy_vn, dim3(dt_blocks(nv, 256)), dim3(256), 0, (hipStream_t)stream, v.vn, nv,
                     N);
  DT_CHECK_LAUNCH();
  return DT_OK;
}
