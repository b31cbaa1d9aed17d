// Silhouette (mask) term: each pixel's coverage by the object and the
// gradient of a loss on it with respect to the vertices through the motion of
// the object's outline (the visibility gradient that the interior derivatives
// of the tracer do not carry; the paper's mask loss, Sec. 3.1 "Mask-based
// Geometry Initialization" and the appendix on the ray tracer's mesh
// regularization).
//
// The mask of pixel p is the fraction of its unit square (pixel (x, y) covers
// [x, x+1) x [y, y+1) in continuous image coordinates) covered by the
// object's projection.  Its value is taken at the pixel centre; its
// derivative is the boundary integral of the outline's normal velocity over
// the part of the outline inside p.  The outline is made of silhouette edges
// (one adjacent face facing the eye and the other not, or an edge with one
// face) at points whose camera line meets no other triangle.  The integral is
// a fixed quadrature: an edge whose projection is l pixels long gets
// n = max(1, ceil(rho l)) points at the midpoints t_k = (k + 1/2) / n of its
// 3D parameter, weight |dx/dt| / n, each added to the pixel containing its
// projection, and a point moves with its two vertices with weights 1 - t_k
// and t_k.
//
// Kernels: k_mask_forward casts the pixel-centre rays, a wave per tile of 64;
// k_mask_facing decides for every face which cameras it faces (in FP64:
// products of FP32 inputs are exact, so the decision matches an FP64
// evaluation); k_mask_grad finds the silhouette edges (an edge is taken by the
// face holding it as (a, b) with a < b, or by its only face; its other face is
// found in the blob's vertex-to-face lists), spreads their quadrature points
// over the lanes, casts them with the tracer's wave traversal and adds the
// visible ones' FP32 terms to dV atomically.
#include "dt_queue.h"

namespace {

constexpr int MT = 256;

struct MaskCams {
  CamDev c[DT_MASK_MAX_CAMERAS];
  int n;
};

__device__ __forceinline__ v3 vtx(const float* V, int i) { return load3(V + 3 * (size_t)i); }

// Ray casts of one wave: whether each active lane's line o + s d, s > t_eps,
// meets any triangle but f1 and f2.  The tracer's wave traversal, stopped at
// a lane's first hit; stack entries past the LDS part go to the lane's private
// memory.  A full stack is reported as a hit (conservative: the point is then
// not counted on the outline) and flagged.
struct MaskLds {
  uint2 stk[DT_STACK_LDS * 64];
  LeafQueue lq;
};

__device__ __forceinline__ bool lines_blocked(const BvhView& bv, bool active, v3 o, v3 d, int f1, int f2,
                                              float t_eps, MaskLds& lds, bool* overflow) {
  uint2 deep[DT_STACK - DT_STACK_LDS];
  const Hit h = closest_hit_wave<DT_STACK_LDS, true, false, true>(
      bv, active, o, d, f1, t_eps, lds.stk + (threadIdx.x & 63u), 64, deep, DT_STACK - DT_STACK_LDS, lds.lq,
      overflow, f2);
  return h.tri >= 0 || *overflow;
}

__device__ __forceinline__ bool front_facing(v3 p0, v3 p1, v3 p2, const float* eye) {
  const double ax = (double)p1.x - p0.x, ay = (double)p1.y - p0.y, az = (double)p1.z - p0.z;
  const double bx = (double)p2.x - p0.x, by = (double)p2.y - p0.y, bz = (double)p2.z - p0.z;
  const double nx = ay * bz - az * by, ny = az * bx - ax * bz, nz = ax * by - ay * bx;
  return nx * ((double)p0.x - eye[0]) + ny * ((double)p0.y - eye[1]) + nz * ((double)p0.z - eye[2]) < 0.0;
}

// facing[f] bit c: face f faces camera c's eye
static_assert(DT_MASK_MAX_CAMERAS <= 16, "one bit per camera in a uint16");
__global__ void __launch_bounds__(MT) k_mask_facing(const float* V, const int32_t* F, int32_t nv, int32_t nf,
                                                    MaskCams cams, uint16_t* facing) {
  const int f = blockIdx.x * MT + threadIdx.x;
  if (f >= nf) return;
  const v3 p0 = vtx(V, vclampi(F[3 * f], nv)), p1 = vtx(V, vclampi(F[3 * f + 1], nv));
  const v3 p2 = vtx(V, vclampi(F[3 * f + 2], nv));
  uint32_t m = 0;
  for (int c = 0; c < cams.n; ++c) m |= front_facing(p0, p1, p2, cams.c[c].eye) ? 1u << c : 0u;
  facing[f] = (uint16_t)m;
}

// continuous image position of X, and the rows of d(xi, yi)/dX; false if X
// is not in front of the camera
__device__ __forceinline__ bool project(const CamDev& c, v3 X, float& xi, float& yi, v3* jx, v3* jy) {
  const v3 w = X - mk3(c.eye[0], c.eye[1], c.eye[2]);
  const v3 f = mk3(c.f[0], c.f[1], c.f[2]), r = mk3(c.r[0], c.r[1], c.r[2]), u = mk3(c.u[0], c.u[1], c.u[2]);
  const float z = dot(w, f);
  if (!(z > 1e-9f)) return false;
  const float a = dot(w, r), b = dot(w, u);
  const float sx = 0.5f * (float)c.W / (c.th * c.aspect), sy = 0.5f * (float)c.H / c.th;
  const float iz = 1.0f / z;
  xi = sx * (a * iz) + 0.5f * (float)c.W;
  yi = 0.5f * (float)c.H - sy * (b * iz);
  if (jx) {
    *jx = (r * iz - f * (a * iz * iz)) * sx;
    *jy = (u * iz - f * (b * iz * iz)) * (-sy);
  }
  return true;
}

// Tiles of 64 pixels, 8 x 8 so that a wave's rays walk the same nodes; narrow
// images take tiles of their own width or height, so that most lanes have a pixel
// (and 64 times the tiles of any image stay below a launch's 2^32 threads)
struct MaskTile {
  int lx, ly;   // log2 of width and height
  int64_t tw, n;
};
__host__ __device__ __forceinline__ int ceil_log2_8(int v) { return v >= 5 ? 3 : (v >= 3 ? 2 : v - 1); }
__host__ __device__ __forceinline__ MaskTile mask_tile(int W, int H) {
  MaskTile t;
  t.lx = W < 8 ? ceil_log2_8(W) : 6 - ceil_log2_8(H);
  t.ly = 6 - t.lx;
  t.tw = ((int64_t)W + (1 << t.lx) - 1) >> t.lx;
  t.n = t.tw * (((int64_t)H + (1 << t.ly) - 1) >> t.ly);
  return t;
}

__global__ void __launch_bounds__(64) k_mask_forward(BvhView bv, MaskCams cams, float t_eps, float* mask) {
  __shared__ MaskLds lds;
  const CamDev& c = cams.c[blockIdx.y];
  const MaskTile t = mask_tile(c.W, c.H);
  const int64_t tile = blockIdx.x;
  if (tile >= t.n) return;
  const int lane = (int)threadIdx.x;
  const int64_t x = (tile % t.tw) * (1 << t.lx) + (lane & ((1 << t.lx) - 1));
  const int64_t y = (tile / t.tw) * (1 << t.ly) + (lane >> t.lx);
  const bool in = x < c.W && y < c.H;
  const float px = (2.0f * ((float)x + 0.5f) / (float)c.W - 1.0f) * c.th * c.aspect;
  const float py = (1.0f - 2.0f * ((float)y + 0.5f) / (float)c.H) * c.th;
  const v3 d = normalize3(mk3(c.f[0], c.f[1], c.f[2]) + mk3(c.r[0], c.r[1], c.r[2]) * px +
                          mk3(c.u[0], c.u[1], c.u[2]) * py);
  bool ovf = false;
  const bool hit = lines_blocked(bv, in, mk3(c.eye[0], c.eye[1], c.eye[2]), d, -1, -1, t_eps, lds, &ovf);
  if (in) mask[c.pixel_offset + y * c.W + x] = hit ? 1.0f : 0.0f;
}

// A silhouette edge of one camera in image space: its vertices a < b, the
// projected direction's outward normal (nx, ny) and its number of quadrature
// points; false if a vertex it needs is not in front of the camera or the
// edge projects to a point.
struct SilEdge {
  int a, b;
  float nx, ny;
  int ns;
};

__device__ __forceinline__ bool silhouette_edge(const float* V, const int32_t* F, int nv, const CamDev& c, int f,
                                                int k, int front, float rho, SilEdge& e) {
  const int p = vclampi(F[3 * f + k], nv), q = vclampi(F[3 * f + (k + 1) % 3], nv);
  e.a = p < q ? p : q;
  e.b = p < q ? q : p;
  float xa, ya, xb, yb, xc, yc;
  if (!project(c, vtx(V, e.a), xa, ya, nullptr, nullptr) || !project(c, vtx(V, e.b), xb, yb, nullptr, nullptr))
    return false;
  const int cv = vclampi(F[3 * front] + F[3 * front + 1] + F[3 * front + 2] - e.a - e.b, nv);
  if (!project(c, vtx(V, cv), xc, yc, nullptr, nullptr)) return false;
  const float ex = xb - xa, ey = yb - ya;
  const float len = sqrtf(ex * ex + ey * ey);
  if (!(len > 0.f)) return false;
  e.nx = -ey / len;
  e.ny = ex / len;
  if (e.nx * (xc - xa) + e.ny * (yc - ya) > 0.f) {
    e.nx = -e.nx;
    e.ny = -e.ny;
  }
  e.ns = max(1, (int)ceilf(rho * len));
  return true;
}

// One wave takes `per` edge slots (slot 3 f + k: face f's edge from its corner k)
// for the cameras of its group (blockIdx.y, every gridDim.y-th camera).
// Silhouette edges are a percent or so of all (edge, camera) pairs of a closed
// mesh and carry the only costly work, so the wave first collects them in LDS and
// then deals their quadrature points to its lanes (a thread per (edge, camera)
// that walked the tree for its own points left one lane in fifty busy: 1,900
// against 243 us for 8 views of 512 x 512 and 102,400 faces).
// counts: [0] outline points in an image where the loss gradient is nonzero,
// [1] of those, points on the outline (visible), [2] stack overflows
// How a call is cut into waves.  On an open mesh every boundary edge is on the
// outline of every camera, and a wave that holds many of them works on them one
// after the other while the chip waits, so up to MASK_SMALL slots a wave takes 64
// and a quarter of the cameras; above, there are waves enough, and 128 slots with
// all cameras look for an edge's other face least often.  8 views of 512 x 512, 256
// slots and all cameras / 64 and a quarter / 128 and all: 20,000 separate
// triangles 28.9 / 3.6 / 16.0 ms (14.0 a thread per edge and camera), an open plane
// of 80,000 faces 639 / 102 / 341 us (173), a torus of 102,400 288 / 243 / 272, of
// 1 M 584 / 1,073 / 592
constexpr int64_t MASK_SMALL = (int64_t)1 << 19;
struct MaskCut {
  int per, groups;
};
MaskCut mask_cut(int64_t slots, int cams) {
  if (slots > MASK_SMALL) return {128, 1};
  return {64, cams < 4 ? cams : 4};
}
constexpr int MASK_ITEMS = 128;  // collected edges per round of points

__global__ void __launch_bounds__(64) k_mask_grad(const float* V, const int32_t* F, int32_t nv, int32_t nf,
                                                  BvhView bv, const uint16_t* facing, MaskCams cams,
                                                  const float* grad_mask, float rho, float* dV,
                                                  unsigned long long* counts, int per) {
  __shared__ MaskLds lds;
  __shared__ int4 item[MASK_ITEMS];                      // slot, other face or -1, camera, front face
  __shared__ unsigned long long first[MASK_ITEMS + 1];   // points before the item
  const int lane = (int)threadIdx.x;
  const uint64_t lt = (1ull << lane) - 1ull;
  uint32_t all = 0u;  // the group's cameras
  for (int c = (int)blockIdx.y; c < cams.n; c += (int)gridDim.y) all |= 1u << c;
  int n_items = 0;                    // wave-uniform
  unsigned long long n_points = 0ull; // wave-uniform
  unsigned n_in = 0, n_vis = 0, n_ovf = 0;

  auto cast_points = [&]() {
    if (lane == 0) first[n_items] = n_points;
    wave_lds_sync();
    for (unsigned long long base = 0; base < n_points; base += 64ull) {
      const unsigned long long pt = base + (unsigned)lane;
      bool active = pt < n_points;
      int lo = 0, hi = n_items;  // first[lo] <= pt < first[hi]
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (first[mid] <= pt) lo = mid; else hi = mid;
      }
      const int4 it = item[lo];
      const int f = it.x / 3, cam = it.z;
      const CamDev& c = cams.c[cam];
      SilEdge e;
      e.a = e.b = 0;
      e.ns = 1;
      active = active && silhouette_edge(V, F, nv, c, f, it.x % 3, it.w, rho, e);
      const v3 eye = mk3(c.eye[0], c.eye[1], c.eye[2]);
      const v3 A = vtx(V, e.a), Bv = vtx(V, e.b);
      const v3 BA = Bv - A;
      const float t = ((float)(int)(pt - first[lo]) + 0.5f) / (float)e.ns;
      const v3 X = A * (1.0f - t) + Bv * t;
      float xi = 0.f, yi = 0.f, g = 0.f;
      v3 jx = mk3(0.f, 0.f, 0.f), jy = jx;
      active = active && project(c, X, xi, yi, &jx, &jy);
      active = active && xi >= 0.f && xi < (float)c.W && yi >= 0.f && yi < (float)c.H;
      if (active) {
        const int px = min((int)floorf(xi), c.W - 1), py = min((int)floorf(yi), c.H - 1);
        g = grad_mask[c.pixel_offset + (int64_t)py * c.W + px];
        active = g != 0.f;
      }
      n_in += active ? 1u : 0u;
      bool ovf = false;
      // the line from the eye through X; X sits at parameter 1
      const bool blocked = lines_blocked(bv, active, eye, X - eye, f, it.y, 1e-4f, lds, &ovf);
      if (active && blocked) n_ovf += ovf ? 1u : 0u;
      if (active && !blocked) {
        ++n_vis;
        const float dxt = dot(jx, BA), dyt = dot(jy, BA);
        const float w = sqrtf(dxt * dxt + dyt * dyt) / (float)e.ns;
        const v3 nJ = jx * e.nx + jy * e.ny;
        const v3 ca = nJ * (g * w * (1.0f - t)), cb = nJ * (g * w * t);
        atomicAdd(dV + 3 * (size_t)e.a, ca.x);
        atomicAdd(dV + 3 * (size_t)e.a + 1, ca.y);
        atomicAdd(dV + 3 * (size_t)e.a + 2, ca.z);
        atomicAdd(dV + 3 * (size_t)e.b, cb.x);
        atomicAdd(dV + 3 * (size_t)e.b + 1, cb.y);
        atomicAdd(dV + 3 * (size_t)e.b + 2, cb.z);
      }
    }
    n_items = 0;
    n_points = 0ull;
    wave_lds_sync();
  };

  const int64_t s0 = (int64_t)blockIdx.x * per, s1 = 3 * (int64_t)nf;
  for (int64_t b0 = s0; b0 < s0 + per && b0 < s1; b0 += 64) {
    const int64_t s = b0 + lane;
    uint32_t todo = 0u, fa = 0u;  // cameras whose outline holds this slot's edge
    int f = 0, twin = -1;
    if (s < s1) {
      f = (int)(s / 3);
      const int k = (int)(s % 3);
      const int a = vclampi(F[3 * f + k], nv), b = vclampi(F[3 * f + (k + 1) % 3], nv);
      for (int j = bv.csr_off[b]; j < bv.csr_off[b + 1]; ++j) {
        const int g = bv.csr_idx[j];
        if (g == f) continue;
        if (F[3 * g] == a || F[3 * g + 1] == a || F[3 * g + 2] == a) {
          twin = g;
          break;  // ascending lists: the smallest such face
        }
      }
      if (a < b || twin < 0) {
        fa = facing[f];
        todo = (twin >= 0 ? fa ^ (uint32_t)facing[twin] : 0xFFFFFFFFu) & all;
      }
    }
    while (__ballot(todo != 0u) != 0ull) {
      int cam = 0, front = f;
      SilEdge e;
      e.ns = 0;
      bool ok = false;
      if (todo != 0u) {
        cam = __ffs((int)todo) - 1;
        todo &= todo - 1u;
        if (twin >= 0 && !((fa >> cam) & 1u)) front = twin;
        ok = silhouette_edge(V, F, nv, cams.c[cam], f, (int)(s % 3), front, rho, e);
      }
      const uint64_t m = __ballot(ok);
      if (m == 0ull) continue;
      if (n_items + __popcll(m) > MASK_ITEMS) cast_points();
      // points before this lane's edge: an inclusive scan over the lanes
      unsigned long long inc = ok ? (unsigned long long)e.ns : 0ull;
      for (int st = 1; st < 64; st <<= 1) {
        const unsigned long long up = __shfl_up(inc, st);
        if (lane >= st) inc += up;
      }
      if (ok) {
        const int at = n_items + __popcll(m & lt);
        item[at] = make_int4((int)s, twin, cam, front);
        first[at] = n_points + inc - (unsigned long long)e.ns;
      }
      n_items += __popcll(m);
      n_points += __shfl(inc, 63);
    }
  }
  if (n_items > 0) cast_points();
  if (counts) {
    for (int st = 32; st > 0; st >>= 1) {
      n_in += __shfl_xor(n_in, st);
      n_vis += __shfl_xor(n_vis, st);
      n_ovf += __shfl_xor(n_ovf, st);
    }
    if (lane == 0 && n_in) {
      atomicAdd(counts, (unsigned long long)n_in);
      if (n_vis) atomicAdd(counts + 1, (unsigned long long)n_vis);
      if (n_ovf) atomicAdd(counts + 2, (unsigned long long)n_ovf);
    }
  }
}

__global__ void k_mask_zero(float* p, int64_t n, unsigned long long* counts) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0.f;
  if (counts && blockIdx.x == 0 && threadIdx.x < 3) counts[threadIdx.x] = 0ull;
}

dt_status mask_setup(const dt_scene* sc, const dt_rays* rays, BvhView& bv, MaskCams& mc) {
  DT_REQUIRE(sc && rays, "NULL scene or rays");
  DT_REQUIRE(sc->V && sc->F && sc->bvh, "scene needs V, F and bvh");
  DT_REQUIRE(sc->nv >= 3 && sc->nf >= 1 && sc->nf <= DT_MAX_FACES && sc->nv < (1 << 30),
             "scene needs nv >= 3 and 1 <= nf <= 2^26");
  DT_REQUIRE(rays->kind == DT_RAYS_CAMERAS && rays->cameras, "the mask term takes camera rays");
  DT_REQUIRE(rays->n_cameras >= 1 && rays->n_cameras <= DT_MASK_MAX_CAMERAS,
             "the mask term takes 1..%d cameras per call", DT_MASK_MAX_CAMERAS);
  DT_REQUIRE(rays->n_pixels >= 1 && rays->n_pixels < (1ll << 31), "n_pixels must be in [1, 2^31)");
  mc.n = rays->n_cameras;
  for (int c = 0; c < mc.n; ++c) {
    const dt_camera& cam = rays->cameras[c];
    DT_REQUIRE(cam.width >= 1 && cam.height >= 1 && cam.fov_deg > 0.f && cam.fov_deg < 180.f,
               "camera %d: bad image size or field of view", c);
    DT_REQUIRE(cam.pixel_offset >= 0 && cam.pixel_offset + (int64_t)cam.width * cam.height <= rays->n_pixels,
               "camera %d: image exceeds n_pixels", c);
    if (dt_status st = make_camera(cam, c, mc.c[c])) return st;
  }
  bv = bvh_view(sc->bvh, sc->nv, sc->nf);
  return DT_OK;
}

// the backward's workspace: the faces' facing bits
size_t mask_ws_bytes(int32_t nf) { return dt_align(sizeof(uint16_t) * (size_t)nf); }

}  // namespace

extern "C" dt_status dt_mask_bytes(int32_t nv, int32_t nf, size_t* ws_bytes) {
  DT_REQUIRE(ws_bytes, "dt_mask_bytes: NULL argument");
  DT_REQUIRE(nv >= 3 && nf >= 1 && nf <= DT_MAX_FACES, "dt_mask_bytes: need nv >= 3, 1 <= nf <= 2^26");
  *ws_bytes = mask_ws_bytes(nf);
  return DT_OK;
}

extern "C" dt_status dt_mask_forward(const dt_scene* sc, const dt_rays* rays, float t_eps, float* mask,
                                     void* stream) {
  BvhView bv;
  MaskCams mc;
  if (dt_status st = mask_setup(sc, rays, bv, mc)) return st;
  DT_REQUIRE(mask, "dt_mask_forward: NULL mask");
  DT_REQUIRE(t_eps >= 0.f && t_eps < 1.f, "t_eps must be in [0, 1)");
  hipStream_t s = (hipStream_t)stream;
  int64_t most = 1;  // tiles of the largest image
  for (int c = 0; c < mc.n; ++c)
    most = std::max<int64_t>(most, mask_tile(mc.c[c].W, mc.c[c].H).n);
  hipLaunchKernelGGL(k_mask_forward, dim3((unsigned)most, mc.n), dim3(64), 0, s, bv, mc, t_eps, mask);
  DT_CHECK_LAUNCH();
  return DT_OK;
}

extern "C" dt_status dt_mask_backward(const dt_scene* sc, const dt_rays* rays, const float* grad_mask,
                                      float rho, float* dV, uint64_t* counts, void* ws, size_t ws_bytes,
                                      void* stream) {
  BvhView bv;
  MaskCams mc;
  if (dt_status st = mask_setup(sc, rays, bv, mc)) return st;
  DT_REQUIRE(grad_mask && dV && ws, "dt_mask_backward: NULL argument");
  DT_REQUIRE(rho > 0.f && rho <= 4096.f, "rho must be in (0, 4096]");
  const size_t need = mask_ws_bytes(sc->nf);
  if (ws_bytes < need) {
    dt_set_error("dt_mask_backward: workspace has %zu bytes, needs %zu", ws_bytes, need);
    return DT_ERR_WORKSPACE_TOO_SMALL;
  }
  hipStream_t s = (hipStream_t)stream;
  uint16_t* facing = (uint16_t*)ws;
  const int64_t slots = 3 * (int64_t)sc->nf;
  hipLaunchKernelGGL(k_mask_zero, dim3(dt_blocks(3 * (int64_t)sc->nv, 256) < 4096 ? dt_blocks(3 * (int64_t)sc->nv, 256) : 4096),
                     dim3(256), 0, s, dV, 3 * (int64_t)sc->nv, (unsigned long long*)counts);
  hipLaunchKernelGGL(k_mask_facing, dim3(dt_blocks(sc->nf, MT)), dim3(MT), 0, s, sc->V, sc->F, sc->nv, sc->nf, mc,
                     facing);
  const MaskCut cut = mask_cut(slots, mc.n);
  hipLaunchKernelGGL(k_mask_grad, dim3(dt_blocks(slots, cut.per), cut.groups), dim3(64), 0, s, sc->V, sc->F, sc->nv,
                     sc->nf, bv, facing, mc, grad_mask, rho, dV, (unsigned long long*)counts, cut.per);
  DT_CHECK_LAUNCH();
  return DT_OK;
}
