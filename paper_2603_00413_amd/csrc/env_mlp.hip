// Environment MLP on bf16 matrix cores (gfx950 MFMA 16x16x32, FP32 accumulate).
//
// E(d) = head( relu(... relu(W0 gamma(u) + b0) ...) ), u = d / |d|,
// gamma(u) = [u, sin(2^k pi u), cos(2^k pi u)]_{k < n_freq}, zero-padded to 64.
// Weights are bf16 (exact MFMA operands), biases FP32.  Every activation
// vector (the encoding and each hidden layer's ReLU output) is carried as
// three bf16 vectors (the top, middle and bottom 8 significant bits of the
// FP32 value, cut by truncation, so they sum to it exactly), and each layer is
// three MFMAs (W hi + W mid + W lo) accumulated in FP32: the products of bf16
// weights and bf16 parts are exact, so a layer is as accurate as an FP32
// matrix product.  (A single bf16 rounding per activation would put steps of
// 2^-9 relative into E, and a derivative that depends on which side of a step
// a ray lands.)  The encoding takes sin(pi t), cos(pi t) of t = 2^k u, which
// is exact in FP32 (as is its reduction to a fraction of a turn), so no
// argument rounding error grows with the frequency; the hardware sine and
// cosine then add at most 1.3e-7.
//
// A block first copies the whole network into LDS (laid out so that the rows an
// operand spans fall on different banks; the RGB head padded to 16 rows, the
// extra ones zero), then its waves loop over groups of 16 rays, so the
// weights are read from HBM once per block and every MFMA operand comes from
// LDS.  One wave evaluates 16 rays at a time.  Layers are computed transposed,
// D[out][ray] = W[out][in] * H[in][ray], so W is the MFMA A operand and the
// activations the B operand; the accumulator layout of one layer (lane l holds
// rows 4*(l/16)+j of column l%16) gives each lane four rows of a 16-row
// block, and two consecutive blocks make the eight k values a lane supplies
// to one 16x16x32 product, so activations never leave registers.  The weights'
// columns are stored in the order of that pairing, so an operand of W is one
// 16-byte LDS read.  The input gradient runs the same way with W^T as the A
// operand, which the transposing LDS read takes from the same image (8 bytes a
// lane), and the upstream gradient split into hi + lo (about 16 bits; the
// gradient tolerance is 1e-3).
//
// What bounds it is the issue of vector instructions beside the matrix ones: a
// layer of 16 rays is 24 products (16 x 64 of width 64) against some 100
// instructions of splitting the activations, which therefore work on packed
// pairs (byte permutes and the packed bf16 conversion).  1 M rays, three layers of
// 64: 112 us with 66 % of the vector issue slots taken; four layers of 128, value
// and direction gradient: 617 us (some 1,500 before, when W^T came by two-byte
// reads and the pass ran 4 spilling waves a CU).
#include "dt_queue.h"

namespace {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Four bf16 values of a lane (rows 4q + j of a 16-row block), packed
typedef uint2 Quad;

__device__ __forceinline__ f32x4 mfma16(Quad a, Quad b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(bf16x4, a), __builtin_bit_cast(bf16x4, b), c, 0,
                                                   0, 0);
}
__device__ __forceinline__ f32x4 mfma32(uint4 a, uint4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0,
                                                 0);
}
// K = 32 operand from two K = 16 halves: slots 0..3 take k = 4q + j of the
// first 16-block, slots 4..7 k = 4q + j of the second.  A and B operands are
// always built with the same pairing, so the product sums over the same 32 k
// whatever order the matrix core walks them in.
__device__ __forceinline__ uint4 cat8(Quad lo16, Quad hi16) { return make_uint4(lo16.x, lo16.y, hi16.x, hi16.y); }

// the top halves of two words
__device__ __forceinline__ uint32_t tops(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }

// Three-part bf16 split of FP32 values by truncation: hi keeps the top 8
// significant bits, mid the next 8 of the (exact) remainder, lo the last 8,
// so hi + mid + lo equals the FP32 value exactly (for normal values).
__device__ __forceinline__ void split3(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l) {
  const uint32_t ua = __float_as_uint(a), ub = __float_as_uint(b);
  const float ra = a - __uint_as_float(ua & 0xFFFF0000u), rb = b - __uint_as_float(ub & 0xFFFF0000u);
  const uint32_t va = __float_as_uint(ra), vb = __float_as_uint(rb);
  h = tops(ua, ub);
  m = tops(va, vb);
  l = tops(__float_as_uint(ra - __uint_as_float(va & 0xFFFF0000u)),
           __float_as_uint(rb - __uint_as_float(vb & 0xFFFF0000u)));
}
__device__ __forceinline__ void split3(f32x4 v, Quad& h, Quad& m, Quad& l) {
  split3(v[0], v[1], h.x, m.x, l.x);
  split3(v[2], v[3], h.y, m.y, l.y);
}

// two-part bf16 split with rounding to nearest (ties to even) of both parts:
// hi + lo carries about 17 significant bits of the value
__device__ __forceinline__ uint32_t bf16_pair(float a, float b) {
  const f32x2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ void split2(float a, float b, uint32_t& h, uint32_t& l) {
  h = bf16_pair(a, b);
  l = bf16_pair(a - __uint_as_float(h << 16), b - __uint_as_float(h & 0xFFFF0000u));
}
__device__ __forceinline__ void split2(f32x4 v, Quad& h, Quad& l) {
  split2(v[0], v[1], h.x, l.x);
  split2(v[2], v[3], h.y, l.y);
}

// The encoding in the matrix cores' input order.  Lane group q of a wave holds
// input rows 16 kb + 4 q + j (kb, j < 4) of its ray, so the input rows are
// renumbered: group q < 3 carries axis q in its 16 slots s = 4 kb + j (slot 0:
// u_q; slot 1 + 2f: sin(2^f pi u_q); slot 2 + 2f: cos(2^f pi u_q); f < n_freq
// <= DT_MLP_MAX_FREQ), group 3 and unused slots are zero.  The first layer's
// weight columns are permuted to match when the network is copied to LDS.
#define DT_MLP_MAX_FREQ 7

// input column (in the caller's order: u, then per frequency sin xyz, cos xyz)
// of input row k in the matrix cores' order, or -1 for a zero row
__device__ __forceinline__ int enc_column(int k, int n_freq) {
  const int q = (k & 15) >> 2, s = ((k >> 4) << 2) | (k & 3);
  if (q == 3) return -1;
  if (s == 0) return q;
  const int f = (s - 1) >> 1;
  if (f >= n_freq) return -1;
  return 3 + 6 * f + ((s & 1) ? q : 3 + q);
}

// the input row of input column c, or -1 for a column that the encoding leaves unused
__device__ __forceinline__ int enc_row(int c, int n_freq) {
  const int f = c < 3 ? 0 : (c - 3) / 6, r = c < 3 ? c : (c - 3) % 6;
  if (c >= 3 + 6 * n_freq) return -1;
  const int q = r >= 3 ? r - 3 : r, s = c < 3 ? 0 : 1 + 2 * f + (r >= 3 ? 1 : 0);
  return ((s >> 2) << 4) | (q << 2) | (s & 3);
}

// sin(pi 2^f u), cos(pi 2^f u) for f < n_freq by the hardware sine and cosine
// (arguments in turns: 2^(f-1) u exactly, reduced by its nearest integer,
// also exact); within 1.3e-7 of the true values over |u| <= 1, f < 7
struct EncTrig {
  float sn[DT_MLP_MAX_FREQ], cs[DT_MLP_MAX_FREQ];
};
__device__ __forceinline__ EncTrig enc_trig(float uq, int n_freq) {
  EncTrig t;
#pragma unroll
  for (int f = 0; f < DT_MLP_MAX_FREQ; ++f) {
    t.sn[f] = 0.f;
    t.cs[f] = 0.f;
    if (f < n_freq) {
      float h = uq * (float)(1 << f) * 0.5f;
      h -= rintf(h);
      t.sn[f] = __builtin_amdgcn_sinf(h);
      t.cs[f] = __builtin_amdgcn_cosf(h);
    }
  }
  return t;
}

// slot s of a lane group carrying axis value uq
__device__ __forceinline__ float enc_slot(int s, float uq, const EncTrig& t, int n_freq) {
  if (s == 0) return uq;
  const int f = (s - 1) >> 1;
  if (f >= DT_MLP_MAX_FREQ || f >= n_freq) return 0.f;
  return (s & 1) ? t.sn[f] : t.cs[f];
}

// d slot / d uq
__device__ __forceinline__ float denc_slot(int s, const EncTrig& t, int n_freq) {
  if (s == 0) return 1.f;
  const int f = (s - 1) >> 1;
  if (f >= DT_MLP_MAX_FREQ || f >= n_freq) return 0.f;
  const float w = DT_PI * (float)(1 << f);
  return (s & 1) ? w * t.cs[f] : -w * t.sn[f];
}

constexpr int IN = 64;           // padded input width
constexpr int MLP_T = 512;       // threads per block: 8 waves share one LDS copy of the network

// Layout of the LDS image of a (HID, NL) network: bf16 weights row by row (layer
// 0: HID rows of IN; hidden layers: HID rows of HID; head: 16 rows of HID, rows
// 3..15 zero), then FP32 biases (NL x HID, head 16).  Within 32 columns of a row,
// the four of each 16-block that lane group q supplies to one product stand side
// by side (a chunk of 16 bytes).  64-wide rows are not padded, their chunks are
// exchanged by the row's low bits; 128-wide ones are padded by 16: an operand
// then takes 5.1 to 5.3 cycles of the LDS, a transposed half 4.3 (padded by 8,
// rows of either width: 8.1, and 6.2 or 8.3).
template <int HID, int NL>
struct NetLds {
  static constexpr int LD0 = IN;
  static constexpr int LDH = HID == 64 ? 64 : HID + 16;
  static constexpr int W0 = 0;
  static constexpr int WH = W0 + HID * LD0;
  static constexpr int WO = WH + (NL - 1) * HID * LDH;
  static constexpr int WEND = WO + 16 * LDH;
  static constexpr int BOFF = (WEND * 2 + 15) / 16 * 16;  // byte offset of the biases
  static constexpr int NB = NL * HID + 16;
  static constexpr int BYTES = BOFF + NB * 4;
  static_assert(BYTES <= 160 * 1024, "network does not fit in LDS");
};

// chunk 4 kc + q of a row of stride LD
template <int LD>
__device__ __forceinline__ int chunk_at(int row, int chunk) {
  return row * LD + 8 * (LD == 64 ? chunk ^ (row & 7) : chunk);
}
// column c (its group of four columns stands together)
template <int LD>
__device__ __forceinline__ int col_at(int row, int c) {
  return chunk_at<LD>(row, ((c >> 5) << 2) | ((c >> 2) & 3)) + (((c >> 4) & 1) << 2) + (c & 3);
}

// eight consecutive weights; the caller's array need not be aligned to 16 bytes
__device__ __forceinline__ uint4 load8(const uint16_t* p, bool aligned) {
  if (aligned) return *(const uint4*)p;
  return make_uint4(p[0] | (uint32_t)p[1] << 16, p[2] | (uint32_t)p[3] << 16, p[4] | (uint32_t)p[5] << 16,
                    p[6] | (uint32_t)p[7] << 16);
}

// Cooperative copy of the network (global layout: W[l] row-major [out][in],
// biases concatenated) into its LDS image, eight weights at a time; ends with a
// barrier.
template <int HID, int NL>
__device__ __forceinline__ void load_net(const EnvDev& e, uint16_t* sw, float* sb) {
  using N = NetLds<HID, NL>;
  const uint16_t* W = e.w;
  const bool al = ((uintptr_t)W & 15u) == 0;
  const int T = blockDim.x;
  for (int i = threadIdx.x; i < HID * N::LD0 / 4; i += T) *(uint2*)(sw + N::W0 + 4 * i) = make_uint2(0u, 0u);
  for (int i = threadIdx.x; i < 16 * N::LDH / 4; i += T) *(uint2*)(sw + N::WO + 4 * i) = make_uint2(0u, 0u);
  for (int i = threadIdx.x; i < N::NB; i += T) sb[i] = i < NL * HID + 3 ? e.b[i] : 0.f;
  auto put = [&](uint16_t* w, int row, int c, uint4 v) {
    *(uint2*)(w + col_at<N::LDH>(row, c)) = make_uint2(v.x, v.y);
    *(uint2*)(w + col_at<N::LDH>(row, c + 4)) = make_uint2(v.z, v.w);
  };
  for (int l = 1; l < NL; ++l)
    for (int i = threadIdx.x; i < HID * HID / 8; i += T) {
      const int r = i / (HID / 8), c = i % (HID / 8) * 8;
      put(sw + N::WH + (l - 1) * HID * N::LDH, r, c, load8(W + HID * IN + ((l - 1) * HID + r) * HID + c, al));
    }
  __syncthreads();
  // first layer: columns in the matrix cores' input order
  for (int i = threadIdx.x; i < HID * IN / 8; i += T) {
    const int r = i / (IN / 8), c = i % (IN / 8) * 8;
    const uint4 v = load8(W + r * IN + c, al);
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int k = enc_row(c + j, e.n_freq);
      if (k >= 0) sw[N::W0 + col_at<N::LD0>(r, k)] = (uint16_t)(w[j >> 1] >> (16 * (j & 1)));
    }
  }
  for (int i = threadIdx.x; i < 3 * HID / 8; i += T) {
    const int r = i / (HID / 8), c = i % (HID / 8) * 8;
    put(sw + N::WO, r, c, load8(W + HID * IN + (NL - 1) * HID * HID + r * HID + c, al));
  }
  __syncthreads();
}

// A operand of 16 rows of a weight block: columns 32 kc + 4q + j and 32 kc + 16 +
// 4q + j of row `row`
template <int LD>
__device__ __forceinline__ uint4 wfrag(const uint16_t* w, int row, int kc, int q) {
  return *(const uint4*)(w + chunk_at<LD>(row, 4 * kc + q));
}

typedef short s16x4 __attribute__((ext_vector_type(4)));
// Transposing read: each 16 lanes read a 4 x 16 block, lane i the four values at
// p (row i / 4, columns 4 (i % 4) ..), and lane i gets column i of it, rows 0..3.
__device__ __forceinline__ Quad read_tr(const uint16_t* p) {
  return __builtin_bit_cast(Quad,
                            __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p));
}
// Operand of W^T, K = 16: rows (the weights' columns) 16 ib + r16, k (the
// weights' rows) k0 + 4q + j
template <int LD>
__device__ __forceinline__ Quad wfrag_t16(const uint16_t* w, int ib, int k0, int q, int r16) {
  return read_tr(w + chunk_at<LD>(k0 + 4 * q + (r16 >> 2), 4 * (ib >> 1) + (r16 & 3)) + 4 * (ib & 1));
}
template <int LD>
__device__ __forceinline__ uint4 wfrag_t(const uint16_t* w, int ib, int kc, int q, int r16) {
  return cat8(wfrag_t16<LD>(w, ib, 32 * kc, q, r16), wfrag_t16<LD>(w, ib, 32 * kc + 16, q, r16));
}

// ------------------------------------------------------------------ weight gradient
// dLoss/dW_l = sum over rays of delta_l a_{l-1}^T and dLoss/db_l = sum of
// delta_l, with delta_l the adjoint of layer l's pre-activation and a_{l-1}
// its input (the encoding for l = 0).  The sum over rays is a matrix product
// with the rays as the contraction axis, so it runs on the matrix cores too:
// hi*hi + hi*mid + lo*hi of the deltas' two bf16 parts (about 17 bits) and the
// inputs' hi and mid parts (16 bits); the bias products multiply the deltas by
// ones.  The operands have the rays along k where the layers have the features:
// the 4 waves of a block leave a layer's parts in LDS ray by ray (16 eight-byte
// writes a lane) and the transposing read turns them.  Wave w owns the output
// block w of every layer, so its deltas' operands serve four products; two
// blocks share a CU, and one works while the other waits at a barrier.  Each
// entry of the gradient belongs to one lane of the block; at the end the block
// adds its accumulators into its own row of partial sums, and a final pass sums
// the rows in order.  64-wide networks only.
// (1 M rays of a three-layer network: 613 us with the parts written feature by
// feature in 64 two-byte writes a lane, 8 waves per block and spilled registers;
// 581 us with the whole gradient in each wave's accumulators, no barriers and one
// wave per SIMD; 365 us this way.)
constexpr int WG_T = 256;
constexpr int WG_RAYS = WG_T / 4;           // rays of a round
constexpr int WG_BLOCKS = 2 * MLP_WG_ROWS;  // blocks of the weight-gradient backward (rows of partials)
constexpr int WG_LD = 64 + 4;      // a write takes 7.2 cycles of the LDS, a transposing read 4.3, without conflicts
constexpr int WG_PART = WG_RAYS * WG_LD;  // one staged part: [ray][feature]

template <int NL>
struct Wg {
  // flat parameter layout (weights of every layer, then biases), 64 wide
  static constexpr int64_t n_weights = 4096 * (int64_t)NL + 192;
  static constexpr int64_t n_params = n_weights + 64 * (int64_t)NL + 3;
  f32x4 w[NL][4], b[NL];  // this wave's output block of each layer, by input block; bias
  f32x4 hw, hb;           // head: this wave's input block; bias
};

// leave rows 16 b + 4q + j of this lane's ray (row `ray` of the stage)
__device__ __forceinline__ void wg_put(uint16_t* part, int ray, int b, int q, Quad v) {
  *(Quad*)(part + ray * WG_LD + 16 * b + 4 * q) = v;
}
// operand with row 16 b + r16 and k the rays of 32 ks
__device__ __forceinline__ uint4 wg_get(const uint16_t* part, int b, int ks, int q, int r16) {
  const uint16_t* p = part + (32 * ks + 4 * q + (r16 >> 2)) * WG_LD + 16 * b + 4 * (r16 & 3);
  return cat8(read_tr(p), read_tr(p + 16 * WG_LD));
}

// Stage a layer's deltas (OB blocks) and inputs (4), then add this wave's
// products.  Called by every wave of the block the same number of times (it
// holds two barriers).
template <int OB>
__device__ __forceinline__ void wg_layer(uint16_t* st, const Quad* dh, const Quad* dl, const Quad* ih, const Quad* im,
                                         int wave, int q, int r16, f32x4* w, f32x4& bias) {
  uint16_t *Dh = st, *Dl = st + WG_PART, *Ih = st + 2 * WG_PART, *Im = st + 3 * WG_PART;
  const int ray = 16 * wave + r16;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    if (b < OB) {
      wg_put(Dh, ray, b, q, dh[b]);
      wg_put(Dl, ray, b, q, dl[b]);
    }
    wg_put(Ih, ray, b, q, ih[b]);
    wg_put(Im, ray, b, q, im[b]);
  }
  __syncthreads();
  const uint4 ones = make_uint4(0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u);
  const int ob = OB == 1 ? 0 : wave;
#pragma unroll
  for (int ks = 0; ks < WG_RAYS / 32; ++ks) {
    const uint4 ah = wg_get(Dh, ob, ks, q, r16), al = wg_get(Dl, ob, ks, q, r16);
    constexpr int IB = OB == 1 ? 1 : 4;
    uint4 bh[IB];
#pragma unroll
    for (int k = 0; k < IB; ++k) {
      bh[k] = wg_get(Ih, OB == 1 ? wave : k, ks, q, r16);
      w[k] = mfma32(ah, bh[k], w[k]);
    }
    bias = mfma32(ah, ones, bias);
#pragma unroll
    for (int k = 0; k < IB; ++k) w[k] = mfma32(ah, wg_get(Im, OB == 1 ? wave : k, ks, q, r16), w[k]);
    bias = mfma32(al, ones, bias);
#pragma unroll
    for (int k = 0; k < IB; ++k) w[k] = mfma32(al, bh[k], w[k]);
  }
  __syncthreads();
}

// Add a tile (output block ob, input block ib of layer L, `rows` rows) to the
// flat parameters.  Weight (o, i) of layer 0 is the caller's column enc_column(i).
__device__ __forceinline__ void wg_flush(float* part, int L, int ob, int ib, int rows, f32x4 w, int q, int r16,
                                         int n_freq) {
  int i = 16 * ib + r16;
  if (L == 0) i = enc_column(i, n_freq);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int o = 16 * ob + 4 * q + j;
    if (o < rows && i >= 0) part[4096 * L + 64 * o + i] += w[j];
  }
}
__device__ __forceinline__ void wg_flush_bias(float* bias, int ob, int rows, f32x4 b, int q, int r16) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int o = 16 * ob + 4 * q + j;
    if (r16 == 0 && o < rows) bias[o] += b[j];
  }
}

// ------------------------------------------------------------------ one wave
template <int V>
struct Ld {  // a row stride as a type
  static constexpr int value = V;
};
// One wave: lane l works on ray l % 16 (all four lane groups q = l / 16 carry
// the same ray).  Returns E in lanes with q == 0; when GRAD, also returns
// the direction gradient of dot(gbar(), E) with respect to d (all lanes).
// Activations live in 16-row blocks in the MFMA accumulator layout (lane
// (q, r16) holds rows 4q + j of column r16); two consecutive blocks form the
// B operand of one 16x16x32 product.  WG: the block's stage and the wave's part
// of the gradient.
template <int HID, int NL, bool GRAD, bool WG, class G>
__device__ __forceinline__ v3 mlp_wave(const uint16_t* sw, const float* sb, int n_freq, v3 d, G gbar, v3* dbar,
                                       uint16_t* stage, Wg<NL>* wg) {
  const int wave = threadIdx.x >> 6;
  static_assert(!WG || (GRAD && HID == 64), "weight gradient: 64-wide backward only");
  using N = NetLds<HID, NL>;
  const int l = threadIdx.x & 63, q = l >> 4, r16 = l & 15;
  constexpr int KB = HID / 16, XB = IN / 16;
  float inv_len = 1.0f / sqrtf(dot(d, d));
  v3 u = d * inv_len;
  // this lane group's axis (group 3 carries zeros)
  const float uq = q == 0 ? u.x : (q == 1 ? u.y : (q == 2 ? u.z : 0.f));
  const int nfq = q == 3 ? 0 : n_freq;
  const EncTrig trig = enc_trig(uq, nfq);
  Quad inh[WG ? NL + 1 : 1][4], inm[WG ? NL + 1 : 1][4];  // every layer's input (weight gradient)
  Quad hi[KB > XB ? KB : XB], mi[KB > XB ? KB : XB], lo[KB > XB ? KB : XB];  // the current layer's input
#pragma unroll
  for (int kb = 0; kb < XB; ++kb) {
    f32x4 v;
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = enc_slot(4 * kb + j, uq, trig, nfq);
    split3(v, hi[kb], mi[kb], lo[kb]);
    if constexpr (WG) {
      inh[0][kb] = hi[kb];
      inm[0][kb] = mi[kb];
    }
  }
  // a row block of W x + b, the parts of x from the smallest
  auto row_block = [&](auto ld, const uint16_t* w, int row, int blocks, const float* B) {
    f32x4 acc = *(const f32x4*)(B + 4 * q);
#pragma unroll
    for (int kc = 0; kc < blocks / 2; ++kc) {
      const uint4 a = wfrag<decltype(ld)::value>(w, row, kc, q);
      acc = mfma32(a, cat8(lo[2 * kc], lo[2 * kc + 1]), acc);
      acc = mfma32(a, cat8(mi[2 * kc], mi[2 * kc + 1]), acc);
      acc = mfma32(a, cat8(hi[2 * kc], hi[2 * kc + 1]), acc);
    }
    return acc;
  };
  // relu(v) = med3(v, 0, inf), which like max takes a NaN to 0; with the bound out
  // of the compiler's sight it is one instruction (max first quiets its operand)
  float inf = __builtin_inff();
  asm("" : "+s"(inf));
  // hidden layers; relu' of layer L's row 16 ob + 4q + j is bit 4 KB - 1 - (4 ob + j) of mask[L]
  uint32_t mask[NL];
#pragma unroll
  for (int L = 0; L < NL; ++L) {
    Quad nh[KB], nm[KB], nl[KB];
    uint32_t m = 0;
#pragma unroll
    for (int ob = 0; ob < KB; ++ob) {
      f32x4 acc = L == 0 ? row_block(Ld<N::LD0>(), sw + N::W0, ob * 16 + r16, XB, sb + ob * 16)
                         : row_block(Ld<N::LDH>(), sw + N::WH + (L - 1) * HID * N::LDH, ob * 16 + r16, KB,
                                     sb + L * HID + ob * 16);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        acc[j] = __builtin_amdgcn_fmed3f(acc[j], 0.f, inf);
        // 0 - v is negative where v > 0
        if constexpr (GRAD) m = __builtin_amdgcn_alignbit(m, __float_as_uint(0.f - acc[j]), 31);
      }
      split3(acc, nh[ob], nm[ob], nl[ob]);
      if constexpr (WG) {
        inh[L + 1][ob] = nh[ob];
        inm[L + 1][ob] = nm[ob];
      }
    }
#pragma unroll
    for (int ob = 0; ob < KB; ++ob) {
      hi[ob] = nh[ob];
      mi[ob] = nm[ob];
      lo[ob] = nl[ob];
    }
    mask[L] = m;
  }
  // linear RGB head (3 rows, padded to 16 zero rows)
  const f32x4 out = row_block(Ld<N::LDH>(), sw + N::WO, r16, KB, sb + NL * HID);
  v3 E = mk3(out[0], out[1], out[2]);
  if constexpr (!GRAD) return E;

  // ---- input gradient: delta_out rows 0..2 = gbar, B layout
  auto masked = [&](f32x4 a, int L, int ib) {
    f32x4 r;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      r[j] = __uint_as_float(__float_as_uint(a[j]) &
                             (uint32_t)__builtin_amdgcn_sbfe((int)mask[L], 4 * KB - 1 - (4 * ib + j), 1));
    return r;
  };
  const v3 gb = gbar();
  Quad dh0, dl0;  // delta of the head output, hi / lo parts (rows 0..2 of lane group 0)
  split2(q == 0 ? f32x4{gb.x, gb.y, gb.z, 0.f} : f32x4{0.f, 0.f, 0.f, 0.f}, dh0, dl0);
  if constexpr (WG) wg_layer<1>(stage, &dh0, &dl0, inh[NL], inm[NL], wave, q, r16, &wg->hw, wg->hb);
  // head: delta_hidden = W_head^T delta_out (a K = 16 product over the 16
  // padded head rows), masked by the last ReLU
  Quad nh[KB], nl[KB];
#pragma unroll
  for (int ib = 0; ib < KB; ++ib) {
    const Quad a = wfrag_t16<N::LDH>(sw + N::WO, ib, 0, q, r16);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    acc = mfma16(a, dh0, acc);
    acc = mfma16(a, dl0, acc);
    split2(masked(acc, NL - 1, ib), nh[ib], nl[ib]);
  }
  auto t_block = [&](auto ld, const uint16_t* w, int ib) {  // rows 16 ib .. of W^T delta
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kc = 0; kc < KB / 2; ++kc) {
      const uint4 a = wfrag_t<decltype(ld)::value>(w, ib, kc, q, r16);
      acc = mfma32(a, cat8(nh[2 * kc], nh[2 * kc + 1]), acc);
      acc = mfma32(a, cat8(nl[2 * kc], nl[2 * kc + 1]), acc);
    }
    return acc;
  };
  auto grad_layer = [&](int L) {
    if constexpr (WG) wg_layer<4>(stage, nh, nl, inh[L], inm[L], wave, q, r16, wg->w[L], wg->b[L]);
  };
  // hidden layers NL-1 .. 1: delta_{L-1} = W_L^T delta_L, masked by relu'(layer L-1)
#pragma unroll
  for (int L = NL - 1; L >= 1; --L) {
    grad_layer(L);
    Quad th[KB], tl[KB];
#pragma unroll
    for (int ib = 0; ib < KB; ++ib)
      split2(masked(t_block(Ld<N::LDH>(), sw + N::WH + (L - 1) * HID * N::LDH, ib), L - 1, ib), th[ib], tl[ib]);
#pragma unroll
    for (int ib = 0; ib < KB; ++ib) {
      nh[ib] = th[ib];
      nl[ib] = tl[ib];
    }
  }
  grad_layer(0);
  // first layer: delta_enc = W_0^T delta_0 (64 rows), then d enc / d u_q
  float gq = 0.f;
#pragma unroll
  for (int ib = 0; ib < XB; ++ib) {
    const f32x4 acc = t_block(Ld<N::LD0>(), sw + N::W0, ib);
    // acc[j] = d loss / d (slot 4 ib + j) of ray r16 in this lane group
#pragma unroll
    for (int j = 0; j < 4; ++j) gq += acc[j] * denc_slot(4 * ib + j, trig, nfq);
  }
  // lane group q < 3 holds d / d u_q; the groups of one ray are lanes r16 + 16 q
  float gx = q == 0 ? gq : 0.f, gy = q == 1 ? gq : 0.f, gz = q == 2 ? gq : 0.f;
  gx += __shfl_xor(gx, 16);
  gy += __shfl_xor(gy, 16);
  gz += __shfl_xor(gz, 16);
  gx += __shfl_xor(gx, 32);
  gy += __shfl_xor(gy, 32);
  gz += __shfl_xor(gz, 32);
  // through u = d / |d|
  v3 gu = mk3(gx, gy, gz);
  *dbar = (gu - u * dot(u, gu)) * inv_len;
  return E;
}
template <int HID, int NL>
__device__ __forceinline__ v3 mlp_value(const uint16_t* sw, const float* sb, int n_freq, v3 d) {
  return mlp_wave<HID, NL, false, false>(sw, sb, n_freq, d, [] { return mk3(0.f, 0.f, 0.f); }, nullptr, nullptr,
                                         nullptr);
}

// ------------------------------------------------------------------ kernels
// Every block loads the network into LDS once, then each of its waves takes
// groups of 16 consecutive items in turn; items past the count run on a dummy
// direction and write nothing.  The loops' trip counts are uniform per wave.
#define DT_MLP_PROLOGUE                                                   \
  using N = NetLds<HID, NL>;                                              \
  __shared__ __align__(16) unsigned char net[N::BYTES];                  \
  uint16_t* sw = (uint16_t*)net;                                          \
  float* sb = (float*)(net + N::BOFF);                                    \
  load_net<HID, NL>(e, sw, sb);                                           \
  const int64_t wstep = (int64_t)gridDim.x * (MLP_T / 64) * 16;           \
  const int64_t wfirst = ((int64_t)blockIdx.x * (MLP_T / 64) + (threadIdx.x >> 6)) * 16;

// An opaque zero offset per group: the weight reads then depend on the loop
// iteration, so the compiler streams them from LDS in every group instead of
// hoisting the whole network into registers (which spills for 128-wide nets).
__device__ __forceinline__ const uint16_t* per_group(const uint16_t* sw) {
  int z = 0;
  asm volatile("" : "+s"(z));
  return sw + z;
}

template <int HID, int NL>
__global__ void __launch_bounds__(MLP_T) k_mlp_query(EnvDev e, const float* dirs, int64_t n, float* rgb) {
  DT_MLP_PROLOGUE
  for (int64_t w0 = wfirst; w0 < n; w0 += wstep) {
    int64_t item = w0 + (threadIdx.x & 15);
    bool valid = item < n;
    v3 d = valid ? load3(dirs + 3 * item) : mk3(0.f, 1.f, 0.f);
    v3 E = mlp_value<HID, NL>(per_group(sw), sb, e.n_freq, d);
    if (valid && (threadIdx.x & 63) < 16) {
      rgb[3 * item] = E.x;
      rgb[3 * item + 1] = E.y;
      rgb[3 * item + 2] = E.z;
    }
  }
}

template <int HID, int NL>
__global__ void __launch_bounds__(MLP_T) k_mlp_query_bwd(EnvDev e, const float* dirs, int64_t n, const float* g,
                                                         float* gd) {
  DT_MLP_PROLOGUE
  for (int64_t w0 = wfirst; w0 < n; w0 += wstep) {
    int64_t item = w0 + (threadIdx.x & 15);
    bool valid = item < n;
    v3 d = valid ? load3(dirs + 3 * item) : mk3(0.f, 1.f, 0.f);
    v3 gb = valid ? load3(g + 3 * item) : mk3(0.f, 0.f, 0.f);
    v3 db;
    mlp_wave<HID, NL, true, false>(per_group(sw), sb, e.n_freq, d, [&] { return gb; }, &db, nullptr, nullptr);
    if (valid && (threadIdx.x & 63) < 16) {
      gd[3 * item] = db.x;
      gd[3 * item + 1] = db.y;
      gd[3 * item + 2] = db.z;
    }
  }
}

// One listed ray of a lane.  A wave's next group is fetched while it works on
// the current one (list entry, then ray: two dependent reads, which the few
// waves of these kernels would not hide).
struct MissRay {
  bool valid;
  uint32_t i;
  float4 d, w;
};
__device__ __forceinline__ uint32_t miss_index(const uint32_t* list, int64_t item, int64_t n) {
  return item < n ? list[item] : 0u;
}
__device__ __forceinline__ MissRay miss_ray(const Gen& q, uint32_t i, int64_t item, int64_t n) {
  MissRay r;
  r.valid = item < n;
  r.i = i;
  r.d = r.valid ? q.d[i] : make_float4(0.f, 1.f, 0.f, 0.f);
  r.w = r.valid ? q.w[i] : make_float4(0.f, 0.f, 0.f, 0.f);
  return r;
}
__device__ __forceinline__ v3 miss_grad(const MissRay& r, const float* grad_rgb) {
  if (!r.valid) return mk3(0.f, 0.f, 0.f);
  const v3 gp = load3(grad_rgb + 3 * __float_as_int(r.d.w));
  return mk3(gp.x * r.w.x, gp.y * r.w.y, gp.z * r.w.z);
}
__device__ __forceinline__ void miss_store(const Adj& cur, const MissRay& r, v3 E, v3 db) {
  if (!r.valid || (threadIdx.x & 63) >= 16) return;
  cur.L[r.i] = make_float4(E.x, E.y, E.z, 0.f);
  cur.O[r.i] = make_float4(0.f, 0.f, 0.f, 0.f);
  cur.D[r.i] = make_float4(db.x, db.y, db.z, 0.f);
}
// calls fn(ray) on `groups` groups of 16 listed rays: wfirst, wfirst + wstep, ...
template <class F>
__device__ __forceinline__ void for_misses(const Gen& q, const uint32_t* list, int64_t n, int64_t wfirst,
                                           int64_t wstep, int64_t groups, F fn) {
  const int64_t r16 = threadIdx.x & 15;
  MissRay cur = miss_ray(q, miss_index(list, wfirst + r16, n), wfirst + r16, n);
  uint32_t next = miss_index(list, wfirst + wstep + r16, n);
  int64_t w0 = wfirst;
  for (int64_t k = 0; k < groups; ++k, w0 += wstep) {
    const MissRay ray = cur;
    cur = miss_ray(q, next, w0 + wstep + r16, n);
    next = miss_index(list, w0 + 2 * wstep + r16, n);
    fn(ray);
  }
}

template <int HID, int NL>
__global__ void __launch_bounds__(MLP_T) k_mlp_trace_fwd(EnvDev e, Gen q, const uint32_t* list, const Counters* ctr,
                                                         int g, float* rgb) {
  DT_MLP_PROLOGUE
  const int l = threadIdx.x & 63;
  const int64_t n = ctr->nmiss[g];
  for_misses(q, list, n, wfirst, wstep, wfirst < n ? (n - wfirst + wstep - 1) / wstep : 0, [&](const MissRay& r) {
    const v3 E = mlp_value<HID, NL>(per_group(sw), sb, e.n_freq, xyz(r.d));
    // the 16 rays' 48 values in one instruction: atomics are carried out at the
    // memory side, per line of an instruction
    const int c = l % 3, src = l < 48 ? l / 3 : 0;
    const float vx = __shfl(r.w.x * E.x, src), vy = __shfl(r.w.y * E.y, src), vz = __shfl(r.w.z * E.z, src);
    const int pix = __shfl(r.valid ? __float_as_int(r.d.w) : -1, src);
    if (l < 48 && pix >= 0) atomicAdd(rgb + 3 * (int64_t)pix + c, c == 0 ? vx : (c == 1 ? vy : vz));
  });
}

template <int HID, int NL>
__global__ void __launch_bounds__(MLP_T) k_mlp_trace_bwd(EnvDev e, Gen q, const uint32_t* list, const Counters* ctr,
                                                         int g, const float* grad_rgb, Adj cur) {
  DT_MLP_PROLOGUE
  const int64_t n = ctr->nmiss[g];
  for_misses(q, list, n, wfirst, wstep, wfirst < n ? (n - wfirst + wstep - 1) / wstep : 0, [&](const MissRay& r) {
    const v3 gb = miss_grad(r, grad_rgb);
    v3 db;
    const v3 E = mlp_wave<HID, NL, true, false>(per_group(sw), sb, e.n_freq, xyz(r.d), [&] { return gb; }, &db, nullptr,
                                                nullptr);
    miss_store(cur, r, E, db);
  });
}

// The trace adjoint of k_mlp_trace_bwd for a 64-wide network, also summing the
// weight and bias gradient, the block's sums added into part[blockIdx.x][...]
// at the end.
template <int NL>
__global__ void __launch_bounds__(WG_T, 2) k_mlp_trace_bwd_wg(EnvDev e, Gen q, const uint32_t* list,
                                                              const Counters* ctr, int g, const float* grad_rgb,
                                                              Adj cur, MlpParts part) {
  using N = NetLds<64, NL>;
  using W = Wg<NL>;
  __shared__ __align__(16) unsigned char net[N::BYTES];
  __shared__ __align__(16) uint16_t stage[4 * WG_PART];
  static_assert(N::BYTES + sizeof(stage) <= 80 * 1024, "two blocks share a CU");
  uint16_t* sw = (uint16_t*)net;
  float* sb = (float*)(net + N::BOFF);
  load_net<64, NL>(e, sw, sb);
  const int wave = threadIdx.x >> 6, l = threadIdx.x & 63, lq = l >> 4, r16 = l & 15;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  W wg;
#pragma unroll
  for (int L = 0; L < NL; ++L) {
    wg.b[L] = zero;
#pragma unroll
    for (int ib = 0; ib < 4; ++ib) wg.w[L][ib] = zero;
  }
  wg.hw = wg.hb = zero;
  // rounds of WG_RAYS listed rays: all waves take part in every round (rays past
  // the count carry a zero adjoint)
  const int64_t n = ctr->nmiss[g], rounds = (n + WG_RAYS - 1) / WG_RAYS;
  const int64_t mine = rounds > blockIdx.x ? (rounds - blockIdx.x + gridDim.x - 1) / gridDim.x : 0;
  const int64_t step = (int64_t)gridDim.x * WG_RAYS, first = (int64_t)blockIdx.x * WG_RAYS + 16 * wave;
  for_misses(q, list, n, first, step, mine, [&](const MissRay& r) {
    const v3 gb = miss_grad(r, grad_rgb);
    v3 db;
    const v3 E =
        mlp_wave<64, NL, true, true>(per_group(sw), sb, e.n_freq, xyz(r.d), [&] { return gb; }, &db, stage, &wg);
    miss_store(cur, r, E, db);
  });
  float* row = part.run[blockIdx.x / MLP_WG_ROWS] + (size_t)(blockIdx.x % MLP_WG_ROWS) * W::n_params;
#pragma unroll
  for (int L = 0; L < NL; ++L) {
#pragma unroll
    for (int ib = 0; ib < 4; ++ib) wg_flush(row, L, wave, ib, 64, wg.w[L][ib], lq, r16, e.n_freq);
    wg_flush_bias(row + W::n_weights + 64 * L, wave, 64, wg.b[L], lq, r16);
  }
  wg_flush(row, NL, 0, wave, 3, wg.hw, lq, r16, e.n_freq);
  if (wave == 0) wg_flush_bias(row + W::n_weights + 64 * NL, 0, 3, wg.hb, lq, r16);
}
#undef DT_MLP_PROLOGUE

// d_w[k] (k < n_weights) and d_b[k - n_weights]: the blocks' partial sums,
// added in block order
__global__ void k_mlp_wg_reduce(MlpParts part, int64_t n_params, int64_t n_weights, float* d_w,
                                float* d_b) {
  for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n_params;
       k += (int64_t)gridDim.x * blockDim.x) {
    double s = 0.0;
    for (int r = 0; r < 2; ++r)
      for (int b = 0; b < MLP_WG_ROWS; ++b) s += (double)part.run[r][(size_t)b * n_params + k];
    if (k < n_weights)
      d_w[k] = (float)s;
    else
      d_b[k - n_weights] = (float)s;
  }
}

// dispatch over the supported (hidden width, hidden layers) shapes
#define DT_MLP_SHAPES(X) X(64, 1) X(64, 2) X(64, 3) X(64, 4) X(128, 1) X(128, 2) X(128, 3) X(128, 4)

// enough blocks to cover n items (16 per wave), at most those that are resident
// together: each copies the network once.  A network of one layer holds so few
// registers and so little LDS that three blocks share a CU, and copies so little
// that a fourth in line costs nothing (8 M directions, 512 or 256 blocks against
// 1,024: width 64 316 and 291 us, width 128 557 and 441)
unsigned mlp_blocks(int64_t n, int hidden, int layers) {
  int64_t per = MLP_T / 4;  // 16 items per wave
  int64_t b = (n + per - 1) / per;
  const int64_t cap = layers == 1 ? 1024 : (hidden == 64 ? 512 : 256);
  return (unsigned)(b < 1 ? 1 : (b > cap ? cap : b));
}

}  // namespace

bool mlp_supported(const EnvDev& e) {
  return e.in_pad == IN && (e.hidden == 64 || e.hidden == 128) && e.n_layers >= 1 &&
         e.n_layers <= 4 && e.n_freq >= 0 && e.n_freq <= DT_MLP_MAX_FREQ && e.w && e.b;
}

#define DT_LAUNCH(H, L, kern, grid, ...)                                                    \
  if (e.hidden == H && e.n_layers == L) {                                                   \
    hipLaunchKernelGGL((kern<H, L>), dim3(grid), dim3(MLP_T), 0, s, __VA_ARGS__); \
    DT_CHECK_LAUNCH();                                                                      \
    return DT_OK;                                                                           \
  }

dt_status mlp_query(const EnvDev& e, const float* dirs, int64_t n, float* rgb, hipStream_t s) {
#define X(H, L) DT_LAUNCH(H, L, k_mlp_query, mlp_blocks(n, H, L), e, dirs, n, rgb)
  DT_MLP_SHAPES(X)
#undef X
  dt_set_error("environment MLP shape (hidden %d, layers %d) is not supported", e.hidden, e.n_layers);
  return DT_ERR_UNSUPPORTED;
}

dt_status mlp_query_backward(const EnvDev& e, const float* dirs, int64_t n, const float* g,
                             float* gd, hipStream_t s) {
#define X(H, L) DT_LAUNCH(H, L, k_mlp_query_bwd, mlp_blocks(n, H, L), e, dirs, n, g, gd)
  DT_MLP_SHAPES(X)
#undef X
  dt_set_error("environment MLP shape (hidden %d, layers %d) is not supported", e.hidden, e.n_layers);
  return DT_ERR_UNSUPPORTED;
}

dt_status mlp_trace_forward(const EnvDev& e, Gen q, const uint32_t* list, const Counters* ctr,
                            int g, int64_t cap, float* rgb, hipStream_t s) {
#define X(H, L) DT_LAUNCH(H, L, k_mlp_trace_fwd, mlp_blocks(cap, H, L), e, q, list, ctr, g, rgb)
  DT_MLP_SHAPES(X)
#undef X
  dt_set_error("environment MLP shape (hidden %d, layers %d) is not supported", e.hidden, e.n_layers);
  return DT_ERR_UNSUPPORTED;
}

int64_t mlp_wgrad_params(const EnvDev& e) {
  return e.hidden == 64 ? 4096 * (int64_t)e.n_layers + 192 + 64 * (int64_t)e.n_layers + 3 : 0;
}

static_assert(MLP_WG_BYTES >= sizeof(float) * MLP_WG_ROWS * Wg<4>::n_params, "run of partial sums");

dt_status mlp_wgrad_reduce(const EnvDev& e, MlpParts part, hipStream_t s) {
  const int64_t np = mlp_wgrad_params(e);
  const int64_t nw = np - 64 * (int64_t)e.n_layers - 3;
  hipLaunchKernelGGL(k_mlp_wg_reduce, dim3((unsigned)((np + 255) / 256)), dim3(256), 0, s, part, np, nw,
                     e.d_w, e.d_b);
  DT_CHECK_LAUNCH();
  return DT_OK;
}

dt_status mlp_trace_backward_wgrad(const EnvDev& e, Gen q, const uint32_t* list, const Counters* ctr,
                                   int g, const float* grad_rgb, Adj cur, MlpParts part, hipStream_t s) {
#define X(L)                                                                                    \
  if (e.hidden == 64 && e.n_layers == L) {                                                      \
    hipLaunchKernelGGL(k_mlp_trace_bwd_wg<L>, dim3(WG_BLOCKS), dim3(WG_T), 0, s, e, q, \
                       list, ctr, g, grad_rgb, cur, part);                                      \
    DT_CHECK_LAUNCH();                                                                          \
    return DT_OK;                                                                               \
  }
  X(1) X(2) X(3) X(4)
#undef X
  dt_set_error("environment MLP weight gradient: hidden width 64 only (got %d)", e.hidden);
  return DT_ERR_UNSUPPORTED;
}

dt_status mlp_trace_backward(const EnvDev& e, Gen q, const uint32_t* list, const Counters* ctr,
                             int g, int64_t cap, const float* grad_rgb, Adj cur, hipStream_t s) {
#define X(H, L) DT_LAUNCH(H, L, k_mlp_trace_bwd, mlp_blocks(cap, H, L), e, q, list, ctr, g, grad_rgb, cur)
  DT_MLP_SHAPES(X)
#undef X
  dt_set_error("environment MLP shape (hidden %d, layers %d) is not supported", e.hidden, e.n_layers);
  return DT_ERR_UNSUPPORTED;
}
