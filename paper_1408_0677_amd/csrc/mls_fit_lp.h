#pragma once
// 16-bit matrix-core MLS fit for gfx950 (Muelder et al., Sec. 3.3): the
// weight x feature contraction on v_mfma_f32_16x16x32_{bf16,f16} with
// float32 accumulation, followed by the float64 per-node solve.
//
// Precision design.  The normal equations amplify relative errors of the
// moments by the conditioning of the weighted basis, and a single 16-bit
// rounding of each feature (8 or 11 significant bits) is far too coarse for
// the quadratic basis.  So
//   - every feature g (moment monomial or basis x attribute) is carried as
//     an S-term expansion g = g_1 + ... + g_S of 16-bit numbers (each term
//     the rounding of what the previous terms left);
//   - the weight is carried as w_hi + w_lo (two terms) when S >= 2;
//   - the contraction issues, per feature tile, w_hi x g_s for every term
//     plus w_lo x g_s for every term but the last, all into one float32
//     accumulator (the products are exact).  What is left out,
//     w_hi g_{>S} and w_lo g_{>=S}, is about 2^-24 (bfloat16, S = 3) or
//     2^-22 (float16, S = 2) of the product for every feature alike.  With
//     w_lo x g_1 alone the product would carry w_lo (g - g_1), an error of
//     2^-16 that differs from feature to feature: the moment matrix and the
//     right-hand sides would no longer see one common weight, and the
//     normal equations amplify such inconsistent errors by their
//     conditioning;
//   - the part of the weight below w_hi + w_lo is common to all features
//     of a pair, so it only perturbs the weight function;
//   - attributes are staged in [-1, 1] (mls_stage.hip) and mapped back.
//
// Work split.  A workgroup owns a 16 x 16 node tile and one slab of
// attributes: the slab's features are the moment monomials plus
// basis x attribute products for its D_s attributes, at most 16 NTS
// columns, so the per-node accumulators fit in registers.  Every slab
// repeats the moments, which lets each slab solve its own nodes.
// Twelve waves: waves 0-7 issue the matrix instructions (each owns 2 row
// strips x NTS feature tiles of 16 x 16 float32), waves 8-11 produce.  Two
// matrix waves per SIMD let one wave build its weight operands while the
// other's MFMAs run.  Points
// stream in chunks of 64 through a three-stage pipeline, one barrier per
// chunk:
//   producers, iteration c:  load the raw chunk c + 2 (coordinates, staged
//                            attributes) from global memory into registers;
//                            turn raw chunk c + 1 (in LDS) into weight
//                            tables and 16-bit feature terms; store raw
//                            chunk c + 2 to LDS
//   MFMA waves, iteration c: build the A operands (weights) from the tables
//                            of chunk c and run its MFMAs
// so the global-memory latency of a chunk is hidden behind a whole chunk of
// matrix work.  The chunks walk the points within reach of the tile's nodes
// only.  With the Wendland weight that is the tile's list of cell-sorted
// points (mls_cells.hip).  With the Gaussian the tile first tests every point
// against its own reach and lists the ones inside in LDS (list_points): a
// point outside carries features that are exactly zero, or weights that round
// to zero (float16) or that no sum can see (bfloat16, in_reach and
// list_adaptive).  The test costs a point 8 bytes of L2 and a few
// instructions per tile, against about 2 us of a compute unit per 64 points
// contracted.  50,000 points, 64 attributes, h = 0.015, 2048^2 (bfloat16, two
// passes): 206.3 ms over all points, 14.2 within 8 h (39 chunks a pass), 9.5
// within the adaptive reach (25), 7.8 with attributes loaded and 7.55 with
// fields stored by 16 bytes.
// There a tile takes 280,000 cycles: 42,000 of listing, 87,000 of pass 1,
// 13,000 of solves, about 125,000 of pass 2, 10,000 of stores; in pass 2 the
// vector instructions of the effective weights and the producers bound it, the
// matrix instructions are a quarter.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <string.h>

#include "mls_internal.h"
#include "mls_list.h"
#include "mls_solve.h"

namespace mls {

struct LPParams {
  const float* pts;       // [n][2] (cell order for the Wendland weight)
  const float* vals;      // staged attributes in [-1, 1]: [n][D] (Gaussian) or
                          // [D][n] in cell order (Wendland)
  const float* shift;     // [D]
  const float* scale;     // [D]
  int64_t n;
  int D, Ds, nslab;
  float inv_h;
  double inv_hd;
  double x0, y0, dx, dy;
  int W, H, tiles_x, tiles;
  double tau, floor_w;
  float cutoff2;          // points with u^2 beyond this get no features
  float reach2;           // ... and their weight rounds to zero (float16) beyond this
                          // squared distance (in h^2) from the tile's nodes
  float list_log;         // ln n + 36 ln 2 (bfloat16: reach_sq)
  float* fields;
  uint8_t* deg_out;
  float* grads;           // [D][2][H][W] or null
  const uint32_t* torder;      // tile of each workgroup slot (Wendland)
  int slots;                   // workgroup slots per attribute slab (Wendland)
  const uint32_t* tile_start;  // per-tile point lists (Wendland): [tiles + 1]
  const uint32_t* tile_list;   //   cell-ordered point indices, or null
};

// Arguments of a served batch (fit_lp_batch_kernel).
struct LPBatch {
  const LPParams* __restrict__ reqs;   // [n_req]
  const uint2* items;          // [n_items] (request, block)
  const uint32_t* total;       // [n_req] items of each request
  uint32_t* head;              // next item (zero at launch)
  uint32_t* done;              // [n_req] finished items (zero at launch)
  uint32_t* skipped;           // [n_req] nonzero once an item was skipped (zero at launch)
  uint32_t* complete;          // [n_req] host: 1 or 2 when a request is done
  const uint32_t* cancel;      // [n_req] host: nonzero = skip the request
  int n_items;
};

// The launches of each kernel family (one source file each).
hipError_t launch_lp_bf16(const LPParams& p, int deg, int nts, int terms, hipStream_t s);
hipError_t launch_lp_fp16(const LPParams& p, int deg, int nts, int terms, hipStream_t s);
hipError_t launch_lp_wend_bf16(const LPParams& p, int deg, int nts, int terms, hipStream_t s);
hipError_t launch_lp_wend_fp16(const LPParams& p, int deg, int nts, int terms, hipStream_t s);
hipError_t launch_shape_bf16(const LPParams& p, int deg, int ntv, int terms, hipStream_t s);
hipError_t launch_shape_fp16(const LPParams& p, int deg, int ntv, int terms, hipStream_t s);
hipError_t launch_batch_bf16(const LPBatch& b, int deg, int nts, int grid, hipStream_t s);
hipError_t launch_batch_fp16(const LPBatch& b, int deg, int nts, int grid, hipStream_t s);
// Batch classes of the two-pass form: kBatchShape + attribute tiles in the
// place of the feature tiles.
constexpr int kBatchShape = 8;

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));

#ifndef MLS_LP_MMA_WAVES
#define MLS_LP_MMA_WAVES 8
#endif
constexpr int kMmaWaves = MLS_LP_MMA_WAVES;
constexpr int kProd = 256;                 // producer threads
constexpr int kThreads = kMmaWaves * 64 + kProd;
constexpr int kCols = 16;
constexpr int R = 16 / kMmaWaves;          // row strips per MFMA wave
constexpr int kRows = kMmaWaves * R;       // 16
constexpr int KT = 64;                     // points per chunk (two MFMA k-steps)
constexpr int KSF = KT + 4;                // float32 table stride (floats)
constexpr int KSH = KT + 8;                // 16-bit feature stride (elements, 144 B)
constexpr int RS = KT + 1;                 // raw chunk row stride (floats): a point's
                                           // attributes are stored down a column without
                                           // bank conflicts
constexpr int kDsCap = 40;                 // attributes per slab at most
constexpr int kLdsBytes = 160 * 1024;
// Points listed at a time (Gaussian, mls_list.h).  A segment ends when the
// next round of tests might not fit.
constexpr int kListCap = 4096;
constexpr int kListB = list_bytes(kListCap);

template <typename T> struct Vec8;
template <> struct Vec8<__bf16> { typedef bf16x8 type; };
template <> struct Vec8<_Float16> { typedef halfx8 type; };

// Two float32 values rounded (nearest-even) to a packed pair of 16-bit
// numbers, first value in the low half: one packed conversion per pair.
template <typename T> __device__ __forceinline__ uint32_t pack2(float a, float b);
template <> __device__ __forceinline__ uint32_t pack2<__bf16>(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2){a, b}, bf16x2));
}
template <> __device__ __forceinline__ uint32_t pack2<_Float16>(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2){a, b}, halfx2));
}

// The same, also returning what the rounding left of each value (exact in
// float32): one term of a multi-term 16-bit expansion.
template <typename T>
__device__ __forceinline__ uint32_t pack2_rest(float a, float b, float& ra, float& rb);
template <>
__device__ __forceinline__ uint32_t pack2_rest<__bf16>(float a, float b, float& ra, float& rb) {
  const uint32_t p = pack2<__bf16>(a, b);
  ra = a - __builtin_bit_cast(float, p << 16);
  rb = b - __builtin_bit_cast(float, p & 0xFFFF0000u);
  return p;
}
template <>
__device__ __forceinline__ uint32_t pack2_rest<_Float16>(float a, float b, float& ra, float& rb) {
  const uint32_t p = pack2<_Float16>(a, b);
  const floatx2 back = __builtin_convertvector(__builtin_bit_cast(halfx2, p), floatx2);
  ra = a - back.x;
  rb = b - back.y;
  return p;
}

// Eight float32 weights as the hi + lo pair of 16-bit operands: hi is the
// rounding of w, lo the rounding of what hi leaves.
template <typename T>
__device__ __forceinline__ void split_weights(const float (&w)[8], typename Vec8<T>::type& hi,
                                              typename Vec8<T>::type& lo) {
  u32x4 h, l;
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    float r0, r1;
    h[p] = pack2_rest<T>(w[2 * p], w[2 * p + 1], r0, r1);
    l[p] = pack2<T>(r0, r1);
  }
  hi = __builtin_bit_cast(typename Vec8<T>::type, h);
  lo = __builtin_bit_cast(typename Vec8<T>::type, l);
}

// Common factor applied to every weight before it is rounded to the 16-bit
// operand.  float16 has a 5-bit exponent: a Gaussian weight below 6e-5
// (r > 3.1 h) would land among its subnormals and lose most of its digits,
// so the fp16 path works with weights times 2^15 (largest 32768, still
// below the format's 65504; weights of r < 5.2 h stay normal).  bfloat16
// shares float32's exponent range and needs no factor.  The solve divides
// the weight sum by the factor before the floor test; the pivots are
// equilibrated and do not see it.
template <typename T> struct WeightGain { static constexpr float value = 1.0f; };
template <> struct WeightGain<_Float16> { static constexpr float value = 32768.0f; };

__device__ __forceinline__ floatx4 mfma16(bf16x8 a, bf16x8 b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ floatx4 mfma16(halfx8 a, halfx8 b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

// A chunk: entries [k, k + kn) of the tile's point list.
struct Chunk {
  int64_t k;
  int kn;
  bool valid;
};

struct Walker {
  int64_t k, kend;
};

// Take the next chunk (invalid once the walk is over).
__device__ __forceinline__ Chunk walker_take(Walker& w) {
  Chunk c;
  c.valid = w.k < w.kend;
  c.k = w.k;
  const int64_t left = w.kend - w.k;
  c.kn = !c.valid ? 0 : (left < KT ? (int)left : KT);
  w.k += c.kn;
  return c;
}

template <int DEG, int NTS, int S, typename T>
struct LPLayout {
  static constexpr int m = DEG == 0 ? 1 : (DEG == 1 ? 3 : 6);
  static constexpr int nmom = DEG == 0 ? 1 : (DEG == 1 ? 6 : 15);
  static constexpr int kFP = NTS * 16;
  static constexpr int kDsFit = (kFP - nmom) / m > 0 ? (kFP - nmom) / m : 0;
  static constexpr int kDsMax = kDsFit < kDsCap ? kDsFit : kDsCap;
  // raw chunk: x[RS], y[RS], v[kDsMax][RS]
  static constexpr int kRawFloats = (2 + kDsMax) * RS;
  static constexpr int kRawIt = ((2 + kDsMax) * KT + kProd - 1) / kProd;
  static constexpr int kFeatB = S * kFP * KSH * 2;            // one feature buffer
  static constexpr int kTabB = (kCols + kRows) * KSF * 4;     // one weight table
  static constexpr int kRawB = kRawFloats * 4;
  static constexpr int kFeat0 = 0;
  static constexpr int kTab0 = kFeat0 + 2 * kFeatB;
  static constexpr int kRaw0 = kTab0 + 2 * kTabB;
  static constexpr int kLoop = kRaw0 + 2 * kRawB;
  static constexpr int kEpiStride = kFP + 1;                  // floats
  static constexpr int kEpi = kMmaWaves * 16 * R * kEpiStride * 4;
  static constexpr int kList0 = ((kLoop > kEpi ? kLoop : kEpi) + 15) / 16 * 16;
  static constexpr int kBytes = kList0 + kListB;
  static_assert(kBytes <= kLdsBytes, "LDS budget");
};

// Offset of node column c0 + col (row r0 + row) from the tile anchor, in
// units of h, computed in float64 from the grid definition.
__device__ __forceinline__ double node_offset_xd(const LPParams& p, int c0, int col, float cxr) {
  return (p.x0 + (double)(c0 + col) * p.dx - (double)cxr) * p.inv_hd;
}
__device__ __forceinline__ double node_offset_yd(const LPParams& p, int r0, int row, float cyr) {
  return (p.y0 + (double)(r0 + row) * p.dy - (double)cyr) * p.inv_hd;
}

// Wendland C2 weight (1 - s)^4 (4 s + 1) for s = r / h < 1, from s^2.  The
// hardware square root (about 1 ulp) replaces the correctly rounded
// sequence, which costs eight more instructions per pair: the weight is
// carried as hi + lo bfloat16 terms, about 17 bits, and any rounding of it
// is common to every feature of the pair.
// 1 - s is clamped at 0 (a clamp bit of the subtraction), which makes the
// weight 0 from s = 1 on.
__device__ __forceinline__ float wendland_c2(float s2) {
  const float s = __builtin_amdgcn_sqrtf(s2);
  const float t = __builtin_amdgcn_fmed3f(1.0f - s, 0.0f, 1.0f);
  const float t2 = t * t;
  return t2 * t2 * (4.0f * s + 1.0f);
}

// The reach of a tile's nodes in the tile frame (units of h): a point adds
// nothing beyond `cut2` from the anchor, nor beyond `reach2` from the
// rectangle [xlo, xhi] x [ylo, yhi] of the nodes.
// With bfloat16, which has float32's range, a second test follows from what
// the sums can see (adaptive reach).  The points beyond R h of every node add
// at most n exp(-R^2) R^(2 DEG) to any node's sum of w b_j^2.  R is chosen so
// that this is 2^-36 of the larger of the weight floor and a lower bound S of
// the tile's weight sums: 4,096 times less than the rounding of float32 sums.
// Every sum leaves out the same points, so the fit is that of the weight cut
// to zero there.  Where a node's smallest diagonal moment is below 2^-12 of
// that scale, so that what is left out could be above 2^-24 of it, the tile is
// summed again without this test.
constexpr float kDiagFloor = 0x1p-12f;

struct TileReach {
  float cxr, cyr, inv_h, cut2, reach2, xlo, xhi, ylo, yhi;
};

__device__ __forceinline__ TileReach tile_reach(const LPParams& p, int c0, int r0, float cxr,
                                                float cyr) {
  const float xa = (float)node_offset_xd(p, c0, 0, cxr);
  const float xb = (float)node_offset_xd(p, c0, kCols - 1, cxr);
  const float ya = (float)node_offset_yd(p, r0, 0, cyr);
  const float yb = (float)node_offset_yd(p, r0, kRows - 1, cyr);
  return TileReach{cxr, cyr, p.inv_h, p.cutoff2, p.reach2, fminf(xa, xb), fmaxf(xa, xb),
                   fminf(ya, yb), fmaxf(ya, yb)};
}

// R^2 for a weight sum of at least S, rounded up to a 64th.
template <int DEG>
__device__ __forceinline__ float reach_sq(float list_log, float scale) {
#pragma clang fp contract(off)
  if (!(scale > 0.0f)) return __builtin_inff();
  const float L = list_log - __logf(scale);
  float r2 = L;
#pragma unroll
  for (int it = 0; it < 4; ++it) r2 = L + (float)DEG * __logf(r2);
  return ceilf(r2 * 64.0f) * 0.015625f;
}

// The weight of a point at its farthest node of the tile.
__device__ __forceinline__ float far_weight(const TileReach& t, float x, float y) {
#pragma clang fp contract(off)
  const float ux = (x - t.cxr) * t.inv_h, uy = (y - t.cyr) * t.inv_h;
  const float ex = fmaxf(fabsf(ux - t.xlo), fabsf(ux - t.xhi));
  const float ey = fmaxf(fabsf(uy - t.ylo), fabsf(uy - t.yhi));
  return __expf(-(ex * ex + ey * ey));
}

// Whether the tile must take the point at (x, y).  The anchor test is the
// one the producers zero features by, with room for its rounding; a
// coordinate that is not finite (or whose square overflows) is kept, since
// such a point makes the sums of every node NaN.
// (Every kernel that lists a request's points must list the same ones, so
// nothing here is left to the compiler's choice of fused operations.)
__device__ __forceinline__ bool in_reach(const TileReach& t, float x, float y) {
#pragma clang fp contract(off)
  const float ux = (x - t.cxr) * t.inv_h, uy = (y - t.cyr) * t.inv_h;
  const float u2 = ux * ux + uy * uy;
  const float ex = fmaxf(fmaxf(t.xlo - ux, ux - t.xhi), 0.0f);
  const float ey = fmaxf(fmaxf(t.ylo - uy, uy - t.yhi), 0.0f);
  return ((u2 <= t.cut2 * 1.0001f) & (ex * ex + ey * ey <= t.reach2)) | !(u2 < __builtin_inff());
}

// The next list of a tile's points with the adaptive reach.  Most points of a
// call are far from a tile, so all are tested against a rectangle only, in the
// points' own coordinates (widened by what their rounding and that of its
// middle can be), and the few listed ones against in_reach.  While the reach
// applies (`cut`), the rectangle is that of the reach that the weight floor
// alone gives; the listed points' weights at the farthest node add up to S,
// and the list is cut to the reach that S gives (S of one list is a lower
// bound as well).  Every kernel that lists a request's points must come to the
// same list.
//
// A call, not inlined: its masks and predicates took registers from the loops
// around it (the quadratic two-pass kernel spilled 81 vector and 112 scalar
// registers with its copies, 22 and 50 without).
struct ListedPoints {
  int cnt, taken;   // entries; points of the input that they were chosen from
  float scale;
};

template <int DEG>
__device__ __noinline__ ListedPoints list_adaptive(const float* points, int64_t n, int64_t at,
                                                   float list_log, float floor_w, TileReach t,
                                                   int cut, LdsBytes lds_list) {
#pragma clang fp contract(off)
  // arguments come in vector registers
  points = uniform(points);
  n = uniform(n);
  at = uniform(at);
  list_log = uniform(list_log);
  floor_w = uniform(floor_w);
  t = uniform(t);
  cut = uniform(cut);
  lds_list = uniform(lds_list);
  float scale = __builtin_inff();
  int64_t pos = at;
  if (cut) t.reach2 = reach_sq<DEG>(list_log, floor_w);
  const float R = __builtin_amdgcn_sqrtf(t.reach2), C = __builtin_amdgcn_sqrtf(t.cut2) * 1.001f;
  const float xm = 0.5f * (t.xlo + t.xhi), ym = 0.5f * (t.ylo + t.yhi);
  const float h = __builtin_amdgcn_rcpf(t.inv_h) * 1.001f;
  const float mx = t.cxr + xm * h, my = t.cyr + ym * h;
  const float bx = (fminf(0.5f * (t.xhi - t.xlo) + R, C + fabsf(xm)) + 0.01f * fabsf(xm)) * h +
                   0x1p-20f * fabsf(mx);
  const float by = (fminf(0.5f * (t.yhi - t.ylo) + R, C + fabsf(ym)) + 0.01f * fabsf(ym)) * h +
                   0x1p-20f * fabsf(my);
  const float far = 1e18f * h;   // short of where a square overflows in units of h
  int cnt = list_points<kThreads, kListCap>(points, n, pos, lds_list, [&](float x, float y) {
    const float ax = fabsf(x - mx), ay = fabsf(y - my);
    return ((ax <= bx) & (ay <= by)) | !(ax + ay < far);
  });
  cnt = refine_list<kThreads, kListCap>(
      points, at, cnt, lds_list, [&](float x, float y) { return far_weight(t, x, y); },
      [&](float x, float y, float S) {
        if (cut) {
          // a NaN (a point that is not finite) leaves the floor
          scale = fmaxf(0.99f * S, floor_w);
          t.reach2 = reach_sq<DEG>(list_log, scale);
        }
        return in_reach(t, x, y);
      });
  return ListedPoints{cnt, (int)(pos - at), scale};
}

// The next list of a tile's points from `pos` on; `scale` keeps the smallest
// scale of the adaptive reach.
template <int DEG, bool ADAPT>
__device__ __forceinline__ int next_points(const LPParams& p, const TileReach& t, bool cut,
                                           int64_t& pos, char* lds_list, float& scale) {
  if constexpr (ADAPT) {
    const ListedPoints l = list_adaptive<DEG>(p.pts, p.n, pos, p.list_log, (float)p.floor_w, t,
                                              cut, (LdsBytes)lds_list);
    pos += __builtin_amdgcn_readfirstlane(l.taken);
    scale = fminf(scale, uniform(l.scale));
    return __builtin_amdgcn_readfirstlane(l.cnt);
  } else {
    return list_points<kThreads, kListCap>(p.pts, p.n, pos, (LdsBytes)lds_list,
                                           [&](float x, float y) { return in_reach(t, x, y); });
  }
}

// Producer: global -> registers for one raw chunk, its attributes
// attribute-major (Wendland, points in cell order).
template <int RAWIT>
__device__ __forceinline__ void raw_load_cells(const LPParams& p, const Chunk& ch, int d0, int Ds,
                                               int pt, float (&r)[RAWIT]) {
#pragma unroll
  for (int it = 0; it < RAWIT; ++it) {
    const int e = pt + it * kProd;
    float v = 0.0f;
    if (ch.valid && e < (2 + Ds) * KT) {
      const int row = e / KT, k = e - row * KT;
      if (k < ch.kn) {
        const int64_t gi = (int64_t)global_ptr(p.tile_list)[ch.k + k];
        if (row == 0) v = global_ptr(p.pts)[2 * gi];
        else if (row == 1) v = global_ptr(p.pts)[2 * gi + 1];
        else v = global_ptr(p.vals)[(int64_t)(d0 + row - 2) * p.n + gi];
      }
    }
    r[it] = v;
  }
}

template <int RAWIT>
__device__ __forceinline__ void raw_store_cells(float* raw, int Ds, int pt,
                                                const float (&r)[RAWIT]) {
#pragma unroll
  for (int it = 0; it < RAWIT; ++it) {
    const int e = pt + it * kProd;
    if (e < (2 + Ds) * KT) raw[(e / KT) * RS + e % KT] = r[it];
  }
}

// The same for listed points (Gaussian), whose attributes are point-major:
// consecutive threads read consecutive attributes of a point, then of the
// next one.  Elements: [0, Ds KT) attribute values (point e / Ds), then KT
// coordinates x, then KT coordinates y.  (k0, d0e) is the thread's first
// element's point and attribute, (ks, ds) the step to its next element's.
struct RowWalk {
  int k0, d0, ks, ds;
};

__device__ __forceinline__ RowWalk row_walk(int pt, int Ds) {
  if (Ds <= 0) return RowWalk{KT, 0, 0, 0};
  const int k0 = pt / Ds, ks = kProd / Ds;
  return RowWalk{k0, pt - k0 * Ds, ks, kProd - ks * Ds};
}

template <int RAWIT>
__device__ __forceinline__ void raw_load_rows(const LPParams& p, const Chunk& ch, int64_t base,
                                              const uint16_t* list, int d0, int Ds,
                                              const RowWalk& rw, int pt, float (&r)[RAWIT],
                                              float& rxy) {
  // the segment's first point is in scalar registers; a listed point's
  // offset from it (at most 65,536 rows of 64 floats) fits 32 bits of bytes
  typedef const __attribute__((address_space(1))) char* Bytes;
  const Bytes pts = (Bytes)(global_ptr(p.pts) + 2 * base);
  const Bytes vals = (Bytes)(global_ptr(p.vals) + base * p.D + d0);
  auto at = [](Bytes b, uint32_t off) {
    return *(const __attribute__((address_space(1))) float*)(b + off);
  };
  const uint16_t* lk = list + ch.k;
  const int kn = ch.kn;
  // KT x and KT y coordinates: the first 2 KT threads
  rxy = 0.0f;
  if (pt < 2 * KT && (pt & (KT - 1)) < kn)
    rxy = at(pts, 8u * lk[pt & (KT - 1)] + (pt >= KT ? 4u : 0u));
  int k = rw.k0, d = rw.d0;
#pragma unroll
  for (int it = 0; it < RAWIT; ++it) {
    float v = 0.0f;
    if (k < kn) v = at(vals, 4u * ((uint32_t)lk[k] * (uint32_t)p.D + (uint32_t)d));
    r[it] = v;
    k += rw.ks;
    d += rw.ds;
    if (d >= Ds) {
      d -= Ds;
      ++k;
    }
  }
}

template <int RAWIT>
__device__ __forceinline__ void raw_store_rows(float* raw, int Ds, const RowWalk& rw, int pt,
                                               const float (&r)[RAWIT], float rxy) {
  if (pt < 2 * KT) raw[(pt / KT) * RS + (pt & (KT - 1))] = rxy;
  int k = rw.k0, d = rw.d0;
#pragma unroll
  for (int it = 0; it < RAWIT; ++it) {
    if (k < KT) raw[(2 + d) * RS + k] = r[it];
    k += rw.ks;
    d += rw.ds;
    if (d >= Ds) {
      d -= Ds;
      ++k;
    }
  }
}

constexpr int kTabIt = (kCols + kRows) * KT / kProd;   // table entries per producer thread

// Node offsets (in h, from the tile anchor) of the table rows a producer
// thread fills: entry it is row (pt + it * kProd) / KT, a node column for
// rows < 16 and a node row after that.
__device__ __forceinline__ void table_offsets(const LPParams& p, int pt, int c0, int r0,
                                              float cxr, float cyr, float (&toff)[kTabIt]) {
#pragma unroll
  for (int it = 0; it < kTabIt; ++it) {
    const int row = (pt + it * kProd) / KT;
    toff[it] = row < kCols ? (float)node_offset_xd(p, c0, row, cxr)
                           : (float)node_offset_yd(p, r0, row - kCols, cyr);
  }
}

// Producer: raw chunk (LDS) -> weight tables and feature terms (LDS).
// Features: a thread owns a pair of consecutive points (pp = pt % 32) and
// one eighth of the features (group g = pt / 32): it forms the monomials of
// its two points once, then writes moment monomials j = g (mod 8) and the
// basis x attribute products of attributes d = g (mod 8), each as S packed
// 16-bit term pairs (one 32-bit LDS store per term).
template <int DEG, int NTS, int S, typename T, bool WEND>
__device__ __forceinline__ void make_chunk(const LPParams& p, const float* raw, int kn, int Ds,
                                           float* tab, T* G, int pt, const float (&toff)[kTabIt],
                                           float cxr, float cyr) {
  using L = LPLayout<DEG, NTS, S, T>;
  constexpr int m = L::m, nmom = L::nmom;
  const float* rx = raw;
  const float* ry = raw + RS;
  const float* rv = raw + 2 * RS;
  // weight tables: 32 rows (16 node columns, 16 node rows) x 64 points.
  // Gaussian: the separable factor exp(-u^2); Wendland: u^2 (combined per
  // pair when the A operand is built).  Points past the chunk: Gaussian 0,
  // Wendland a distance beyond the support.
#pragma unroll
  for (int it = 0; it < kTabIt; ++it) {
    const int e = pt + it * kProd;
    const int k = e & (KT - 1), row = e / KT;
    float v = WEND ? 4.0f : 0.0f;
    if (k < kn) {
      const float u = (row < kCols ? rx[k] - cxr : ry[k] - cyr) * p.inv_h - toff[it];
      // the fp16 weight factor rides on the column table (the weight is gx * gy)
      v = WEND ? u * u : __expf(-u * u) * (row < kCols ? WeightGain<T>::value : 1.0f);
    }
    tab[row * KSF + k] = v;
  }
  // features
  const int pp = pt & 31, g = pt >> 5;
  const int k0 = 2 * pp;
  float mo[2][nmom];
#pragma unroll
  for (int h2 = 0; h2 < 2; ++h2) {
    const float ux = (rx[k0 + h2] - cxr) * p.inv_h;
    const float uy = (ry[k0 + h2] - cyr) * p.inv_h;
    // points beyond the reach of every node of the tile get no features
    const float one = (ux * ux + uy * uy <= p.cutoff2) ? 1.0f : 0.0f;
    mo[h2][0] = one;
    if (nmom > 1) {
      mo[h2][1] = one * ux;
      mo[h2][2] = one * uy;
      mo[h2][3] = mo[h2][1] * ux;
      mo[h2][4] = mo[h2][1] * uy;
      mo[h2][5] = mo[h2][2] * uy;
    }
    if (nmom > 6) {
      mo[h2][6] = mo[h2][3] * ux;
      mo[h2][7] = mo[h2][3] * uy;
      mo[h2][8] = mo[h2][4] * uy;
      mo[h2][9] = mo[h2][5] * uy;
      mo[h2][10] = mo[h2][6] * ux;
      mo[h2][11] = mo[h2][6] * uy;
      mo[h2][12] = mo[h2][7] * uy;
      mo[h2][13] = mo[h2][8] * uy;
      mo[h2][14] = mo[h2][9] * uy;
    }
  }
  auto emit = [&](int j, float v0, float v1) {
    T* dst = G + (size_t)j * KSH + k0;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      uint32_t pr;
      if (s + 1 < S) {
        float r0, r1;
        pr = pack2_rest<T>(v0, v1, r0, r1);
        v0 = r0;
        v1 = r1;
      } else {
        pr = pack2<T>(v0, v1);
      }
      *(uint32_t*)(dst + (size_t)s * L::kFP * KSH) = pr;
    }
  };
#pragma unroll
  for (int j = 0; j < nmom; ++j)
    if ((j & 7) == g) emit(j, mo[0][j], mo[1][j]);
  // basis term bj is monomial bj
  for (int d = g; d < Ds; d += 8) {
    const float a0 = rv[d * RS + k0], a1 = rv[d * RS + k0 + 1];
#pragma unroll
    for (int bj = 0; bj < m; ++bj) emit(nmom + bj * Ds + d, mo[0][bj] * a0, mo[1][bj] * a1);
  }
}

// One node tile and attribute slab of a fit: `block` indexes (slab, tile
// slot) as a launch's workgroup index does.  Every thread of the workgroup
// calls it with the same arguments.
// Adaptive reach (bfloat16, Gaussian): the tile is summed once more without it
// where a node could see past it.  With ONCE that is the caller's to do: `reach_on`
// says whether the reach applies, and the result whether to call again without.
template <int DEG, int NTS, int S, typename T, bool WEND, bool CELLS, bool ONCE = false>
__device__ __forceinline__ bool lp_tile(const LPParams& p, int block, char* lds_lp,
                                        bool reach_on = true) {
  using L = LPLayout<DEG, NTS, S, T>;
  typedef typename Vec8<T>::type vec8;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool mma = wave < kMmaWaves;
  const int pt = tid - kMmaWaves * 64;   // producer thread index
  // with the cell list, p.slots workgroup slots per slab map to tiles
  // through the supertile order; empty slots return before any barrier
  const int per_slab = CELLS ? p.slots : p.tiles;
  const int slab = block / per_slab;
  const uint32_t tile_u = CELLS ? p.torder[block % per_slab] : (uint32_t)(block % per_slab);
  if (tile_u == 0xFFFFFFFFu) return false;
  const int tile = (int)tile_u;
  const int c0 = (tile % p.tiles_x) * kCols;
  const int r0 = (tile / p.tiles_x) * kRows;
  const int d0 = slab * p.Ds;
  const int Ds = min(p.Ds, p.D - d0);
  // tile anchor (rounded to float32; node offsets are taken in this frame)
  const float cxr = (float)(p.x0 + (double)(c0 + kCols / 2) * p.dx);
  const float cyr = (float)(p.y0 + (double)(r0 + kRows / 2) * p.dy);

  // double buffers, selected by chunk parity b
  auto feat = [&](int b) { return (T*)(lds_lp + L::kFeat0 + b * L::kFeatB); };
  auto tab = [&](int b) { return (float*)(lds_lp + L::kTab0 + b * L::kTabB); };
  auto raw = [&](int b) { return (float*)(lds_lp + L::kRaw0 + b * L::kRawB); };

  // The tile's points, a list at a time: the whole cell list (Wendland), or
  // segments of the points in reach (Gaussian).  Matrix and producer waves
  // run separate loops with the same barriers, so that neither holds the
  // other's registers.
  const uint16_t* list = (const uint16_t*)(lds_lp + L::kList0);
  const TileReach reach = CELLS ? TileReach{} : tile_reach(p, c0, r0, cxr, cyr);
  // Adaptive reach: whether it still applies, and the scale it was chosen by.
  constexpr bool ADAPT = !CELLS && __is_same(T, __bf16);
  bool cut = ADAPT && reach_on;
  float scale = __builtin_inff();
  auto next_list = [&](int64_t& pos, Walker& wk) {
    if (CELLS) {
      wk.k = (int64_t)p.tile_start[tile];
      wk.kend = (int64_t)p.tile_start[tile + 1];
      pos = p.n;
    } else {
      wk.k = 0;
      wk.kend = next_points<DEG, ADAPT>(p, reach, cut, pos, lds_lp + L::kList0, scale);
    }
  };
  for (;;) {
  // feature rows past this slab's F are never written: zero them once in
  // both buffers
  {
    const int Fs = L::nmom + L::m * Ds;
    const int pad = (L::kFP - Fs) * KSH;
    for (int b = 0; b < 2; ++b)
      for (int s = 0; s < S; ++s) {
        T* z = feat(b) + ((size_t)s * L::kFP + Fs) * KSH;
        for (int e = tid; e < pad; e += kThreads) z[e] = (T)0.0f;
      }
  }
  // the first list, mostly the only one, by code that all waves share (their
  // own copies of it would each come from the L2 once per tile)
  int64_t base = 0, pos = 0;
  Walker wk;
  next_list(pos, wk);
  floatx4 acc[R][NTS];
  if (mma) {
#pragma unroll
    for (int t = 0; t < R; ++t)
#pragma unroll
      for (int q = 0; q < NTS; ++q) acc[t][q] = floatx4{0.f, 0.f, 0.f, 0.f};
    const int i = lane & 15;
    const int k8 = (lane >> 4) * 8;   // this lane's 8 points of a 32-point k-step
    for (;;) {
      __syncthreads();   // raw 0 and 1
      __syncthreads();   // chunk 0
      int c = 0;
      for (Chunk ch = walker_take(wk); ch.valid; ch = walker_take(wk), ++c) {
        const float* gx = tab(c & 1);
        const float* gy = tab(c & 1) + kCols * KSF;
        const T* G = feat(c & 1);
#pragma unroll
        for (int ks = 0; ks < KT; ks += 32) {
          float wx[8];
#pragma unroll
          for (int q = 0; q < 8; ++q) wx[q] = gx[i * KSF + ks + k8 + q];
          vec8 ahi[R], alo[R];
          float smin = 4.0f;   // Wendland: the smallest u^2 among this lane's pairs
#pragma unroll
          for (int t = 0; t < R; ++t) {
            const float* gyr = gy + (wave * R + t) * KSF + ks + k8;
            float w[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
              if (WEND) {
                const float s2 = wx[q] + gyr[q];
                smin = fminf(smin, s2);
                w[q] = wendland_c2(s2) * WeightGain<T>::value;
              } else {
                w[q] = wx[q] * gyr[q];
              }
            }
            split_weights<T>(w, ahi[t], alo[t]);
          }
          // compact support: a k-step in which no pair of this wave's nodes
          // lies inside the support (all weights zero) adds nothing; its
          // matrix instructions are skipped
          if (WEND && !__any(smin < 1.0f)) continue;
#pragma unroll
          for (int q = 0; q < NTS; ++q) {
#pragma unroll
            for (int s = 0; s < S; ++s) {
              const vec8 b = *(const vec8*)(G + ((size_t)s * L::kFP + q * 16 + i) * KSH + ks + k8);
#pragma unroll
              for (int t = 0; t < R; ++t) acc[t][q] = mfma16(ahi[t], b, acc[t][q]);
              if (s + 1 < S) {
#pragma unroll
                for (int t = 0; t < R; ++t) acc[t][q] = mfma16(alo[t], b, acc[t][q]);
              }
            }
          }
          // each k-step reads and multiplies by itself, the last one before the
          // barrier: the compiler gathers both steps' LDS reads at the top
          // otherwise, so that no matrix instruction runs under their latency, and
          // moves the second step's past the barrier (20,000 points, us before /
          // with this: all in reach, 256^2, float16 quadratic d = 4 695 / 600,
          // constant d = 8 508 / 433, bfloat16 551 / 508; h = 0.05, 512^2, float16
          // 652 / 556 and 475 / 400, bfloat16 591 / 533)
          __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
      }
      if (pos >= p.n) break;
      next_list(pos, wk);
    }
  } else {
    // (made again where the tile is summed again: held over the solve, what
    // follows from the thread's index takes more registers than there are)
    int ptl = pt;
    if (ADAPT && !ONCE) asm volatile("" : "+v"(ptl));
    __builtin_assume(ptl >= 0 && ptl < kProd);
    const int pt = ptl;
    float toff[kTabIt];
    const RowWalk rw = row_walk(pt, Ds);
    bool first = true;
    for (;;) {
      Chunk ch0 = walker_take(wk);
      Chunk ch1 = walker_take(wk);
      float rr[L::kRawIt], rxy = 0.0f;
      auto load = [&](const Chunk& ch) {
        if (CELLS) raw_load_cells(p, ch, d0, Ds, pt, rr);
        else raw_load_rows(p, ch, base, list, d0, Ds, rw, pt, rr, rxy);
      };
      auto store = [&](int b) {
        if (CELLS) raw_store_cells(raw(b), Ds, pt, rr);
        else raw_store_rows(raw(b), Ds, rw, pt, rr, rxy);
      };
      auto make = [&](const Chunk& ch, int b) {
        make_chunk<DEG, NTS, S, T, WEND>(p, raw(b), ch.kn, Ds, tab(b), feat(b), pt, toff, cxr,
                                         cyr);
      };
      // raw 0 and 1 to LDS, then chunk 0's tables and features
      float r1[L::kRawIt], rxy1 = 0.0f;
      load(ch0);
      if (CELLS) raw_load_cells(p, ch1, d0, Ds, pt, r1);
      else raw_load_rows(p, ch1, base, list, d0, Ds, rw, pt, r1, rxy1);
      if (first) table_offsets(p, pt, c0, r0, cxr, cyr, toff);   // loads in flight
      first = false;
      store(0);
      if (CELLS) raw_store_cells(raw(1), Ds, pt, r1);
      else raw_store_rows(raw(1), Ds, rw, pt, r1, rxy1);
      __syncthreads();
      if (ch0.valid) make(ch0, 0);
      __syncthreads();
      for (int c = 0; ch0.valid; ++c) {
        const Chunk ch2 = walker_take(wk);
        load(ch2);      // chunk c + 2, in flight
        if (ch1.valid) make(ch1, (c + 1) & 1);
        store(c & 1);
        __syncthreads();
        ch0 = ch1;
        ch1 = ch2;
      }
      if (pos >= p.n) break;
      base = pos;
      next_list(pos, wk);
    }
  }

  // Epilogue: accumulators -> LDS [wave][node][feature] (float32) -> solve.
  float* epi = (float*)lds_lp;
  if (mma) {
    float* e = epi + wave * 16 * R * L::kEpiStride;
#pragma unroll
    for (int t = 0; t < R; ++t)
#pragma unroll
      for (int q = 0; q < NTS; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          // f32 16x16 MFMA result: lane holds row 4 (lane/16) + r, column lane%16
          const int node = t * 16 + 4 * (lane >> 4) + r;
          const int feat_i = q * 16 + (lane & 15);
          e[node * L::kEpiStride + feat_i] = acc[t][q][r];
        }
  }
  __syncthreads();
  // one node per lane on the first four waves (one per SIMD): the float64
  // solve is issued by four full waves rather than eight half-empty ones
  bool low = false;
  if (tid < kRows * kCols) {
    const int w = tid / (16 * R), local = tid % (16 * R);
    const float* e = epi + (w * 16 * R + local) * L::kEpiStride;
    const int64_t plane = (int64_t)p.W * p.H;
    const int t = local / 16, col = local % 16;
    const int r = r0 + w * R + t, cc = c0 + col;
    if (r < p.H && cc < p.W) {
      const double ex = node_offset_xd(p, c0, col, cxr);
      const double ey = node_offset_yd(p, r0, w * R + t, cyr);
      const int64_t off = (int64_t)r * p.W + cc;
      double diag;
      uint8_t code = solve_node<DEG, float>(e, Ds, ex, ey, p.tau, p.floor_w,
                                            p.fields + (int64_t)d0 * plane + off, plane,
                                            p.shift + d0, p.scale + d0,
                                            (double)WeightGain<T>::value,
                                            p.grads ? p.grads + (int64_t)(2 * d0) * plane + off
                                                    : nullptr,
                                            p.inv_hd, ADAPT ? &diag : nullptr);
      low = ADAPT && diag < (double)(scale * kDiagFloor);
      if (p.deg_out && slab == 0) p.deg_out[off] = code;
    }
  }
  // once more without the adaptive reach where a node could see past it
  if (!ADAPT || !cut) return false;
  if (!__syncthreads_or(low)) return false;
  if (ONCE) return true;
  cut = false;
  }
}

template <int DEG, int NTS, int S, typename T, bool WEND, bool CELLS>
__global__ __launch_bounds__(kThreads) void fit_lp_kernel(LPParams p) {
  extern __shared__ __attribute__((aligned(16))) char lds_lp[];
  (void)lp_tile<DEG, NTS, S, T, WEND, CELLS>(p, blockIdx.x, lds_lp);
}

// ---------------------------------------------------------------------------
// Two-pass (shape-function) form of the same fit with the Gaussian weight.
// The field at node p is
//   field_d(p) = y_p^T R_t,d = sum_i w_ip (y_p^T b_t(u_i)) f_i,d,
// y_p = T'^T M_p'^{-1} e_0 the tile-frame coefficients of the node's shape
// function (mls_solve.h).  Pass 1 contracts the weights with the moment
// monomials only (one 16-column feature tile, S1 terms, split weight) and
// solves every node's ladder for y_p; pass 2 streams the points again and
// contracts the effective weights w_ip (y_p^T b_t(u_i)), formed per pair in
// float32 and split hi + lo, with the attributes (two 16-bit terms each).
// The contraction width falls from n_mom + m D to n_mom + D (399 -> 79 for
// the quadratic basis with 64 attributes); the solve runs once per node and
// attribute slab instead of per feature.  The error stays the float32
// accumulation of the moments in pass 1: the effective weights and the
// attribute terms add about 2^-16 (bfloat16) or 2^-22 (float16) relative per
// pair, which is not amplified by the conditioning, and float16 weighs a pair
// in both passes by the same rounded weight (pair_weight).
//
// float16 needs its range looked after.  The weights carry their gain 2^15
// into pass 1, which leaves y_p 2^-15 of its size.  An effective weight is at
// most sum_j |z_j| c_j, z the node-frame coefficients and c_j the largest |b_j(u)|
// exp(-u^2) of a point that weighs no more than the node's weight sum (at most
// 1), so each node's y_p is scaled by the power of two that brings this bound
// to 2^14 .. 2^15 (shape_scale).  With c_j = 1, the effective weights of nodes
// that only far points determine were as small as the sum below that and lost
// their digits: at sums of 1e-6 to 1e-5 the linear basis with 48 attributes was
// off by 8.1e-4 rms, where one pass is off by 1.2e-4.  The attributes are scaled by 2^10 so
// that the second term of a value near 0 keeps its digits.  The node's power
// and the 2^10 are taken out of the float32 sum at the end, exactly.
//
// The producers run ahead of the solve: while the first four waves turn the
// moments into y_p, they load the first two chunks of pass 2.
// ---------------------------------------------------------------------------

constexpr int kShapeDsCap = 64;    // attributes per workgroup slab
constexpr int kShapeS2 = 2;        // 16-bit terms per attribute value
template <typename T> struct AttrGain { static constexpr float value = 1.0f; };
template <> struct AttrGain<_Float16> { static constexpr float value = 1024.0f; };

template <int DEG, int NTV, int S1>
struct ShapeLayout {
  static constexpr int m = DEG == 1 ? 3 : 6;
  static constexpr int nmom = DEG == 1 ? 6 : 15;
  static constexpr int kRows1 = S1 * 16;                 // pass 1 feature rows
  static constexpr int kRows2 = kShapeS2 * NTV * 16;     // pass 2 feature rows
  static constexpr int kFeatRows = kRows1 > kRows2 ? kRows1 : kRows2;
  static constexpr int kDs = NTV * 16;
  // a raw chunk: coordinates (2 rows of KT), then kDs attributes per point,
  // 16 bytes more a point so that eight lanes' 16 bytes of consecutive points
  // lie in different banks
  static constexpr int kRawRows = 2 * RS + 2;
  static constexpr int kRawStride = kDs + 4;
  static constexpr int kRawFloats = kRawRows + KT * kRawStride;
  static constexpr int kRawIt = kDs / 4 * KT / kProd;    // 16-byte loads a thread
  static constexpr int kFeatB = kFeatRows * KSH * 2;
  static constexpr int kTabB = (kCols + kRows) * KSF * 4;
  static constexpr int kBasB = 3 * KSF * 4;              // 1, u_x, u_y per point
  static constexpr int kRawB = kRawFloats * 4;
  static constexpr int kFeat0 = 0;
  static constexpr int kTab0 = kFeat0 + 2 * kFeatB;
  static constexpr int kBas0 = kTab0 + 2 * kTabB;
  static constexpr int kRaw0 = kBas0 + 2 * kBasB;
  static constexpr int kLoop = kRaw0 + 2 * kRawB;
  // the moments between the passes, apart from the chunk buffers, which the
  // producers fill for pass 2 meanwhile
  static constexpr int kEpiStride = 16 + 1;
  static constexpr int kEpi0 = kLoop;
  static constexpr int kEpiB = kMmaWaves * 16 * R * kEpiStride * 4;
  // per node: the shape coefficients y (float32), the factor that maps its
  // sums back, and the degree code
  static constexpr int kY0 = kEpi0 + kEpiB;
  static constexpr int kScale0 = kY0 + kRows * kCols * m * 4;
  static constexpr int kCode0 = kScale0 + kRows * kCols * 4;
  static constexpr int kList0 = (kCode0 + kRows * kCols + 15) / 16 * 16;
  static constexpr int kBytes = kList0 + kListB;
  static_assert(kBytes <= kLdsBytes, "LDS budget");
  static_assert(kRaw0 % 16 == 0 && kRawB % 16 == 0 && kRawRows % 4 == 0, "16-byte rows");
};

// Producers of pass 2: a raw chunk with its attributes by 16 bytes, global ->
// registers -> LDS, in the order of raw_load_rows with four attributes in the
// place of one (a point's rows are only 4-byte aligned, which a global load
// takes).  A slab's last load may take attributes of the next slab, which
// nothing reads; past the point's own it takes single ones.  Against 4 bytes a
// load, which cost the producers more instructions than the terms: 50,000
// points, 64 attributes, 2048^2 (bfloat16) 9.54 -> 7.79 ms.
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

template <int IT>
__device__ __forceinline__ void quad_load(const LPParams& p, const Chunk& ch, int64_t base,
                                          const uint16_t* list, int d0, int quads,
                                          const RowWalk& rw, int pt, f32x4 (&r)[IT],
                                          float& rxy) {
  typedef const __attribute__((address_space(1))) char* Bytes;
  const Bytes pts = (Bytes)(global_ptr(p.pts) + 2 * base);
  const Bytes vals = (Bytes)(global_ptr(p.vals) + base * p.D + d0);
  auto at = [](Bytes b, uint32_t off) {
    return *(const __attribute__((address_space(1))) float*)(b + off);
  };
  const uint16_t* lk = list + ch.k;
  const int kn = ch.kn, width = p.D - d0;
  rxy = 0.0f;
  if (pt < 2 * KT && (pt & (KT - 1)) < kn)
    rxy = at(pts, 8u * lk[pt & (KT - 1)] + (pt >= KT ? 4u : 0u));
  int k = rw.k0, q = rw.d0;
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
    if (k < kn) {
      const uint32_t off = 4u * ((uint32_t)lk[k] * (uint32_t)p.D + 4u * (uint32_t)q);
      if (4 * q + 4 <= width) {
        v = *(const __attribute__((address_space(1))) f32x4u*)(vals + off);
      } else {
        v[0] = at(vals, off);
        if (4 * q + 1 < width) v[1] = at(vals, off + 4);
        if (4 * q + 2 < width) v[2] = at(vals, off + 8);
      }
    }
    r[it] = v;
    k += rw.ks;
    q += rw.ds;
    if (q >= quads) {
      q -= quads;
      ++k;
    }
  }
}

template <int IT>
__device__ __forceinline__ void quad_store(float* raw, int rows, int stride, int quads,
                                           const RowWalk& rw, int pt, const f32x4 (&r)[IT],
                                           float rxy) {
  if (pt < 2 * KT) raw[(pt / KT) * RS + (pt & (KT - 1))] = rxy;
  int k = rw.k0, q = rw.d0;
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    if (k < KT) *(f32x4*)(raw + rows + k * stride + 4 * q) = r[it];
    k += rw.ks;
    q += rw.ds;
    if (q >= quads) {
      q -= quads;
      ++k;
    }
  }
}

// Producer: the separable Gaussian tables of a chunk (32 rows: 16 node
// columns, then 16 node rows, x 64 points; zero past the chunk).
template <typename T>
__device__ __forceinline__ void gauss_tables(const LPParams& p, const float* raw, int kn,
                                             float* tab, int pt, const float (&toff)[kTabIt],
                                             float cxr, float cyr) {
#pragma unroll
  for (int it = 0; it < kTabIt; ++it) {
    const int e = pt + it * kProd;
    const int k = e & (KT - 1), row = e / KT;
    float v = 0.0f;
    if (k < kn) {
      const float u = (row < kCols ? raw[k] - cxr : raw[RS + k] - cyr) * p.inv_h - toff[it];
      v = __expf(-u * u) * (row < kCols ? WeightGain<T>::value : 1.0f);
    }
    tab[row * KSF + k] = v;
  }
}

// Split two float32 values into `S` 16-bit terms each (each term the
// rounding of what the earlier ones left), written as pairs at rows
// dst + s * stride.
template <int S, typename T>
__device__ __forceinline__ void emit_terms(T* dst, size_t stride, float v0, float v1) {
#pragma unroll
  for (int s = 0; s < S; ++s) {
    uint32_t pr;
    if (s + 1 < S) {
      float r0, r1;
      pr = pack2_rest<T>(v0, v1, r0, r1);
      v0 = r0;
      v1 = r1;
    } else {
      pr = pack2<T>(v0, v1);
    }
    *(uint32_t*)(dst + (size_t)s * stride) = pr;
  }
}

// Monomials u_x^a u_y^b (a + b <= 2 DEG) of a point in the tile frame, in
// mono_index order; zero for points beyond the reach of every node.
template <int DEG>
__device__ __forceinline__ void point_monomials(const LPParams& p, float x, float y, float cxr,
                                                float cyr, float (&mo)[DEG == 1 ? 6 : 15]) {
  const float ux = (x - cxr) * p.inv_h;
  const float uy = (y - cyr) * p.inv_h;
  const float one = (ux * ux + uy * uy <= p.cutoff2) ? 1.0f : 0.0f;
  mo[0] = one;
  mo[1] = one * ux;
  mo[2] = one * uy;
  mo[3] = mo[1] * ux;
  mo[4] = mo[1] * uy;
  mo[5] = mo[2] * uy;
  if (DEG == 2) {
    mo[6] = mo[3] * ux;
    mo[7] = mo[3] * uy;
    mo[8] = mo[4] * uy;
    mo[9] = mo[5] * uy;
    mo[10] = mo[6] * ux;
    mo[11] = mo[6] * uy;
    mo[12] = mo[7] * uy;
    mo[13] = mo[8] * uy;
    mo[14] = mo[9] * uy;
  }
}

// Producer, pass 1: tables and the moment monomials (S1 terms, rows
// s * 16 + j).  Pass 2: tables, the basis values u_x, u_y of the chunk's
// points (float32, rows 1-2 of `bas`; zero past the reach), and the
// attribute terms (rows s * kDs + d), zero past the reach: a point beyond
// every node's reach then adds nothing whatever its effective weight, so
// the matrix lanes need no reach mask of their own.
// A thread owns two consecutive points and one eighth of the rows.
template <int DEG, int NTV, int S1, typename T, bool PASS2>
__device__ __forceinline__ void shape_chunk(const LPParams& p, const float* raw, int kn, int nv,
                                            float* tab, float* bas, T* G, int pt,
                                            const float (&toff)[kTabIt], float cxr,
                                            float cyr) {
  using L = ShapeLayout<DEG, NTV, S1>;
  gauss_tables<T>(p, raw, kn, tab, pt, toff, cxr, cyr);
  const int pp = pt & 31, g = pt >> 5;
  const int k0 = 2 * pp;
  float mo0[L::nmom], mo1[L::nmom];
  point_monomials<DEG>(p, raw[k0], raw[RS + k0], cxr, cyr, mo0);
  point_monomials<DEG>(p, raw[k0 + 1], raw[RS + k0 + 1], cxr, cyr, mo1);
  if (!PASS2) {
#pragma unroll
    for (int j = 0; j < L::nmom; ++j)
      if ((j & 7) == g)
        emit_terms<S1, T>(G + (size_t)j * KSH + k0, (size_t)16 * KSH, mo0[j], mo1[j]);
    return;
  }
#pragma unroll
  for (int j = 1; j < 3; ++j)   // u_x, u_y (the matrix waves form the rest)
    if ((j & 7) == g) {
      bas[j * KSF + k0] = mo0[j];
      bas[j * KSF + k0 + 1] = mo1[j];
    }
  const float* r0 = raw + L::kRawRows + k0 * L::kRawStride;
  const float a0 = mo0[0] * AttrGain<T>::value, a1 = mo1[0] * AttrGain<T>::value;
  for (int d = 4 * g; d < nv; d += 32) {   // four attributes at a time
    const f32x4 v0 = *(const f32x4*)(r0 + d), v1 = *(const f32x4*)(r0 + L::kRawStride + d);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (d + j < nv)
        emit_terms<kShapeS2, T>(G + (size_t)(d + j) * KSH + k0, (size_t)L::kDs * KSH, a0 * v0[j],
                                a1 * v1[j]);
  }
}

// A pair's weight as pass 1 saw it.  Its hi + lo terms in float16 end at 2^-24,
// the format's smallest number, and the moments and the products have to see
// the same weight (the top of this file), so it is rounded to that here as
// well: below 0.5 the sum with 0.5 ends at 2^-24, above it at about the digits
// of hi + lo.  One instruction per pair: 7,351 points, 19 attributes,
// 701 x 643 545 -> 548 us.
template <typename T>
__device__ __forceinline__ float pair_weight(float gx, float gy) {
  if constexpr (__is_same(T, _Float16)) return fmaf(gx, gy, 0.5f) - 0.5f;
  return gx * gy;
}

// The power of two that brings an effective weight's bound, `b`, to 2^14 ..
// 2^15 (float16; at most 2^+-100), 1 for bfloat16.
template <typename T>
__device__ __forceinline__ float shape_scale(double b) {
  if constexpr (__is_same(T, _Float16)) {
    int e;
    (void)frexp(b, &e);              // b < 2^e
    e = 15 - e;
    e = e > 100 ? 100 : (e < -100 ? -100 : e);
    return b > 0.0 && b < __builtin_inf() ? ldexpf(1.0f, e) : 1.0f;
  } else {
    return 1.0f;
  }
}

// One node tile and attribute slab: `block` indexes (slab, tile) as a launch's
// workgroup index does.  Every thread of the workgroup calls it with the same
// arguments.
template <int DEG, int NTV, int S1, typename T>
__device__ __forceinline__ void shape_tile(const LPParams& p, int block, char* lds_sh) {
  using L = ShapeLayout<DEG, NTV, S1>;
  typedef typename Vec8<T>::type vec8;
  constexpr int m = L::m;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool mma = wave < kMmaWaves;
  const int pt = tid - kMmaWaves * 64;
  const int slab = block / p.tiles;
  const int tile = block % p.tiles;
  const int c0 = (tile % p.tiles_x) * kCols;
  const int r0 = (tile / p.tiles_x) * kRows;
  const int d0 = slab * p.Ds;
  const int nv = min(p.Ds, p.D - d0);
  const float cxr = (float)(p.x0 + (double)(c0 + kCols / 2) * p.dx);
  const float cyr = (float)(p.y0 + (double)(r0 + kRows / 2) * p.dy);

  auto feat = [&](int b) { return (T*)(lds_sh + L::kFeat0 + b * L::kFeatB); };
  auto tab = [&](int b) { return (float*)(lds_sh + L::kTab0 + b * L::kTabB); };
  auto bas = [&](int b) { return (float*)(lds_sh + L::kBas0 + b * L::kBasB); };
  auto raw = [&](int b) { return (float*)(lds_sh + L::kRaw0 + b * L::kRawB); };
  float* epi = (float*)(lds_sh + L::kEpi0);
  float* ybuf = (float*)(lds_sh + L::kY0);
  float* back = (float*)(lds_sh + L::kScale0);
  uint8_t* codes = (uint8_t*)(lds_sh + L::kCode0);

  const int i = lane & 15;
  const int k8 = (lane >> 4) * 8;
  const int64_t plane = (int64_t)p.W * p.H;

  // The points in reach, a list at a time; `kept` is the last list, which
  // pass 2 uses again if it was the only one.
  constexpr bool ADAPT = __is_same(T, __bf16);
  // Whether a k-step's instructions stay together, as in the one-pass form:
  // float16 only (7,351 points, 19 attributes, 701 x 643, us without / with 550 /
  // 530; bfloat16, 50,000 points, 64 attributes, 2048^2, 7,558 / 7,791).
  constexpr bool kFence = __is_same(T, _Float16);
  const uint16_t* list = (const uint16_t*)(lds_sh + L::kList0);
  const TileReach reach = tile_reach(p, c0, r0, cxr, cyr);
  bool cut = ADAPT;   // the adaptive reach applies
  float scale = __builtin_inff();
  int kept = 0, segments = 0;
  auto next_list = [&](int64_t& pos) {
    return next_points<DEG, ADAPT>(p, reach, cut, pos, lds_sh + L::kList0, scale);
  };
  // rows of a chunk's 16-bit terms that are never written: zero in both buffers
  auto zero_rows = [&](int rows, int stride, int terms, int t, int threads) {
    for (int b = 0; b < 2; ++b)
      for (int s = 0; s < terms; ++s) {
        T* z = feat(b) + ((size_t)s * stride + rows) * KSH;
        for (int e = t; e < (stride - rows) * KSH; e += threads) z[e] = (T)0.0f;
      }
  };
  // producers: a chunk's loads, its tables and terms
  const RowWalk rw1 = row_walk(pt, 0);
  const int quads = (nv + 3) / 4;   // a point's 16-byte loads
  float toff[kTabIt];
  auto make1 = [&](const Chunk& ch, int b) {
    shape_chunk<DEG, NTV, S1, T, false>(p, raw(b), ch.kn, 0, tab(b), bas(b), feat(b), pt, toff,
                                        cxr, cyr);
  };
  auto make2 = [&](const Chunk& ch, int b) {
    shape_chunk<DEG, NTV, S1, T, true>(p, raw(b), ch.kn, nv, tab(b), bas(b), feat(b), pt, toff,
                                       cxr, cyr);
  };
  // the first two raw chunks of a list at `base` to LDS, then chunk 0's tables
  // and terms once the producers' stores are visible (`sync`)
  auto load2 = [&](int64_t base, const Chunk& ch0, const Chunk& ch1) {
    f32x4 ra[L::kRawIt], rb[L::kRawIt];
    float xa = 0.0f, xb = 0.0f;
    // (the walk's steps made here: held over pass 1 and its solve, they spill)
    RowWalk rw2 = row_walk(pt, quads);
    asm volatile("" : "+v"(rw2.k0), "+v"(rw2.d0));
    quad_load(p, ch0, base, list, d0, quads, rw2, pt, ra, xa);
    quad_load(p, ch1, base, list, d0, quads, rw2, pt, rb, xb);
    quad_store(raw(0), L::kRawRows, L::kRawStride, quads, rw2, pt, ra, xa);
    quad_store(raw(1), L::kRawRows, L::kRawStride, quads, rw2, pt, rb, xb);
  };

  // ---- pass 1: moments, then the ladder and the shape coefficients ----
  // Once within the adaptive reach; once more without it where a node could
  // see past it.
  for (;;) {
    zero_rows(L::nmom, 16, S1, tid, kThreads);
    floatx4 acc[R];
    // the first list, mostly the only one, by code that all waves share
    // (their own copies of it would each come from the L2 once per tile)
    int64_t base = 0, pos = 0;
    kept = next_list(pos);
    segments = 1;
    if (mma) {
#pragma unroll
      for (int t = 0; t < R; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
      for (;;) {
        __syncthreads();   // raw 0 and 1
        __syncthreads();   // chunk 0
        Walker wk{0, kept};
        int c = 0;
        for (Chunk ch = walker_take(wk); ch.valid; ch = walker_take(wk), ++c) {
          const float* gx = tab(c & 1);
          const float* gy = tab(c & 1) + kCols * KSF;
          const T* G = feat(c & 1);
#pragma unroll
          for (int ks = 0; ks < KT; ks += 32) {
            float wx[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) wx[q] = gx[i * KSF + ks + k8 + q];
            vec8 ahi[R], alo[R];
#pragma unroll
            for (int t = 0; t < R; ++t) {
              const float* gyr = gy + (wave * R + t) * KSF + ks + k8;
              float w[8];
#pragma unroll
              for (int q = 0; q < 8; ++q) w[q] = wx[q] * gyr[q];
              split_weights<T>(w, ahi[t], alo[t]);
            }
#pragma unroll
            for (int s = 0; s < S1; ++s) {
              const vec8 b = *(const vec8*)(G + ((size_t)s * 16 + i) * KSH + ks + k8);
#pragma unroll
              for (int t = 0; t < R; ++t) acc[t] = mfma16(ahi[t], b, acc[t]);
              if (s + 1 < S1) {
#pragma unroll
                for (int t = 0; t < R; ++t) acc[t] = mfma16(alo[t], b, acc[t]);
              }
            }
            if (kFence) __builtin_amdgcn_sched_barrier(0);
          }
          __syncthreads();
        }
        if (pos >= p.n) break;
        kept = next_list(pos);
        ++segments;
      }
      // moments -> LDS [wave][node][monomial]
      float* e = epi + wave * 16 * R * L::kEpiStride;
#pragma unroll
      for (int t = 0; t < R; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          e[(t * 16 + 4 * (lane >> 4) + r) * L::kEpiStride + (lane & 15)] = acc[t][r];
    } else {
      for (;;) {
        Walker wk{0, kept};
        Chunk ch0 = walker_take(wk);
        Chunk ch1 = walker_take(wk);
        float rr[1], rxy = 0.0f, rxy1 = 0.0f;   // coordinates only
        raw_load_rows(p, ch0, base, list, d0, 0, rw1, pt, rr, rxy);
        raw_load_rows(p, ch1, base, list, d0, 0, rw1, pt, rr, rxy1);
        if (segments == 1) {   // loads in flight
          int ptl = pt;
          if (ADAPT) asm volatile("" : "+v"(ptl));
          __builtin_assume(ptl >= 0 && ptl < kProd);
          table_offsets(p, ptl, c0, r0, cxr, cyr, toff);
        }
        raw_store_rows(raw(0), 0, rw1, pt, rr, rxy);
        raw_store_rows(raw(1), 0, rw1, pt, rr, rxy1);
        __syncthreads();
        if (ch0.valid) make1(ch0, 0);
        __syncthreads();
        for (int c = 0; ch0.valid; ++c) {
          const Chunk ch2 = walker_take(wk);
          raw_load_rows(p, ch2, base, list, d0, 0, rw1, pt, rr, rxy);
          if (ch1.valid) make1(ch1, (c + 1) & 1);
          raw_store_rows(raw(c & 1), 0, rw1, pt, rr, rxy);
          __syncthreads();
          ch0 = ch1;
          ch1 = ch2;
        }
        if (pos >= p.n) break;
        base = pos;
        kept = next_list(pos);
        ++segments;
      }
    }
    __syncthreads();
    // one node per lane on the first four waves (one per SIMD)
    bool low = false;
    if (tid < kRows * kCols) {
      const int w = tid / (16 * R), local = tid % (16 * R);
      const float* e = epi + (w * 16 * R + local) * L::kEpiStride;
      const int t = local / 16, col = local % 16;
      const int row = w * R + t;
      const double ex = node_offset_xd(p, c0, col, cxr);
      const double ey = node_offset_yd(p, r0, row, cyr);
      Ladder<DEG> lad;
      const int code = ladder_solve<DEG>(e, ex, ey, p.tau, p.floor_w,
                                         (double)WeightGain<T>::value, lad);
      const bool in = r0 + row < p.H && c0 + col < p.W;
      low = ADAPT && in && code != 255 && lad.diag < (double)(scale * kDiagFloor);
      float g = 1.0f;
      if (__is_same(T, _Float16) && code != 255) {
        // z = S w in the node's frame, times the weights' gain.  No point weighs
        // more than the sum, so for sums below 1/e the largest |b_j| exp(-u^2)
        // is that at u^2 = -ln sum
        const float sum = e[0] * (1.0f / WeightGain<T>::value);
        const float u2 = fmaxf(1.0f, -__logf(sum)), most = fminf(1.0f, sum * 1.01f);
        double b = 0.0;
#pragma unroll
        for (int j = 0; j < m; ++j) {
          const float size = j == 0 ? 1.0f : (j < 3 ? __builtin_amdgcn_sqrtf(u2) : u2);
          if (j < lad.mk) b += fabs(lad.s[j] * lad.w[j]) * (double)fminf(1.0f, most * size);
        }
        g = shape_scale<T>(b * (double)WeightGain<T>::value);
      }
      float* yv = ybuf + (row * kCols + col) * m;
#pragma unroll
      for (int j = 0; j < m; ++j)
        yv[j] = code == 255 ? 0.0f : (float)(lad.y[j] * (double)g);
      back[row * kCols + col] = 1.0f / (g * AttrGain<T>::value);
      codes[row * kCols + col] = (uint8_t)code;
      if (p.deg_out && slab == 0 && in)
        p.deg_out[(int64_t)(r0 + row) * p.W + c0 + col] = (uint8_t)code;
    } else if (!mma && segments == 1) {
      // the list is still there: pass 2's first chunks to LDS meanwhile
      Walker wk{0, kept};
      const Chunk ch0 = walker_take(wk), ch1 = walker_take(wk);
      load2(0, ch0, ch1);
    }
    const bool redo = ADAPT && cut && __syncthreads_or(low);
    if (!(ADAPT && cut)) __syncthreads();
    if (!redo) break;
    cut = false;
  }

  // ---- pass 2: effective weights x attribute terms ----
  floatx4 acc[R][NTV];
  int64_t base = 0, pos = segments == 1 ? p.n : 0;
  if (segments > 1) kept = next_list(pos);
  if (mma) {
#pragma unroll
    for (int t = 0; t < R; ++t)
#pragma unroll
      for (int q = 0; q < NTV; ++q) acc[t][q] = floatx4{0.f, 0.f, 0.f, 0.f};
    // the shape coefficients of this lane's nodes (column i of its strips)
    float yv[R][m];
#pragma unroll
    for (int t = 0; t < R; ++t)
#pragma unroll
      for (int j = 0; j < m; ++j) yv[t][j] = ybuf[((wave * R + t) * kCols + i) * m + j];
    for (;;) {
      // (with one list its raw chunks 0 and 1 are in LDS)
      if (segments > 1) __syncthreads();   // raw 0 and 1
      __syncthreads();                     // chunk 0
      Walker wk{0, kept};
      int c = 0;
      for (Chunk ch = walker_take(wk); ch.valid; ch = walker_take(wk), ++c) {
        const float* gx = tab(c & 1);
        const float* gy = tab(c & 1) + kCols * KSF;
        const float* bs = bas(c & 1);
        const T* G = feat(c & 1);
#pragma unroll
        for (int ks = 0; ks < KT; ks += 32) {
          vec8 ahi[R], alo[R];
          u32x4 hv[R], lv[R];
          // two points at a time: their basis values and column factors,
          // then the effective weight of each of the lane's nodes, split
          // hi + lo with one packed conversion per pair
#pragma unroll
          for (int q = 0; q < 8; q += 2) {
            float w[R][2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
              const int k = ks + k8 + q + e;
              // b = (1, u_x, u_y[, u_x^2, u_x u_y, u_y^2]): the quadratic
              // terms follow from the linear ones (Horner), so a point
              // needs two values, not five (past the reach its attribute
              // terms are zero)
              const float b1 = bs[KSF + k], b2 = bs[2 * KSF + k];
              const float wxq = gx[i * KSF + k];
#pragma unroll
              for (int t = 0; t < R; ++t) {
                float sh;
                if constexpr (DEG == 1) {
                  sh = fmaf(yv[t][2], b2, fmaf(yv[t][1], b1, yv[t][0]));
                } else {
                  const float s1 = fmaf(yv[t][3], b1, fmaf(yv[t][4], b2, yv[t][1]));
                  const float s2 = fmaf(yv[t][5], b2, yv[t][2]);
                  sh = fmaf(b1, s1, fmaf(b2, s2, yv[t][0]));
                }
                w[t][e] = pair_weight<T>(wxq, gy[(wave * R + t) * KSF + k]) * sh;
              }
            }
#pragma unroll
            for (int t = 0; t < R; ++t) {
              float r0, r1;
              hv[t][q / 2] = pack2_rest<T>(w[t][0], w[t][1], r0, r1);
              lv[t][q / 2] = pack2<T>(r0, r1);
            }
          }
#pragma unroll
          for (int t = 0; t < R; ++t) {
            ahi[t] = __builtin_bit_cast(vec8, hv[t]);
            alo[t] = __builtin_bit_cast(vec8, lv[t]);
          }
#pragma unroll
          for (int q = 0; q < NTV; ++q) {
            const vec8 b1 = *(const vec8*)(G + ((size_t)q * 16 + i) * KSH + ks + k8);
            const vec8 b2 = *(const vec8*)(G + ((size_t)L::kDs + q * 16 + i) * KSH + ks + k8);
#pragma unroll
            for (int t = 0; t < R; ++t) {
              acc[t][q] = mfma16(ahi[t], b1, acc[t][q]);
              acc[t][q] = mfma16(alo[t], b1, acc[t][q]);
              acc[t][q] = mfma16(ahi[t], b2, acc[t][q]);
            }
          }
          if (kFence) __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
      }
      if (pos >= p.n) break;
      kept = next_list(pos);
    }
  } else {
    zero_rows(nv, L::kDs, kShapeS2, pt, kProd);
    const RowWalk rw2 = row_walk(pt, quads);
    for (;;) {
      Walker wk{0, kept};
      Chunk ch0 = walker_take(wk);
      Chunk ch1 = walker_take(wk);
      if (segments > 1) {
        load2(base, ch0, ch1);
        __syncthreads();
      }
      if (ch0.valid) make2(ch0, 0);
      __syncthreads();
      f32x4 rr[L::kRawIt];
      float rxy = 0.0f;
      for (int c = 0; ch0.valid; ++c) {
        const Chunk ch2 = walker_take(wk);
        quad_load(p, ch2, base, list, d0, quads, rw2, pt, rr, rxy);
        if (ch1.valid) make2(ch1, (c + 1) & 1);
        quad_store(raw(c & 1), L::kRawRows, L::kRawStride, quads, rw2, pt, rr, rxy);
        __syncthreads();
        ch0 = ch1;
        ch1 = ch2;
      }
      if (pos >= p.n) break;
      base = pos;
      kept = next_list(pos);
    }
  }
  // fields: the accumulators are the normalised values times the node's
  // scale; lane holds node columns 4 (lane / 16) + r of strip t for attribute
  // q * 16 + lane % 16
  if (mma) {
    // four columns a store where every row of every plane is 16-byte aligned
    // (64 attributes, 2048^2: 7.80 -> 7.55 ms)
    const bool wide = (p.W & 3) == 0 && ((uintptr_t)p.fields & 15) == 0;
#pragma unroll
    for (int q = 0; q < NTV; ++q) {
      const int dd = q * 16 + (lane & 15);
      if (dd >= nv) continue;
      const double sh = (double)p.shift[d0 + dd], sc = (double)p.scale[d0 + dd];
      float* fd = p.fields + (int64_t)(d0 + dd) * plane;
#pragma unroll
      for (int t = 0; t < R; ++t) {
        const int row = wave * R + t, rg = r0 + row;
        if (rg >= p.H) continue;
        const int cg = c0 + 4 * (lane >> 4);
        f32x4 v;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int node = row * kCols + 4 * (lane >> 4) + r;
          const bool und = codes[node] == 255;
          v[r] = und ? __builtin_nanf("")
                     : (float)(sh + sc * ((double)acc[t][q][r] * (double)back[node]));
        }
        float* out = fd + (int64_t)rg * p.W + cg;
        if (wide) {
          if (cg < p.W) *(f32x4*)out = v;   // W is a multiple of four
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (cg + r < p.W) out[r] = v[r];
        }
      }
    }
  }
}

template <int DEG, int NTV, int S1, typename T>
__global__ __launch_bounds__(kThreads) void fit_shape_kernel(LPParams p) {
  extern __shared__ __attribute__((aligned(16))) char lds_sh[];
  shape_tile<DEG, NTV, S1, T>(p, blockIdx.x, lds_sh);
}

template <int DEG, int NTV, int S1, typename T>
hipError_t launch_shape_impl(const LPParams& p, hipStream_t s) {
  using L = ShapeLayout<DEG, NTV, S1>;
  const size_t lds = (size_t)L::kBytes;
  const void* fn = (const void*)fit_shape_kernel<DEG, NTV, S1, T>;
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  const int64_t blocks = (int64_t)p.tiles * p.nslab;
  hipLaunchKernelGGL((fit_shape_kernel<DEG, NTV, S1, T>), dim3((unsigned)blocks), dim3(kThreads),
                     lds, s, p);
  return hipGetLastError();
}

template <int DEG, int S1, typename T>
hipError_t launch_shape_ntv(const LPParams& p, int ntv, hipStream_t s) {
  switch (ntv) {
    case 1: return launch_shape_impl<DEG, 1, S1, T>(p, s);
    case 2: return launch_shape_impl<DEG, 2, S1, T>(p, s);
    case 3: return launch_shape_impl<DEG, 3, S1, T>(p, s);
    default: return launch_shape_impl<DEG, 4, S1, T>(p, s);
  }
}

template <int S1, typename T>
hipError_t launch_shape_deg(const LPParams& p, int deg, int ntv, hipStream_t s) {
  return deg == 1 ? launch_shape_ntv<1, S1, T>(p, ntv, s) : launch_shape_ntv<2, S1, T>(p, ntv, s);
}

template <typename T>
hipError_t launch_shape_terms(const LPParams& p, int deg, int ntv, int terms, hipStream_t s) {
  switch (terms) {
    case 1: return launch_shape_deg<1, T>(p, deg, ntv, s);
    case 2: return launch_shape_deg<2, T>(p, deg, ntv, s);
    default: return launch_shape_deg<3, T>(p, deg, ntv, s);
  }
}

// Persistent batch of served fits sharing one kernel shape: every
// workgroup takes (request, block) work items from a device counter until
// the list is exhausted (every workgroup reaches the end of the list, so the
// grid drains).  Before an item the request's cancel flag (host memory) is
// read; a cancelled request's items are counted but not computed, and the
// request is marked as skipped.  Items are listed request by request, so a
// workgroup meets each request in one run of items; when it moves on to the
// next request (or the list ends) it releases its output writes at device
// scope and adds the run's length to the request's count.  The workgroup
// whose addition completes a request acquires the other additions and sets
// the request's completion flag in host memory (1: every item computed, 2:
// items skipped) with a system-scope release, so the host sees each request
// finish, its outputs written, while the batch runs on.  (A release per
// item would write back the L2 after every tile, and costs about a tenth of
// the batch's time.)

// The tile body as a call of its own in the batch kernel, so that its
// registers are allocated apart from the item loop's.  Arguments of a call
// travel in vector registers and read as per-lane values; the parameter
// address and the block are made scalar again here, so that the parameters
// are loaded through the scalar cache as kernel arguments are, and the
// work area is named as the dynamic LDS array itself, so that its accesses
// are LDS instructions rather than flat ones.
// SHAPE: the two-pass form, NTS attribute tiles.  The one-pass form's second run
// without the adaptive reach is a call as well (`reach_on`, result as lp_tile's):
// a loop around the tile makes values of the first run live over its solve, 34 to
// 149 spilled registers of the quadratic basis (six requests of 2,000 points, 24
// attributes, 300^2, bfloat16 1,152 -> 1,075 us).  A direct launch, whose tile is not
// a call otherwise, lost 4 to 10% by it.
template <int DEG, int NTS, int S, typename T, bool SHAPE>
__device__ __noinline__ int lp_tile_item(const LPParams* __restrict__ pp, int block,
                                         int reach_on) {
  extern __shared__ __attribute__((aligned(16))) char lds_lp[];
  // the parameter block is written before the launch and only read by the
  // kernel: in the constant address space its loads are scalar loads that
  // the compiler may repeat instead of holding their values in registers
  const uint64_t a = (uint64_t)(uintptr_t)pp;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
  typedef const __attribute__((address_space(4))) LPParams* ConstParams;
  const ConstParams pc = (ConstParams)(uintptr_t)(((uint64_t)hi << 32) | lo);
  if constexpr (SHAPE) {
    shape_tile<DEG, NTS, S, T>(*(const LPParams*)pc, __builtin_amdgcn_readfirstlane(block),
                               lds_lp);
    return 0;
  } else {
    return lp_tile<DEG, NTS, S, T, false, false, true>(
        *(const LPParams*)pc, __builtin_amdgcn_readfirstlane(block), lds_lp,
        __builtin_amdgcn_readfirstlane(reach_on) != 0);
  }
}

// Thread 0 takes the next item in a branch at the top of the loop; it
// counts a finished run of items in a second branch, under a condition held
// in scalar registers, and every path from there back to the top of the
// loop passes a barrier.  (With only the back edge between two thread-0
// branches the compiler threads the path of the other threads from the
// last barrier straight to the first, and the loop it builds from that runs
// their path until they leave it, which they never do: no item is taken
// without thread 0.)
template <int DEG, int NTS, int S, typename T, bool SHAPE>
__global__ __launch_bounds__(kThreads) void fit_lp_batch_kernel(LPBatch b) {
  __shared__ int sh_item, sh_skip;
  int cur_req = -1;       // request of the current run of items
  uint32_t cur_cnt = 0;   // items of the run finished here, not yet counted
  for (;;) {
    if (threadIdx.x == 0) {
      const int it = (int)atomicAdd(b.head, 1u);
      int skip = 0;
      if (it < b.n_items) {
        const uint32_t r = b.items[it].x;
        skip = __hip_atomic_load(b.cancel + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) != 0;
        // released with the run's count
        if (skip) __hip_atomic_store(b.skipped + r, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      sh_item = it;
      sh_skip = skip;
    }
    __syncthreads();
    const int item = __builtin_amdgcn_readfirstlane(sh_item);
    const int skip = __builtin_amdgcn_readfirstlane(sh_skip);
    __syncthreads();
    const bool more = item < b.n_items;
    const uint2 w = more ? b.items[item] : make_uint2(0xFFFFFFFFu, 0u);
    const int req = __builtin_amdgcn_readfirstlane((int)w.x);   // -1 past the end
    const int block = __builtin_amdgcn_readfirstlane((int)w.y);
    if (cur_cnt > 0 && req != cur_req) {
      // the run of cur_req ends here: release its output writes, count it
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      __syncthreads();
      if (threadIdx.x == 0) {
        const uint32_t prev = atomicAdd(b.done + cur_req, cur_cnt);
        if (prev + cur_cnt == b.total[cur_req]) {
          // every item of the request is counted: acquire the other runs'
          // releases (and skip marks), then publish to the host
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
          const uint32_t sk = __hip_atomic_load(b.skipped + cur_req, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_store(b.complete + cur_req, sk ? 2u : 1u, __ATOMIC_RELEASE,
                             __HIP_MEMORY_SCOPE_SYSTEM);
        }
      }
      cur_cnt = 0;
    }
    if (!more) break;
    cur_req = req;
    if (!skip) {
      // read in place (uniform, read-only): fields are loaded where used,
      // as kernel arguments are, instead of held in registers
      const int again = lp_tile_item<DEG, NTS, S, T, SHAPE>(b.reqs + req, block, 1);
      if (!SHAPE && __is_same(T, __bf16) && __builtin_amdgcn_readfirstlane(again))
        (void)lp_tile_item<DEG, NTS, S, T, SHAPE>(b.reqs + req, block, 0);
    }
    ++cur_cnt;
    __syncthreads();
  }
}

template <int DEG, int NTS, int S, typename T, bool WEND>
hipError_t launch_lp_impl(LPParams p, hipStream_t s) {
  using L = LPLayout<DEG, NTS, S, T>;
  const size_t lds = (size_t)L::kBytes;
  // Wendland weights walk the cell list; the Gaussian lists its own points
  const void* fn = (const void*)fit_lp_kernel<DEG, NTS, S, T, WEND, WEND>;
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  const int64_t blocks = (int64_t)(WEND ? p.slots : p.tiles) * p.nslab;
  hipLaunchKernelGGL((fit_lp_kernel<DEG, NTS, S, T, WEND, WEND>), dim3((unsigned)blocks),
                     dim3(kThreads), lds, s, p);
  return hipGetLastError();
}

template <int DEG, int S, typename T, bool WEND>
hipError_t launch_lp_nts(const LPParams& p, int nts, hipStream_t s) {
  switch (nts) {
    case 1: return launch_lp_impl<DEG, 1, S, T, WEND>(p, s);
    case 2: return launch_lp_impl<DEG, 2, S, T, WEND>(p, s);
    case 3: return launch_lp_impl<DEG, 3, S, T, WEND>(p, s);
    case 4: return launch_lp_impl<DEG, 4, S, T, WEND>(p, s);
    case 5: return launch_lp_impl<DEG, 5, S, T, WEND>(p, s);
    case 6: return launch_lp_impl<DEG, 6, S, T, WEND>(p, s);
    case 7: return launch_lp_impl<DEG, 7, S, T, WEND>(p, s);
    default: return launch_lp_impl<DEG, 8, S, T, WEND>(p, s);
  }
}

template <int S, typename T, bool WEND>
hipError_t launch_lp_deg(const LPParams& p, int deg, int nts, hipStream_t s) {
  switch (deg) {
    case 0: return launch_lp_nts<0, S, T, WEND>(p, nts, s);
    case 1: return launch_lp_nts<1, S, T, WEND>(p, nts, s);
    default: return launch_lp_nts<2, S, T, WEND>(p, nts, s);
  }
}

template <typename T, bool WEND>
hipError_t launch_lp_terms(const LPParams& p, int deg, int nts, int terms, hipStream_t s) {
  switch (terms) {
    case 1: return launch_lp_deg<1, T, WEND>(p, deg, nts, s);
    case 2: return launch_lp_deg<2, T, WEND>(p, deg, nts, s);
    default: return launch_lp_deg<3, T, WEND>(p, deg, nts, s);
  }
}

// One workgroup per resident slot of the device (compute units x the
// kernel's occupancy), at most one per item, at most max_grid if nonzero.
template <int DEG, int NTS, int S, typename T, bool SHAPE>
hipError_t launch_batch_impl(const LPBatch& b, int max_grid, hipStream_t s) {
  size_t lds;
  if constexpr (SHAPE) lds = (size_t)ShapeLayout<DEG, NTS, S>::kBytes;
  else lds = (size_t)LPLayout<DEG, NTS, S, T>::kBytes;
  const void* fn = (const void*)fit_lp_batch_kernel<DEG, NTS, S, T, SHAPE>;
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  int dev = 0, cus = 0, per_cu = 0;
  if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
  if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess)
    return e;
  if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, kThreads, lds)) !=
      hipSuccess)
    return e;
  int64_t grid = (int64_t)cus * (per_cu > 0 ? per_cu : 1);
  if (grid > b.n_items) grid = b.n_items;
  if (max_grid > 0 && grid > max_grid) grid = max_grid;
  if (grid < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL((fit_lp_batch_kernel<DEG, NTS, S, T, SHAPE>), dim3((unsigned)grid),
                     dim3(kThreads), lds, s, b);
  return hipGetLastError();
}

template <int DEG, int S, typename T>
hipError_t launch_batch_nts(const LPBatch& b, int nts, int grid, hipStream_t s) {
  switch (nts) {
    case 1: return launch_batch_impl<DEG, 1, S, T, false>(b, grid, s);
    case 2: return launch_batch_impl<DEG, 2, S, T, false>(b, grid, s);
    case 3: return launch_batch_impl<DEG, 3, S, T, false>(b, grid, s);
    case 4: return launch_batch_impl<DEG, 4, S, T, false>(b, grid, s);
    case 5: return launch_batch_impl<DEG, 5, S, T, false>(b, grid, s);
    case 6: return launch_batch_impl<DEG, 6, S, T, false>(b, grid, s);
    case 7: return launch_batch_impl<DEG, 7, S, T, false>(b, grid, s);
    case 8: return launch_batch_impl<DEG, 8, S, T, false>(b, grid, s);
    default: break;
  }
  if constexpr (DEG > 0) {
    // the two-pass form, kBatchShape + its attribute tiles
    switch (nts - kBatchShape) {
      case 1: return launch_batch_impl<DEG, 1, S, T, true>(b, grid, s);
      case 2: return launch_batch_impl<DEG, 2, S, T, true>(b, grid, s);
      case 3: return launch_batch_impl<DEG, 3, S, T, true>(b, grid, s);
      case 4: return launch_batch_impl<DEG, 4, S, T, true>(b, grid, s);
      default: break;
    }
  }
  return hipErrorInvalidValue;
}

template <int S, typename T>
hipError_t launch_batch_deg(const LPBatch& b, int deg, int nts, int grid, hipStream_t s) {
  switch (deg) {
    case 0: return launch_batch_nts<0, S, T>(b, nts, grid, s);
    case 1: return launch_batch_nts<1, S, T>(b, nts, grid, s);
    default: return launch_batch_nts<2, S, T>(b, nts, grid, s);
  }
}

}  // namespace
}  // namespace mls
