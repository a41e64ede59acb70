// Float64 matrix-core fits: parameters and the device code that the one-pass
// kernel (mls_fit_f64.hip) and the two-pass kernel (mls_fit_f64_shape.hip)
// share.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "mls_internal.h"
#include "mls_list.h"
#include "mls_solve.h"

namespace mls {

typedef double doublex4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int kWaves = 4;
constexpr int kCols = 16;      // node columns per tile (one M-tile)
constexpr int KT = 64;         // points per LDS chunk
// LDS row stride in doubles.  A lane reads four consecutive doubles (two
// 16-byte reads) of row i = lane % 16; with a stride of KT + 2 = 66
// doubles (132 dwords, 4 mod 64) the sixteen rows of one read start in
// sixteen different 4-bank groups, so the reads are free of bank
// conflicts (a stride of 68 doubles puts rows i and i + 8 on the same
// banks).
constexpr int KS = KT + 2;
static_assert(KS % 2 == 0 && KT % 16 == 0, "rows must start on 16-byte boundaries");
struct F64Params {
  const float* pts;
  const float* vals;
  int64_t n;
  int D, F;
  double h, inv_h;
  double alpha;        // inverse-distance exponent (WM_INV kernels)
  // Gaussian over all points, WM_TABLE: factors of every grid column and row
  const double* tab;   // rows [0, tab_cols) the columns, then the grid's rows
  int64_t tab_n;       // points per row
  int tab_cols;
  double x0, y0, dx, dy;
  int W, H, tiles_x;
  double tau, floor_w;
  float* fields;
  uint8_t* deg_out;
  float* grads;        // [D][2][H][W] or null
  bool rigid;          // rigid map (EPI 2 kernels)
  // Gaussian: reach of the tiles (tile_reach), and the result of the look over
  // the attributes' sizes (look_kernel; null: the tiles look themselves)
  double list_log;     // ln n + 54 ln 2, or infinite: every tile sums all points
  const uint32_t* sizes;
  bool vec4;           // rows of the fields and of the slopes are 16-byte aligned
  bool fine;           // a tile spans at most kFineSpan h on either axis
};

constexpr double kFineSpan = 8.0;
constexpr double kFineReach2 = 18.0 * 18.0;

// Weight modes of the kernel: the Gaussian over the points in reach, the
// inverse-distance weight per pair (any exponent, or alpha = 1 and alpha = 2
// through a reciprocal), the Gaussian over all points with factors from tables
// of the launch or formed by the tile.
constexpr int WM_GAUSS = 0, WM_INV = 1, WM_INV1 = 2, WM_INV2 = 3, WM_TABLE = 4, WM_STEP = 5;

// One-pass fits by source file (mls_fit_f64_kernel.h).
hipError_t launch_fit_f64_inv(const F64Params& p, int degree, int nt, hipStream_t s);
hipError_t launch_fit_f64_all(const F64Params& p, int degree, int nt, double* tab, hipStream_t s);

// Two-pass form of the Gaussian fit (mls_fit_f64_shape.hip).
hipError_t launch_fit_f64_shape(const F64Params& p, int degree, hipStream_t s);
bool f64_use_shape_form(int degree, int D);
// Matrix and weight cycles of one strip's 64 node-point pairs: 64 per 16 columns
// (17 per 4 with the four-block form, up to 12), 4 for a weight.
inline int f64_pair_cycles(int columns, bool blocks4) {
  return 4 + (blocks4 && columns <= 12 ? 17 * ((columns + 3) / 4) : 64 * ((columns + 15) / 16));
}
// Strips of 16 nodes per wave (1, 2 or 4, at most `most`; a tile is 16 x 4 R
// nodes).  A chunk costs a workgroup its production, whatever R, and the sweep of
// R strips, whose `cycles` count per 64 pairs over its `passes`; the fullest
// compute unit decides, and where it holds one workgroup, the waits between the
// two are not covered either.  Over 390 calls (200 to 30,000 points, 128^2 to
// 1024^2, every form) the choice was within 0.2% of the best on average and 16%
// at worst.  (Taking the largest R that leaves 1,024 workgroups, whatever the
// chunks cost, was 10% slower on average and twice as slow where a tile's list
// is long: 30,000 points, all in reach, 256^2, one attribute 1,591 us with R = 1,
// 1,043 with R = 2.)
inline int f64_tile_strips(int W, int H, int most, int passes, int cycles) {
  int best = most;
  int64_t least = 0;
  for (int R = most; R >= 1; R /= 2) {
    const int64_t tiles =
        (int64_t)((W + kCols - 1) / kCols) * ((H + kWaves * R - 1) / (kWaves * R));
    const int64_t per_unit = (tiles + 255) / 256;
    const int64_t cost =
        per_unit * (600 * passes + 16 * R * cycles) + (per_unit == 1 ? 1500 * passes : 0);
    if (R == most || cost < least) {
      best = R;
      least = cost;
    }
  }
  return best;
}

namespace {

constexpr int kListCap = 2048;
constexpr int kListB = list_bytes(kListCap);

__device__ __forceinline__ void read4(const double* src, double* dst) {
  const double2* v = reinterpret_cast<const double2*>(src);
  const double2 lo = v[0], hi = v[1];
  dst[0] = lo.x;
  dst[1] = lo.y;
  dst[2] = hi.x;
  dst[3] = hi.y;
}

// ---- reach of a tile (Gaussian) ----
//
// A tile sums only the points within R h of the rectangle of its nodes.  What
// it leaves out of any node's sum of w b_j^2 (b_j up to degree DEG in u) is
// at most n exp(-R^2) R^(2 DEG).  R is chosen so that this is 2^-54 of the
// larger of the weight floor (nodes below it are undetermined) and a lower
// bound S of the weight sum at the tile's nodes: less than the rounding of
// the sums themselves.  Every sum leaves out the same points, so the fit is
// that of the weight cut to zero there.  A node whose smallest diagonal
// moment is itself below 2^-14 of that scale (its near points all on one
// line through it, say) could still see what is left out above 2^-40: its
// tile is then summed again over all points (kDiagFloor).
//
// The products with an attribute see the weights times its values, and a value
// far away may be larger than those near a node by more than the weights fall
// (a marker of 1e30 for a missing value, an attribute that grows
// exponentially).  So what is left out has to be small against the attribute's
// smallest magnitude other than 0: where the largest is more than 2^kSizeFree
// times that, the bound above is taken smaller by the rest, which leaves at
// most 2^-30 of what the near points add, a 64th of the float32 result's
// rounding.  Attributes of up to 2^24 from the smallest to the largest, which
// is most, have the reach of the weights alone.
constexpr double kDiagFloor = 0x1p-14;
constexpr int kSizeFree = 24;
constexpr int kSizeNotFinite = 1 << 20;

// Magnitudes of an attribute as bits of |f|, which order as the values do:
// the largest, and the smallest other than 0.
struct Sizes {
  uint32_t hi = 0, lo = 0x7F800000u;
  __device__ __forceinline__ void add(float f) {
    const uint32_t m = __builtin_bit_cast(uint32_t, f) & 0x7FFFFFFFu;
    hi = m > hi ? m : hi;
    lo = m != 0 && m < lo ? m : lo;
  }
};

// Binary digits that the bound gains for an attribute: at least the log2 of
// the ratio of its sizes, less kSizeFree; kSizeNotFinite for an infinity or a
// NaN.
__device__ __forceinline__ int size_digits(uint32_t hi, uint32_t lo) {
  if (hi >= 0x7F800000u) return kSizeNotFinite;
  if (hi == 0) return 0;
  // (subnormal numbers go down to 2^-149, the exponent field of 2^-126 being 1)
  const int eh = (int)(hi >> 23), el = lo >> 23 ? (int)(lo >> 23) : -22;
  const int digits = (eh > 1 ? eh : 1) + 1 - el - kSizeFree;
  return digits > 0 ? digits : 0;
}

// A value that is the same in every lane, into scalar registers.
__device__ __forceinline__ double uniform(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
  const uint64_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
  return __builtin_bit_cast(double, (hi << 32) | lo);
}

// The tile's node rectangle is |u - m| <= e per axis (tile frame, units of h).
struct F64Reach {
  double ox, oy;         // u = x inv_h - o, with the rectangle's centre as origin
  double inv_h, ex, ey;
  double r2;             // R^2 (infinite: every point)
  double scale;          // max(S, weight floor)
};

// Whether the tile must take the point at (x, y): not if it is farther than R
// from the rectangle.  (With an input that is not finite r2 is infinite, and
// the comparison keeps every point.)
__device__ __forceinline__ bool in_reach(const F64Reach& t, float x, float y) {
  const double ax = fmax(fabs(fma((double)x, t.inv_h, -t.ox)) - t.ex, 0.0);
  const double ay = fmax(fabs(fma((double)y, t.inv_h, -t.oy)) - t.ey, 0.0);
  return !(ax * ax + ay * ay > t.r2);
}

// The look over n x D values by the workgroup's T threads (the first T / D * D
// of them: each keeps to one attribute), into LDS words hi[D] and lo[D], which the caller has set to 0 and 0x7F800000 before a barrier and
// reads after one.  A coordinate that is not finite counts as an attribute 0
// that is not.  Elements are taken from block `b` of `nb`.
template <int T>
__device__ __forceinline__ void look_sizes(const float* vals, int64_t n, int D, const float* pts,
                                           int b, int nb, uint32_t* hi, uint32_t* lo) {
  const auto v = global_ptr(vals);
  const auto q = global_ptr(pts);
  const int tid = threadIdx.x, per = T / D * D;
  Sizes sz;
  if (tid < per) {
    const int64_t step = (int64_t)nb * per, total = n * D;
#pragma unroll 8
    for (int64_t e = (int64_t)b * per + tid; e < total; e += step) sz.add(v[e]);
    atomicMax(hi + tid % D, sz.hi);
    atomicMin(lo + tid % D, sz.lo);
  }
  bool bad = false;
#pragma unroll 4
  for (int64_t e = (int64_t)b * T + tid; e < 2 * n; e += (int64_t)nb * T)
    bad |= !(fabsf(q[e]) < __builtin_inff());
  if (bad) atomicMax(hi, 0x7F800000u);
}

// The reach of the tile whose anchor node is (c0 + 8, r0 + rows / 2).  Every
// thread of the workgroup calls it; `shared` is LDS for kWaves floats and 2 D
// words, and the call ends with a barrier.  S is the sum over the points of
// the weight at their farthest node of the tile; below kFloorPoints, where a
// pass over them costs as much as it saves, S = 0.
constexpr int kFloorPoints = 1024;

template <int DEG>
__device__ __forceinline__ F64Reach tile_reach(const F64Params& p, int rows, double cx, double cy,
                                               float* shared) {
  F64Reach t;
  // the rectangle's centre lies half a node before the anchor
  t.ox = uniform((cx - 0.5 * p.dx) * p.inv_h);
  t.oy = uniform((cy - 0.5 * p.dy) * p.inv_h);
  t.inv_h = p.inv_h;
  // a little more than half the rectangle: the test's own rounding
  t.ex = uniform(0.5 * (double)(kCols - 1) * fabs(p.dx) * p.inv_h + 0x1p-40 * (1.0 + fabs(t.ox)));
  t.ey = uniform(0.5 * (double)(rows - 1) * fabs(p.dy) * p.inv_h + 0x1p-40 * (1.0 + fabs(t.oy)));
  t.scale = uniform(p.floor_w);
  t.r2 = __builtin_inf();
  if (!(p.list_log < __builtin_inf())) return t;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int D = p.D;
  uint32_t* hi = (uint32_t*)shared + kWaves;
  uint32_t* lo = hi + D;
  if (!p.sizes) {
    if (tid < D) {
      hi[tid] = 0;
      lo[tid] = 0x7F800000u;
    }
    __syncthreads();
  }
  const auto pts = global_ptr(p.pts);
  float S = 0.0f;
  if (p.n >= kFloorPoints) {
#pragma unroll 4
    for (int i = tid; i < (int)p.n; i += kThreads) {
      const float ax = (float)(fabs(fma((double)pts[2 * i], p.inv_h, -t.ox)) + t.ex);
      const float ay = (float)(fabs(fma((double)pts[2 * i + 1], p.inv_h, -t.oy)) + t.ey);
      S += __expf(-(ax * ax + ay * ay));
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) S += __shfl_xor(S, o, 64);
  }
  if (!p.sizes) look_sizes<kThreads>(p.vals, p.n, D, p.pts, 0, 1, hi, lo);
  if (lane == 0) shared[wave] = S;
  __syncthreads();
  S = 0.0f;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) S += shared[w];
  int digits = 0;
  if (p.sizes) {
    digits = (int)*global_ptr(p.sizes);
  } else {
    for (int d = lane; d < D; d += 64) digits = max(digits, size_digits(hi[d], lo[d]));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) digits = max(digits, __shfl_xor(digits, o, 64));
  }
  digits = __builtin_amdgcn_readfirstlane(digits);
  __syncthreads();
  // inputs that are not finite reach every node (0 x NaN): sum all points
  const bool any = digits >= kSizeNotFinite || !(S < __builtin_inff());
  t.scale = uniform(fmax(0.99 * (double)S, p.floor_w));
  if (!any && t.scale > 0.0) {
    const double L = p.list_log + (double)digits * 0.6931471805599453 - log(t.scale);
    double r2 = L;
#pragma unroll
    for (int it = 0; it < 4; ++it) r2 = L + DEG * log(r2);
    t.r2 = uniform(r2);
  }
  return t;
}

// Gaussian factors g_c = exp(-(u - e_c)^2), e_c = (c - c_mid) s, of one point
// at a half of the nodes of one axis (`cnt` of them, the upper half or the
// lower).  They follow by stepping: g_{c+1} / g_c = exp(2 s (u - e_c) - s^2),
// and that ratio itself shrinks by q = exp(-2 s^2) per step: two
// multiplications per node after two exponentials.
// On fine grids (kFineSpan), for a list within a reach of kFineReach2, one
// thread steps through a half from its first node: a listed point is at most
// R + 8 h from it, and the exponents stay above -(18 + 8)^2 = -676, short of
// where exp loses digits (-708).  Otherwise (a tiny weight floor makes R as
// large as 27) start at the node nearest to u (the largest factor), so that
// every exponent is <= 0; the upper half's thread steps up from it and the
// lower half's down.
template <int CNT>
__device__ __forceinline__ void gauss_steps(bool fine, double u, double s, double q, bool up,
                                            double* g) {
  constexpr int mid = CNT / 2;
  if (fine) {
    const int c1 = up ? mid : 0;
    const double dc = u - (double)(c1 - mid) * s;
    double v = exp(-(dc * dc));
    double r = exp(2.0 * s * dc - s * s);
    g += c1 * KS;
#pragma unroll
    for (int c = 0; c < mid; ++c) {
      g[c * KS] = v;
      v *= r;
      r *= q;
    }
    return;
  }
  const double t = u / s + (double)mid;
  const int cs = (int)fmin(fmax(rint(t), 0.0), (double)(CNT - 1));
  const double dc = u - (double)(cs - mid) * s;
  const double gv = exp(-(dc * dc));
  double r = exp((up ? 2.0 : -2.0) * s * dc - s * s);
  double v = gv;
  if (up) {
    g[cs * KS] = gv;
    for (int c = cs + 1; c < CNT; ++c) {
      v *= r;
      r *= q;
      g[c * KS] = v;
    }
  } else {
    for (int c = cs - 1; c >= 0; --c) {
      v *= r;
      r *= q;
      g[c * KS] = v;
    }
  }
}

// The factors of a chunk of kn points, gx [16][KS] and gy [ROWS][KS] after
// it: one thread per point, axis and half.  Points past the chunk weigh 0.
template <int ROWS>
__device__ __forceinline__ void put_gauss(bool fine, const double* ux, const double* uy,
                                          double* gx, int kn, double sx, double sy, double qx,
                                          double qy, int tid) {
  double* gy = gx + kCols * KS;
  const int k = tid & (KT - 1);
  const bool xaxis = (tid & KT) == 0, up = tid < 2 * KT;
  if (k < kn) {
    if (xaxis) gauss_steps<kCols>(fine, ux[k], sx, qx, up, gx + k);
    else gauss_steps<ROWS>(fine, uy[k], sy, qy, up, gy + k);
  } else {
    double* g = (xaxis ? gx : gy) + k;
    const int mid = (xaxis ? kCols : ROWS) / 2;
    for (int c = 0; c < mid; ++c) g[((up ? mid : 0) + c) * KS] = 0.0;
  }
}

// Moment monomials of a chunk's tile-frame coordinates, rows of G: a point per
// lane, the rows spread over the waves.
template <int NMOM>
__device__ __forceinline__ void put_monomials(const double* ux, const double* uy, double* G,
                                              int lane, int wave) {
  const double x = ux[lane], y = uy[lane];
  double px[5], py[5];
  px[0] = py[0] = 1.0;
#pragma unroll
  for (int a = 1; a < 5; ++a) {
    px[a] = px[a - 1] * x;
    py[a] = py[a - 1] * y;
  }
  int j = 0;
#pragma unroll
  for (int t = 0; t < 5; ++t)
#pragma unroll
    for (int b = 0; b <= t; ++b, ++j)   // ordered by total degree, then by y power
      if (j < NMOM && (j & 3) == wave) G[j * KS + lane] = px[t - b] * py[b];
}

}  // namespace
}  // namespace mls
