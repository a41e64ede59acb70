// Input staging for the low-precision fit paths.
//
// The attributes are fitted as f' = (f - shift_d) / scale_d with
// shift_d = (max_d + min_d) / 2 and scale_d = (max_d - min_d) / 2 over the
// input values, so every attribute lies in [-1, 1] before it is rounded to a
// 16-bit format.  Moving least squares is affine-equivariant in the values
// (the fit of a f + b is a fit(f) + b: Eq. 5-8 are linear in q and reproduce
// constants), so the solve maps the result back exactly.
//
// The staged payload (float32) is point-major, vals[i][d] = f'_{i,d}, for the
// dense weights, whose tiles gather the points in their reach: a point's
// attributes are one run, so a gathered point costs one or two cache lines
// (attribute-major it cost a line per attribute).  The compact-support fit
// takes it attribute-major, vals_t[d][i], and sorts each row into cell order
// (mls_cells.hip).  Bound: HBM (one read of values, one write).
//
// Point-major, an attribute with a NaN takes a NaN shift and scale: the NaN
// reaches every node of its field, as it does when all points are summed (0 x
// NaN), also where the tile never meets the point.  Attribute-major the range
// is that of the other values and the NaN stays at its point, so that only the
// tiles that list the point see it, as the compact support means it.  An
// infinite value reaches every node either way (an infinite range).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "../../include/mls.h"
#include "mls_internal.h"

namespace mls {
namespace {

constexpr int kRowsPerBlock = 1024;
constexpr int kRangeRows = 32;      // rows a range block reads at a time
// Up to this many partial ranges in all the staging blocks reduce them
// themselves, eight loads per thread, which saves the reduction's own launch
// (about 5 us).
constexpr int64_t kFusedRanges = 2048;
constexpr int kMaxAttrs = 1024;     // attributes of a 16-bit fit
static_assert(MLS_MAX_D_LP <= kMaxAttrs, "attributes in LDS");

// min and max that return NaN when either operand is one (KEEP) or the other
// operand then.
template <bool KEEP>
__device__ __forceinline__ float range_min(float a, float b) {
  return KEEP && (a != a || b != b) ? a + b : fminf(a, b);
}
template <bool KEEP>
__device__ __forceinline__ float range_max(float a, float b) {
  return KEEP && (a != a || b != b) ? a + b : fmaxf(a, b);
}

// Partial min / max of each attribute over a block of rows.  Block (32, 32):
// threadIdx.x walks 32 consecutive attributes of a row (coalesced),
// threadIdx.y the block's rows, 32 at a time and four such steps in flight
// (a block is a chain of loads: 8 rows at a time, one in flight, took 19 us
// for 20,011 points of 5 attributes where this takes 8.6).
template <bool KEEP>
__global__ __launch_bounds__(32 * kRangeRows) void attr_range_kernel(const float* vals, int64_t n,
                                                                     int D, float* pmin,
                                                                     float* pmax) {
  __shared__ float smin[kRangeRows][33], smax[kRangeRows][33];
  const int d = blockIdx.y * 32 + threadIdx.x;
  const int64_t r0 = (int64_t)blockIdx.x * kRowsPerBlock;
  const int64_t r1 = r0 + kRowsPerBlock < n ? r0 + kRowsPerBlock : n;
  float lo = INFINITY, hi = -INFINITY;
  if (d < D) {
    for (int64_t r = r0 + threadIdx.y; r < r1; r += 4 * kRangeRows) {
      float v[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {   // past the end the last row again
        const int64_t rq = r + q * kRangeRows;
        v[q] = vals[(rq < r1 ? rq : r1 - 1) * D + d];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        lo = range_min<KEEP>(lo, v[q]);
        hi = range_max<KEEP>(hi, v[q]);
      }
    }
  }
  smin[threadIdx.y][threadIdx.x] = lo;
  smax[threadIdx.y][threadIdx.x] = hi;
  __syncthreads();
  for (int half = kRangeRows / 2; half > 0; half /= 2) {
    if ((int)threadIdx.y < half) {
      smin[threadIdx.y][threadIdx.x] =
          range_min<KEEP>(smin[threadIdx.y][threadIdx.x], smin[threadIdx.y + half][threadIdx.x]);
      smax[threadIdx.y][threadIdx.x] =
          range_max<KEEP>(smax[threadIdx.y][threadIdx.x], smax[threadIdx.y + half][threadIdx.x]);
    }
    __syncthreads();
  }
  if (threadIdx.y == 0 && d < D) {
    pmin[(int64_t)blockIdx.x * D + d] = smin[0][threadIdx.x];
    pmax[(int64_t)blockIdx.x * D + d] = smax[0][threadIdx.x];
  }
}

// Shift and scale of a range: the float64 midpoint and half-range, rounded
// once; a scale of 1 for a constant attribute.
__device__ __forceinline__ void range_map(float lo, float hi, float* shift, float* scale) {
  const double mid = 0.5 * ((double)lo + (double)hi);
  const double half = 0.5 * ((double)hi - (double)lo);
  *shift = (float)mid;
  *scale = half > 0.0 || half != half ? (float)half : 1.0f;
}

// Shift and scale of attributes d0 .. d0 + nd of the partial ranges into LDS,
// by the block's threads (`t` of `threads`); the caller synchronises.
template <bool KEEP>
__device__ __forceinline__ void fused_map(const float* pmin, const float* pmax, int nblk, int D,
                                          int d0, int nd, int t, int threads, float* sshift,
                                          float* sscale) {
  for (int d = t; d < nd; d += threads) {
    float lo = INFINITY, hi = -INFINITY;
#pragma unroll 8
    for (int b = 0; b < nblk; ++b) {
      lo = range_min<KEEP>(lo, pmin[(int64_t)b * D + d0 + d]);
      hi = range_max<KEEP>(hi, pmax[(int64_t)b * D + d0 + d]);
    }
    range_map(lo, hi, sshift + d, sscale + d);
  }
}

// One block per attribute: min / max over the partial ranges (min and max
// are exact, so the order of the reduction does not matter).
template <bool KEEP>
__global__ __launch_bounds__(256) void attr_finalize_kernel(const float* pmin, const float* pmax,
                                                            int nblk, int D, float* shift,
                                                            float* scale) {
  __shared__ float slo[4], shi[4];
  const int d = blockIdx.x;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  float lo = INFINITY, hi = -INFINITY;
  for (int b = t; b < nblk; b += 256) {
    lo = range_min<KEEP>(lo, pmin[(int64_t)b * D + d]);
    hi = range_max<KEEP>(hi, pmax[(int64_t)b * D + d]);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    lo = range_min<KEEP>(lo, __shfl_xor(lo, o, 64));
    hi = range_max<KEEP>(hi, __shfl_xor(hi, o, 64));
  }
  if (lane == 0) {
    slo[wave] = lo;
    shi[wave] = hi;
  }
  __syncthreads();
  if (t != 0) return;
  lo = range_min<KEEP>(range_min<KEEP>(slo[0], slo[1]), range_min<KEEP>(slo[2], slo[3]));
  hi = range_max<KEEP>(range_max<KEEP>(shi[0], shi[1]), range_max<KEEP>(shi[2], shi[3]));
  range_map(lo, hi, shift + d, scale + d);
}

// vals_t[d][i] = (vals[i][d] - shift[d]) / scale[d], through a 32 x 32 LDS
// tile so that both the read and the write are coalesced.  nblk > 0: shift
// and scale come from the partial ranges, and the first block stores them.
__global__ __launch_bounds__(256) void stage_values_kernel(const float* vals, int64_t n, int D,
                                                           float* shift, float* scale,
                                                           const float* pmin, const float* pmax,
                                                           int nblk, float* vals_t) {
  __shared__ float tile[32][33];
  __shared__ float sshift[32], sscale[32];
  const int64_t i0 = (int64_t)blockIdx.x * 32;
  const int d0 = blockIdx.y * 32;
  const int nd = D - d0 < 32 ? D - d0 : 32;
  const int t = threadIdx.y * 32 + threadIdx.x;
  if (nblk > 0) {
    fused_map<false>(pmin, pmax, nblk, D, d0, nd, t, 256, sshift, sscale);
    if (blockIdx.x == 0 && t < nd) {
      shift[d0 + t] = sshift[t];
      scale[d0 + t] = sscale[t];
    }
  } else if (t < nd) {
    sshift[t] = shift[d0 + t];
    sscale[t] = scale[d0 + t];
  }
  __syncthreads();
  for (int q = threadIdx.y; q < 32; q += 8) {
    const int64_t i = i0 + q;
    const int d = threadIdx.x;
    float v = 0.0f;
    if (i < n && d < nd)
      v = (float)(((double)vals[i * D + d0 + d] - (double)sshift[d]) / (double)sscale[d]);
    tile[q][threadIdx.x] = v;
  }
  __syncthreads();
  for (int q = threadIdx.y; q < 32; q += 8) {
    const int d = d0 + q;
    const int64_t i = i0 + threadIdx.x;
    if (i < n && d < D) vals_t[(int64_t)d * n + i] = tile[threadIdx.x][q];
  }
}

// vals_s[i][d] = (vals[i][d] - shift[d]) / scale[d], the input's layout.
// nblk as above.
__global__ __launch_bounds__(256) void stage_rows_kernel(const float* vals, int64_t total, int D,
                                                         float* shift, float* scale,
                                                         const float* pmin, const float* pmax,
                                                         int nblk, float* vals_s) {
  __shared__ float sshift[kMaxAttrs], sscale[kMaxAttrs];
  const int t = threadIdx.x;
  if (nblk > 0) {
    fused_map<true>(pmin, pmax, nblk, D, 0, D, t, 256, sshift, sscale);
    // a thread stores what it found itself
    for (int d = t; blockIdx.x == 0 && d < D; d += 256) {
      shift[d] = sshift[d];
      scale[d] = sscale[d];
    }
  } else {
    for (int d = t; d < D; d += 256) {
      sshift[d] = shift[d];
      sscale[d] = scale[d];
    }
  }
  __syncthreads();
  for (int64_t e = (int64_t)blockIdx.x * 256 + t; e < total; e += (int64_t)gridDim.x * 256) {
    const int d = (int)(e % D);
    vals_s[e] = (float)(((double)vals[e] - (double)sshift[d]) / (double)sscale[d]);
  }
}

}  // namespace

int64_t stage_partial_blocks(int64_t n) { return (n + kRowsPerBlock - 1) / kRowsPerBlock; }

template <bool ROWS>
static hipError_t launch_stage_impl(const float* vals, int64_t n, int D, float* pmin, float* pmax,
                                    float* shift, float* scale, float* vals_s, hipStream_t s) {
  const int64_t nblk = stage_partial_blocks(n);
  const int dblk = (D + 31) / 32;
  hipLaunchKernelGGL(attr_range_kernel<ROWS>, dim3((unsigned)nblk, dblk), dim3(32, kRangeRows), 0,
                     s, vals, n, D, pmin, pmax);
  const int fused = nblk * D <= kFusedRanges ? (int)nblk : 0;
  if (!fused)
    hipLaunchKernelGGL(attr_finalize_kernel<ROWS>, dim3(D), dim3(256), 0, s, pmin, pmax,
                       (int)nblk, D, shift, scale);
  if (ROWS) {
    // 1,024 values a block, so that the fused reduction repeats less
    const int64_t nb = (n * D + 1023) / 1024;
    hipLaunchKernelGGL(stage_rows_kernel, dim3((unsigned)(nb < 65536 ? nb : 65536)), dim3(256), 0,
                       s, vals, n * D, D, shift, scale, pmin, pmax, fused, vals_s);
  } else {
    hipLaunchKernelGGL(stage_values_kernel, dim3((unsigned)((n + 31) / 32), dblk), dim3(32, 8),
                       0, s, vals, n, D, shift, scale, pmin, pmax, fused, vals_s);
  }
  return hipGetLastError();
}

hipError_t launch_stage(const float* vals, int64_t n, int D, float* pmin, float* pmax,
                        float* shift, float* scale, float* vals_s, bool rows, hipStream_t s) {
  return rows ? launch_stage_impl<true>(vals, n, D, pmin, pmax, shift, scale, vals_s, s)
              : launch_stage_impl<false>(vals, n, D, pmin, pmax, shift, scale, vals_s, s);
}

}  // namespace mls
