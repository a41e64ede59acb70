// Space mappings of the MLS fields (Muelder et al., Sec. 3.4, Fig. 5b-d):
// discrete colour bands and adaptive contour lines, per grid node.
//
// Bands: the band of a value is the number of isovalues at or below it
// (the contour cases' tie rule), 255 for NaN; with a colour map the node
// also takes its band's RGBA colour (0 for NaN).
//
// Adaptive lines: level j = 0 .. L-1 has lines at origin + k spacing / 2^j.
// At a node the field changes by r = |(g_x dx, g_y dy)| per pixel (the
// gradient in pixel coordinates), so level j's lines are s_j = (spacing /
// 2^j) / r pixels apart; level 0 is always drawn, finer levels with opacity
// clamp((s_j - fade_lo) / (fade_hi - fade_lo), 0, 1) -- more lines where
// space is expanded, fewer where it is compressed.  The intensity is the
// largest opacity x (1 - e_j / halfwidth)+ over the levels, e_j the pixel
// distance to the nearest level-j line.  Float64 arithmetic per node.
//
// Both are elementwise: one read of the field (and gradient), one write per
// node, bound by HBM.  On 13 fields of 1024^2 (10 isovalues with colours; 3
// levels) bands move 122 MB and lines 218 MB, 24 and 42 us at the rate of a
// large copy.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "mls_internal.h"

namespace mls {
namespace {

constexpr int kBandIso = 256;   // isovalues a launch can take, padded

// iso: the field's isovalues in LDS, padded to a multiple of 4 with NaN
// (which no value reaches).
__device__ __forceinline__ int value_band(float v, const float* iso, int n4) {
  int b = 0;
  for (int k = 0; k < n4; k += 4) {
    const float4 q = *(const float4*)(iso + k);
    b += (v >= q.x ? 1 : 0) + (v >= q.y ? 1 : 0) + (v >= q.z ? 1 : 0) + (v >= q.w ? 1 : 0);
  }
  return v != v ? 255 : b;
}

// A row of workgroups per field (blockIdx.y), its isovalues and colours in
// LDS; four consecutive nodes per thread when P % 4 == 0 and the arrays are
// aligned for it (16-byte loads, 4-byte band and 16-byte colour stores), one
// per thread otherwise.  Finding a node's field by a 64-bit division and
// reading isovalues and colours through the cache took 43.4 us instead of
// 25 on the 13 fields above.
template <bool VEC>
__global__ __launch_bounds__(256) void map_bands_kernel(MapBandsArgs a) {
  __shared__ __attribute__((aligned(16))) float iso[kBandIso];
  __shared__ uint32_t cm[kBandIso];   // entry 255: NaN
  const int tid = threadIdx.x;
  const int n4 = (a.n_iso + 3) / 4 * 4;
  for (int d = blockIdx.y; d < a.D; d += gridDim.y) {
    __syncthreads();
    if (tid < n4) iso[tid] = tid < a.n_iso ? a.iso[(int64_t)d * a.n_iso + tid] : __builtin_nanf("");
    if (a.rgba)
      cm[tid] = tid <= a.n_iso ? a.colormap[(int64_t)d * (a.n_iso + 1) + tid] : 0u;
    __syncthreads();
    const float* f = a.fields + (int64_t)d * a.P;
    const int64_t units = VEC ? a.P / 4 : a.P;
    for (int64_t u = (int64_t)blockIdx.x * 256 + tid; u < units; u += (int64_t)gridDim.x * 256) {
      const int64_t i = (int64_t)d * a.P + (VEC ? 4 * u : u);
      if (VEC) {
        const float4 v = ((const float4*)f)[u];
        const int b0 = value_band(v.x, iso, n4), b1 = value_band(v.y, iso, n4);
        const int b2 = value_band(v.z, iso, n4), b3 = value_band(v.w, iso, n4);
        if (a.bands)
          *(uint32_t*)(a.bands + i) = (uint32_t)b0 | ((uint32_t)b1 << 8) | ((uint32_t)b2 << 16) |
                                      ((uint32_t)b3 << 24);
        if (a.rgba) *(uint4*)(a.rgba + i) = make_uint4(cm[b0], cm[b1], cm[b2], cm[b3]);
      } else {
        const int b = value_band(f[u], iso, n4);
        if (a.bands) a.bands[i] = (uint8_t)b;
        if (a.rgba) a.rgba[i] = cm[b];
      }
    }
  }
}

// Per-launch constants of the adaptive lines.
struct LineConsts {
  double inv_fade, inv_hw;   // 1 / (fade_hi - fade_lo), 1 / halfwidth
};

// 1 / sqrt(q) for a positive finite q: the hardware estimate (about 23 bits)
// and two Newton steps, to about an ulp, in a third of the instructions of
// the correctly rounded square root and reciprocal.
__device__ __forceinline__ double inv_sqrt(double q) {
  double y = __builtin_amdgcn_rsq(q);
  y = fma(y, fma(-(q * y), 0.5 * y, 0.5), y);
  return fma(y, fma(-(q * y), 0.5 * y, 0.5), y);
}

__device__ __forceinline__ float adaptive_intensity(const MapAdaptiveArgs& a, const LineConsts& c,
                                                    double f, double gx, double gy, double origin,
                                                    double spacing, double inv_spacing) {
  const double px = gx * a.dx, py = gy * a.dy;
  const double q = px * px + py * py;
  // squares past the estimate's range (a slope of 1e-150 or 1e150 per pixel)
  // take the square root and division
  const double inv_r = q > 1e-300 && q < 1e300 ? inv_sqrt(q) : 1.0 / sqrt(q);
  double t = (f - origin) * inv_spacing;   // position in level-0 steps
  double s = spacing * inv_r;              // level-0 spacing in pixels
  double best = fmax(1.0 - fabs(t - rint(t)) * s * c.inv_hw, 0.0);
  for (int j = 1; j < a.n_levels; ++j) {
    t *= 2.0;
    s *= 0.5;
    const double op = fmin(fmax((s - a.fade_lo) * c.inv_fade, 0.0), 1.0);
    const double e = fabs(t - rint(t)) * s;
    best = fmax(best, op * fmax(1.0 - e * c.inv_hw, 0.0));
  }
  if (f != f) return __builtin_nanf("");
  return q > 0.0 && q < __builtin_inf() && spacing > 0.0 ? (float)best : 0.0f;
}

// A row of workgroups per field; four consecutive nodes per thread when
// P % 4 == 0 and the arrays are 16-byte aligned.  A node is about 60 float64
// instructions (40 us on the fields above; with the correctly rounded
// square root and three divisions per node, two of them by launch constants,
// 54 us).
template <bool VEC>
__global__ __launch_bounds__(256) void map_adaptive_kernel(MapAdaptiveArgs a, LineConsts c) {
  for (int d = blockIdx.y; d < a.D; d += gridDim.y) {
    const double origin = (double)a.levels[2 * d], spacing = (double)a.levels[2 * d + 1];
    const double inv_spacing = 1.0 / spacing;
    const float* fp = a.fields + (int64_t)d * a.P;
    const float* gxp = a.grads + (int64_t)(2 * d) * a.P;
    const float* gyp = gxp + a.P;
    float* out = a.out + (int64_t)d * a.P;
    const int64_t units = VEC ? a.P / 4 : a.P;
    for (int64_t u = (int64_t)blockIdx.x * 256 + threadIdx.x; u < units;
         u += (int64_t)gridDim.x * 256) {
      if (VEC) {
        const float4 f = ((const float4*)fp)[u];
        const float4 gx = ((const float4*)gxp)[u], gy = ((const float4*)gyp)[u];
        float4 o;
        o.x = adaptive_intensity(a, c, f.x, gx.x, gy.x, origin, spacing, inv_spacing);
        o.y = adaptive_intensity(a, c, f.y, gx.y, gy.y, origin, spacing, inv_spacing);
        o.z = adaptive_intensity(a, c, f.z, gx.z, gy.z, origin, spacing, inv_spacing);
        o.w = adaptive_intensity(a, c, f.w, gx.w, gy.w, origin, spacing, inv_spacing);
        ((float4*)out)[u] = o;
      } else {
        out[u] = adaptive_intensity(a, c, fp[u], gxp[u], gyp[u], origin, spacing, inv_spacing);
      }
    }
  }
}

// One row of workgroups per field (at most 65,535 rows; the kernels stride
// over the rest), enough in all to fill the chip several times over.
dim3 map_grid(int D, int64_t units) {
  const int64_t rows = D < 65535 ? D : 65535;
  const int64_t most = (8192 + rows - 1) / rows, need = (units + 255) / 256;
  return dim3((unsigned)(need < most ? (need > 0 ? need : 1) : most), (unsigned)rows);
}

}  // namespace

hipError_t launch_map_bands(const MapBandsArgs& a, hipStream_t s) {
  const bool vec = (a.P & 3) == 0 && ((uintptr_t)a.fields & 15) == 0 &&
                   ((uintptr_t)a.bands & 3) == 0 && ((uintptr_t)a.rgba & 15) == 0;
  if (vec)
    hipLaunchKernelGGL(map_bands_kernel<true>, map_grid(a.D, a.P / 4), dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL(map_bands_kernel<false>, map_grid(a.D, a.P), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_map_adaptive(const MapAdaptiveArgs& a, hipStream_t s) {
  const bool vec = (a.P & 3) == 0 && ((uintptr_t)a.fields & 15) == 0 &&
                   ((uintptr_t)a.grads & 15) == 0 && ((uintptr_t)a.out & 15) == 0;
  const LineConsts c{1.0 / (a.fade_hi - a.fade_lo), 1.0 / a.halfwidth};
  if (vec)
    hipLaunchKernelGGL(map_adaptive_kernel<true>, map_grid(a.D, a.P / 4), dim3(256), 0, s, a, c);
  else
    hipLaunchKernelGGL(map_adaptive_kernel<false>, map_grid(a.D, a.P), dim3(256), 0, s, a, c);
  return hipGetLastError();
}

}  // namespace mls
