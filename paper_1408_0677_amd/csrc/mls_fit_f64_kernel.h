// The one-pass float64 kernel (described at the top of mls_fit_f64.hip) and
// its launches, for the source files that instantiate it: mls_fit_f64.hip
// (Gaussian, points in reach), mls_fit_f64_all.hip (Gaussian, all points) and
// mls_fit_f64_inv.hip (inverse distance).
#pragma once

#include "mls_fit_f64.h"

namespace mls {
namespace {

// Waves that run the epilogue at the same time: the epilogue needs a
// [nodes][features] float64 staging area per wave, and sharing it keeps the
// kernel's LDS small enough for two workgroups per CU.
constexpr int kEpiWaves = 2;

template <int DEG, int NT, int R>
struct F64Layout {
  static constexpr int kRows = kWaves * R;
  static constexpr int kFP = NT * 16;                    // padded features
  static constexpr int m = DEG == 0 ? 1 : (DEG == 1 ? 3 : 6);
  static constexpr int nmom = DEG == 0 ? 1 : (DEG == 1 ? 6 : 15);
  // most attributes NT feature tiles can hold, and the per-thread registers
  // that hold one chunk of their values
  static constexpr int kDMax = (kFP - nmom) / m;
  static constexpr int kValRegs =
      kDMax > 0 ? (KT * kDMax + kThreads - 1) / kThreads : 1;
  // per-thread registers that hold one chunk of table factors (16 + 4R rows)
  static constexpr int kTabRegs = ((kCols + kRows) * KT + kThreads - 1) / kThreads;
  // chunk phase
  static constexpr int kUx = 0;                          // [KT] tile-frame u_x
  static constexpr int kUy = kUx + KT;                   // [KT]
  static constexpr int kGx = kUy + KT;                   // [16][KS]
  static constexpr int kGy = kGx + kCols * KS;           // [kRows][KS]
  static constexpr int kG = kGy + kRows * KS;            // [kFP][KS]
  static constexpr int kChunk = kG + kFP * KS;
  // epilogue phase: per solving wave [16R nodes][kFP + 1]
  static constexpr int kEpiStride = kFP + 1;
  static constexpr int kEpi = kEpiWaves * 16 * R * kEpiStride;
  static constexpr int kDoubles = kChunk > kEpi ? kChunk : kEpi;
  static constexpr int kBytes = 8 * kDoubles;            // then the list (Gaussian)
};

template <int DEG, int R, int EPI>
__device__ bool solve_tile_nodes(const F64Params& p, const double* epi, int stride, int lane,
                                 int wave, int r0, int c0, int rows, int64_t plane,
                                 double diag_min);

// Inverse-distance weight (Eq. 4) of a node-point pair r^2 = ox^2 + oy^2 (in
// units of h): r2^(-alpha).  log2 of r^2 is taken as its binary exponent
// plus the float32 log2 of its mantissa (so r^2 far outside float32's range
// keeps an exact exponent), and the power is rebuilt as 2^frac scaled by
// ldexp, so it cannot overflow float32 either; the relative error is that
// of the float32 exp2/log2 (about 1e-7), a common factor of all features of
// the pair.  Padding points carry an infinite offset and weigh 0.
__device__ __forceinline__ double invpow_weight(double r2, double alpha) {
  if (!(r2 < 1e300)) return 0.0;
  int ex;
  const double mant = frexp(r2, &ex);
  const double l2 = (double)ex + (double)__log2f((float)mant);
  const double e = fmin(-alpha * l2, 1000.0);
  const double ip = floor(e);
  return ldexp((double)exp2f((float)(e - ip)), (int)ip);
}

// Smallest squared offset along x: a node on a point (r^2 = 0) gets a large
// finite weight; such nodes are overwritten by the exact-hit pass.  Far below
// any other pair's r^2, also where h is a unit many times the points' distances
// (a pair 1e-9 apart has r^2 = 1e-58 with h = 1e20), and such that its square's
// reciprocal times the features stays finite.
template <int WM>
constexpr double kMinOffset2 = WM == WM_INV2 ? 1e-140 : 1e-300;

// The same weight for alpha = 1 and alpha = 2: the hardware's float64
// reciprocal estimate (relative error at most 4.5e-8, 1.0e-8 rms over
// [1e-8, 1e4], measured; the float32 reciprocal's are 1.2e-7 and 3.8e-8),
// squared for alpha = 2.  With the squared offsets tabled a pair costs one
// addition and the estimate, 20 cycles per 64 pairs instead of 28 with the
// float32 reciprocal and its conversions.  Padding points (infinite offset)
// get 1 / inf = 0.
template <int ALPHA>
__device__ __forceinline__ double invpow_weight_int(double r2) {
  const double r = __builtin_amdgcn_rcp(r2);
  return ALPHA == 1 ? r : r * r;
}

// Epilogue EPI: 0 fields, 1 fields and the slopes of the local fits (the
// extra solves raise the epilogue's register count, so they are separate
// instantiations and the plain kernels keep two workgroups per CU), 2 the
// rigid map of 2-vector values from the linear moments.
//
// Q4 > 0 (one feature tile, F <= 4 Q4 <= 12): the contraction runs on the
// four-block 4x4x4 FP64 MFMA instead of the 16x16x4 one.  Block b of that
// instruction takes nodes 4b .. 4b + 3, the same four points k and four
// feature columns c: lane l holds A (node l % 16, point l / 16) exactly as
// the 16x16x4 instruction takes it, B (point l / 16, feature l % 4, the
// same in every block) and the result for node 4 ((l / 4) % 4) + l / 16 and
// feature l % 4.  Each instruction covers the same 64 node-point pairs over
// 4 feature columns instead of 16, at about a quarter of the cycles, so the
// small shapes (Mean MLS F = 3, Affine and Rigid MLS F = 12) issue one to
// three short instructions where the 16x16x4 one carries 4 to 13 empty
// columns.
template <int DEG, int NT, int R, int WM, int EPI, int Q4 = 0>
__global__ __launch_bounds__(kThreads, WM == WM_GAUSS && NT <= 4 ? (NT == 1 ? 3 : 2) : 1)
void fit_f64_kernel(F64Params p) {
  static_assert(Q4 == 0 || NT == 1, "the 4x4x4 form covers one feature tile");
  constexpr bool INV = WM == WM_INV || WM == WM_INV1 || WM == WM_INV2;
  using L = F64Layout<DEG, NT, R>;
  constexpr int m = DEG == 0 ? 1 : (DEG == 1 ? 3 : 6);
  constexpr int nmom = DEG == 0 ? 1 : (DEG == 1 ? 6 : 15);
  extern __shared__ double lds[];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int tile_c = blockIdx.x % p.tiles_x;
  const int tile_r = blockIdx.x / p.tiles_x;
  const int c0 = tile_c * kCols;
  const int r0 = tile_r * L::kRows;
  // tile anchor: the node at the tile's centre (may lie beyond the grid)
  const double cx = p.x0 + (double)(c0 + kCols / 2) * p.dx;
  const double cy = p.y0 + (double)(r0 + L::kRows / 2) * p.dy;

  double* ux = lds + L::kUx;
  double* uy = lds + L::kUy;
  double* gx = lds + L::kGx;
  double* gy = lds + L::kGy;
  double* G = lds + L::kG;

  const int D = p.D, F = p.F;
  // Gaussian: the points in reach, a list at a time; all points otherwise
  constexpr bool LIST = WM == WM_GAUSS;
  char* lds_list = (char*)lds + L::kBytes;
  const uint16_t* list = (const uint16_t*)lds_list;
  F64Reach reach{};
  if (LIST) reach = tile_reach<DEG>(p, L::kRows, cx, cy, (float*)lds);
  const int64_t plane = (int64_t)p.W * p.H;

  // The chunk at entry k0 of the current list, which starts at point `base`
  // and has `cnt` entries.
  int64_t base = 0, cnt = 0;
  // Raw chunk data is prefetched into registers one chunk ahead, so that
  // the global-memory latency overlaps the previous chunk's MFMA sweep.
  float pf_x = 0.0f, pf_y = 0.0f;
  float pf_v[L::kValRegs];
  // (point, attribute) of this thread's first feature element and the step
  // to its next one (kThreads elements on)
  const int fk0 = tid / D, fd0 = tid - fk0 * D;
  const int fks = kThreads / D, fds = kThreads - fks * D;
  auto prefetch = [&](int64_t k0) {
    const int kn = (int)((cnt - k0) < KT ? (cnt - k0) : KT);
    if (tid < KT && tid < kn) {
      const int64_t g = LIST ? base + list[k0 + tid] : k0 + tid;
      pf_x = p.pts[2 * g];
      pf_y = p.pts[2 * g + 1];
    }
    if constexpr (!LIST) {
      // consecutive threads read consecutive values of the chunk (coalesced)
      const float* v = p.vals + k0 * (int64_t)D;
#pragma unroll
      for (int it = 0; it < L::kValRegs; ++it) {
        const int e = tid + it * kThreads;
        pf_v[it] = e < kn * D ? v[e] : 0.0f;
      }
    } else {
      // of a listed point, then of the next one; bytes from the list's first
      // point: at most 65,536 rows of 255 floats
      const char* rows = (const char*)(p.vals + base * (int64_t)D);
      int k = fk0, d = fd0;
#pragma unroll
      for (int it = 0; it < L::kValRegs; ++it) {
        pf_v[it] = 0.0f;
        if (k < kn)
          pf_v[it] = *(const float*)(rows + 4u * ((uint32_t)list[k0 + k] * (uint32_t)D +
                                                  (uint32_t)d));
        k += fks;
        d += fds;
        if (d >= D) {
          d -= D;
          ++k;
        }
      }
    }
  };
  // table factors of a chunk: row e / KT of the tile's 16 + 4R rows, point
  // e % KT (consecutive threads read consecutive points of a row)
  double tv[WM == WM_TABLE ? L::kTabRegs : 1];
  auto tab_load = [&](int64_t k0) {
    if constexpr (WM == WM_TABLE) {
#pragma unroll
      for (int it = 0; it < L::kTabRegs; ++it) {
        const int e = tid + it * kThreads;
        const int row = e / KT, k = e % KT;
        if (row < kCols + L::kRows) {
          const int64_t trow = row < kCols ? (int64_t)(c0 + row)
                                           : (int64_t)p.tab_cols + r0 + (row - kCols);
          tv[it] = p.tab[trow * p.tab_n + k0 + k];
        }
      }
    }
  };
  // Gaussian step factors of the tile (exp(-2 s^2) per node step)
  const double sx = p.dx * p.inv_h, sy = p.dy * p.inv_h;
  const double qx = exp(-2.0 * sx * sx), qy = exp(-2.0 * sy * sy);

  // 1. tile-frame coordinates of a chunk, from the prefetched raw data;
  //    the first chunk's now, each later one right after the MFMA sweep of
  //    its predecessor (which does not read them)
  auto put_coords = [&](int kn_) {
    if (tid < KT) {
      double x = 0.0, y = 0.0;
      if (tid < kn_) {
        x = ((double)pf_x - cx) * p.inv_h;
        y = ((double)pf_y - cy) * p.inv_h;
      }
      ux[tid] = x;
      uy[tid] = y;
    }
  };

  // Once over the points in reach; where a node's moments turn out so small
  // that what lies beyond could matter, once more over all points.
  for (;;) {
  doublex4 acc[R][NT];
  double acc4[R][Q4 > 0 ? Q4 : 1];
#pragma unroll
  for (int t = 0; t < R; ++t) {
#pragma unroll
    for (int q = 0; q < NT; ++q) acc[t][q] = doublex4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < (Q4 > 0 ? Q4 : 1); ++q) acc4[t][q] = 0.0;
  }
  // padding features stay zero for the whole sweep
  for (int e = tid; e < (L::kFP - F) * KS; e += kThreads) G[F * KS + e] = 0.0;

  for (int64_t pos = 0; pos < p.n;) {
  base = pos;
  if (LIST) {
    cnt = list_points<kThreads, kListCap>(
        p.pts, p.n, pos, (LdsBytes)lds_list, [&](float x, float y) { return in_reach(reach, x, y); });
  } else {
    cnt = pos = p.n;
  }
  if (cnt == 0) continue;
  prefetch(0);
  put_coords((int)(cnt < KT ? cnt : KT));
  __syncthreads();
  for (int64_t k0 = 0; k0 < cnt; k0 += KT) {
    const int kn = (int)((cnt - k0) < KT ? (cnt - k0) : KT);
    if constexpr (WM == WM_TABLE) {
      // 2a. the chunk's factors: loaded now, stored after the monomials and
      // features, so that their latency overlaps that work
      tab_load(k0);
    } else if constexpr (!INV) {
      // 2a. separable Gaussian factors (WM_STEP: points however far)
      put_gauss<L::kRows>(LIST && p.fine && reach.r2 <= kFineReach2, ux, uy, gx, kn, sx, sy, qx,
                          qy, tid);
    } else {
      // inverse-distance weights do not separate: the tables hold the squared
      // node offsets, and the A operand forms the weight per pair
      const int k = tid & (KT - 1);
      const bool xaxis = (tid & KT) == 0, up = tid < 2 * KT;
      const int mid = (xaxis ? kCols : L::kRows) / 2;
      const double s = xaxis ? sx : sy;
      double* g = (xaxis ? gx : gy) + (up ? mid : 0) * KS + k;
      const double u = xaxis ? ux[k] : uy[k];
      for (int c = 0; c < mid; ++c) {
        const double o = u - (double)(c - (up ? 0 : mid)) * s;
        g[c * KS] = k < kn ? fma(o, o, xaxis ? kMinOffset2<WM> : 0.0) : __builtin_inf();
      }
    }
    // 2b. moment monomials of the tile-frame coordinates
    put_monomials<nmom>(ux, uy, G, lane, wave);
    // 2c. basis x attribute products from the prefetched values
    {
      int k = fk0, d = fd0;
#pragma unroll
      for (int it = 0; it < L::kValRegs; ++it) {
        if (k < KT) {
          const double f = (double)pf_v[it];
          G[(nmom + d) * KS + k] = f;
          if (m >= 3) {
            const double bx = ux[k], by = uy[k];
            G[(nmom + D + d) * KS + k] = bx * f;
            G[(nmom + 2 * D + d) * KS + k] = by * f;
            if (m >= 6) {
              G[(nmom + 3 * D + d) * KS + k] = bx * bx * f;
              G[(nmom + 4 * D + d) * KS + k] = bx * by * f;
              G[(nmom + 5 * D + d) * KS + k] = by * by * f;
            }
          }
        }
        k += fks;
        d += fds;
        if (d >= D) {
          d -= D;
          ++k;
        }
      }
    }
    if constexpr (WM == WM_TABLE) {
#pragma unroll
      for (int it = 0; it < L::kTabRegs; ++it) {   // zero past n
        const int e = tid + it * kThreads;
        const int row = e / KT, k = e % KT;
        if (row < kCols) gx[row * KS + k] = tv[it];
        else if (row < kCols + L::kRows) gy[(row - kCols) * KS + k] = tv[it];
      }
    }
    // next chunk's raw data: in flight during the MFMA sweep
    if (k0 + KT < cnt) prefetch(k0 + KT);
    __syncthreads();

    // 3. MFMA sweep over the chunk
    const int i = lane & 15;        // A row (node column) / B column
    const int kq = (lane >> 4) * 4; // this lane's 4 points in each group of 16
#pragma unroll 1
    for (int kg = 0; kg < KT; kg += 16) {
      // four consecutive doubles of a row as two 16-byte reads (rows start
      // on 16-byte boundaries: KS is even and kg + kq a multiple of 4)
      double ax[4], ay[R][4], bv[Q4 > 0 ? Q4 : NT][4];
      read4(gx + i * KS + kg + kq, ax);
#pragma unroll
      for (int t = 0; t < R; ++t) read4(gy + (wave * R + t) * KS + kg + kq, ay[t]);
      if constexpr (Q4 > 0) {
        // feature 4 q + lane % 4 of the lane's four points
#pragma unroll
        for (int q = 0; q < Q4; ++q) read4(G + (q * 4 + (lane & 3)) * KS + kg + kq, bv[q]);
      } else {
#pragma unroll
        for (int q = 0; q < NT; ++q) read4(G + (q * 16 + i) * KS + kg + kq, bv[q]);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
#pragma unroll
        for (int t = 0; t < R; ++t) {
          const double a = WM == WM_INV1   ? invpow_weight_int<1>(ax[j] + ay[t][j])
                           : WM == WM_INV2 ? invpow_weight_int<2>(ax[j] + ay[t][j])
                           : INV           ? invpow_weight(ax[j] + ay[t][j], p.alpha)
                                           : ax[j] * ay[t][j];
          if constexpr (Q4 > 0) {
#pragma unroll
            for (int q = 0; q < Q4; ++q)
              acc4[t][q] = __builtin_amdgcn_mfma_f64_4x4x4f64(a, bv[q][j], acc4[t][q], 0, 0, 0);
          } else {
#pragma unroll
            for (int q = 0; q < NT; ++q)
              acc[t][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, bv[q][j], acc[t][q], 0, 0, 0);
          }
        }
      }
    }
    if (k0 + KT < cnt) put_coords((int)((cnt - k0 - KT) < KT ? (cnt - k0 - KT) : KT));
    __syncthreads();
  }
  }

  // Epilogue: accumulators -> LDS [node][feature] -> one node per lane,
  // kEpiWaves waves at a time.  (The main loop ended with a barrier.)
  bool again = false;
  const double diag_min = LIST ? reach.scale * kDiagFloor : 0.0;
#pragma unroll 1
  for (int g = 0; g < kWaves; g += kEpiWaves) {
    const bool mine = wave >= g && wave < g + kEpiWaves;
    double* epi = lds + (wave - g) * 16 * R * L::kEpiStride;
    if (mine) {
      if constexpr (Q4 > 0) {
#pragma unroll
        for (int t = 0; t < R; ++t)
#pragma unroll
          for (int q = 0; q < Q4; ++q) {
            // f64 4x4x4 MFMA result: lane holds node 4 ((lane/4) % 4) + lane/16, feature lane%4
            const int node = t * 16 + 4 * ((lane >> 2) & 3) + (lane >> 4);
            const int feat = q * 4 + (lane & 3);
            epi[node * L::kEpiStride + feat] = acc4[t][q];
          }
      } else {
#pragma unroll
        for (int t = 0; t < R; ++t)
#pragma unroll
          for (int q = 0; q < NT; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              // f64 16x16 MFMA result: lane holds row (lane/16 + 4r), column lane%16
              const int node = t * 16 + (lane >> 4) + 4 * r;
              const int feat = q * 16 + (lane & 15);
              epi[node * L::kEpiStride + feat] = acc[t][q][r];
            }
      }
    }
    __syncthreads();
    if (mine)
      again = solve_tile_nodes<DEG, R, EPI>(p, epi, L::kEpiStride, lane, wave, r0, c0, L::kRows,
                                            plane, diag_min);
    __syncthreads();
  }
  // the second time r2 is infinite
  if (!LIST || DEG == 0 || EPI == 2 || !(reach.r2 < __builtin_inf())) break;
  if (!__syncthreads_or(again)) break;
  reach.r2 = __builtin_inf();
  }
}

// One node per lane: the float64 ladder solve of the nodes of one wave.
// Returns whether some node has a diagonal moment below diag_min.
template <int DEG, int R, int EPI>
__device__ bool solve_tile_nodes(const F64Params& p, const double* epi, int stride, int lane,
                                 int wave, int r0, int c0, int rows, int64_t plane,
                                 double diag_min) {
  const int D = p.D;
  bool low = false;
  for (int node = lane; node < 16 * R; node += 64) {
    const int t = node / 16, col = node % 16;
    const int r = r0 + wave * R + t, c = c0 + col;
    if (r >= p.H || c >= p.W) continue;
    // node offset from the anchor, the same expression the weight factors use
    const double ex = (double)(col - kCols / 2) * p.dx * p.inv_h;
    const double ey = (double)(wave * R + t - rows / 2) * p.dy * p.inv_h;
    const int64_t off = (int64_t)r * p.W + c;
    uint8_t code;
    double diag = __builtin_inf();
    if constexpr (EPI == 2)
      code = rigid_node(epi + node * stride, ex, ey, p.h, p.floor_w, p.fields + off, plane);
    else
      code = solve_node<DEG>(epi + node * stride, D, ex, ey, p.tau, p.floor_w, p.fields + off,
                             plane, nullptr, nullptr, 1.0, EPI == 1 ? p.grads + off : nullptr,
                             p.inv_h, &diag);
    if (p.deg_out) p.deg_out[off] = code;
    low = low || diag < diag_min;
  }
  return low;
}

template <int DEG, int NT, int R, int WM, int EPI, int Q4 = 0>
hipError_t launch_impl(const F64Params& prm, hipStream_t s) {
  using L = F64Layout<DEG, NT, R>;
  F64Params p = prm;
  const int tiles_x = (p.W + kCols - 1) / kCols;
  const int tiles_y = (p.H + L::kRows - 1) / L::kRows;
  p.tiles_x = tiles_x;
  const size_t lds_bytes = (size_t)L::kBytes + (WM == WM_GAUSS ? kListB : 0);
  hipError_t e = hipFuncSetAttribute((const void*)fit_f64_kernel<DEG, NT, R, WM, EPI, Q4>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds_bytes);
  if (e != hipSuccess) return e;
  const int64_t blocks = (int64_t)tiles_x * tiles_y;
  hipLaunchKernelGGL((fit_f64_kernel<DEG, NT, R, WM, EPI, Q4>), dim3((unsigned)blocks),
                     dim3(kThreads), lds_bytes, s, p);
  return hipGetLastError();
}

// R (row strips per wave): with one feature tile, where registers allow any,
// what the grid and the sweep make best (f64_tile_strips).
template <int DEG, int NT, int WM, int EPI, int Q4>
hipError_t launch_strips(const F64Params& p, hipStream_t s) {
  if constexpr (NT == 1) {
    switch (f64_tile_strips(p.W, p.H, 4, 1, f64_pair_cycles(p.F, Q4 > 0))) {
      case 1: return launch_impl<DEG, NT, 1, WM, EPI, Q4>(p, s);
      case 2: return launch_impl<DEG, NT, 2, WM, EPI, Q4>(p, s);
      default: return launch_impl<DEG, NT, 4, WM, EPI, Q4>(p, s);
    }
  } else {
    return launch_impl<DEG, NT, NT <= 3 ? 4 : (NT <= 6 ? 2 : 1), WM, EPI, Q4>(p, s);
  }
}

template <int DEG, int NT, int WM, int Q4>
hipError_t launch_epi(const F64Params& p, hipStream_t s) {
  if (p.rigid) {
    if constexpr (DEG == 1 && NT == 1) return launch_strips<DEG, NT, WM, 2, Q4>(p, s);
    return hipErrorInvalidValue;
  }
  return p.grads ? launch_strips<DEG, NT, WM, 1, Q4>(p, s)
                 : launch_strips<DEG, NT, WM, 0, Q4>(p, s);
}

// At most 12 features (constant basis with D <= 11, linear basis with
// D <= 2, the timing-table shapes among them) run the 4x4x4 form: the
// 16x16x4 instruction would carry 4 or more empty feature columns.
template <int DEG, int NT, int WM>
hipError_t launch_nt(const F64Params& p, hipStream_t s) {
  if constexpr (NT == 1 && DEG < 2) {
    if (p.F <= 4) return launch_epi<DEG, NT, WM, 1>(p, s);
    if (p.F <= 8) return launch_epi<DEG, NT, WM, 2>(p, s);
    if (p.F <= 12) return launch_epi<DEG, NT, WM, 3>(p, s);
  }
  return launch_epi<DEG, NT, WM, 0>(p, s);
}

template <int DEG, int WM>
hipError_t launch_deg(const F64Params& p, int nt, hipStream_t s) {
  if constexpr (WM == WM_INV1 || WM == WM_INV2) {
    // the reciprocal forms serve one and two feature tiles, where the
    // weight is most of the vector work per matrix instruction
    return nt == 1 ? launch_nt<DEG, 1, WM>(p, s) : launch_nt<DEG, 2, WM>(p, s);
  } else if constexpr (WM == WM_GAUSS && DEG == 1) {
    // wider Gaussian fits take the two-pass form (f64_use_shape_form)
    return nt == 1 ? launch_nt<DEG, 1, WM>(p, s) : hipErrorInvalidValue;
  } else if constexpr ((WM == WM_TABLE || WM == WM_STEP) && DEG > 0) {
    // and over all points the ones of more than three tiles (f64_sums_all)
    switch (nt) {
      case 1: return launch_nt<DEG, 1, WM>(p, s);
      case 2: return launch_nt<DEG, 2, WM>(p, s);
      case 3: return launch_nt<DEG, 3, WM>(p, s);
      default: return hipErrorInvalidValue;
    }
  } else {
    switch (nt) {
      case 1: return launch_nt<DEG, 1, WM>(p, s);
      case 2: return launch_nt<DEG, 2, WM>(p, s);
      case 3: return launch_nt<DEG, 3, WM>(p, s);
      case 4: return launch_nt<DEG, 4, WM>(p, s);
      case 5: case 6: return launch_nt<DEG, 6, WM>(p, s);
      case 7: case 8: return launch_nt<DEG, 8, WM>(p, s);
      case 9: case 10: case 11: case 12: return launch_nt<DEG, 12, WM>(p, s);
      default: return launch_nt<DEG, 16, WM>(p, s);
    }
  }
}

template <int WM>
hipError_t launch_kind(const F64Params& p, int degree, int nt, hipStream_t s) {
  switch (degree) {
    case 0: return launch_deg<0, WM>(p, nt, s);
    case 1: return launch_deg<1, WM>(p, nt, s);
    default:
      if constexpr (WM == WM_GAUSS) return hipErrorInvalidValue;
      else return launch_deg<2, WM>(p, nt, s);
  }
}

}  // namespace
}  // namespace mls
