// Two-pass (shape-function) float64 MLS fit with the Gaussian weight
// (Muelder et al., Sec. 3.3).  The field at node p is
//   field_d(p) = y_p^T R_t,d = sum_i w_ip (y_p^T b_t(u_i)) f_i,d,
// y_p the tile-frame coefficients of the node's shape function
// (mls_solve.h).  Pass 1 contracts the weights with the moment monomials only
// and solves every node's ladder for y_p; pass 2 streams the points again and
// contracts the effective weights w_ip (y_p^T b_t(u_i)), formed per pair in
// float64, with the attributes.  The contraction width falls from
// n_mom + m D to n_mom + D columns (linear basis, 13 attributes: 45 to 19),
// for a second set of weights of 16 (linear) or 28 (quadratic) cycles per 64
// pairs.  All of it in float64, as the one-pass kernel (mls_fit_f64.hip).
// The slopes of the local fits are two more such contractions, with the rows
// of e_1 and e_2 in the place of y_p, over the same chunk in LDS; the fields
// are computed as without them, bit for bit.
//
// Bound: the float64 matrix instructions (64 cycles per 16 columns, 17 per 4
// with the four-block 4x4x4 form, and 64 node-point pairs), and the vector
// work beside them, which does not run at the same time on a SIMD.  A
// workgroup owns 16 x 4R nodes; each wave R strips of 16 nodes, which it also
// solves by itself, one node per lane, between the passes.  Three workgroups
// share a compute unit, so that one's chunk production and solves run under
// the others' matrix instructions (two, without spills, measured 1,085 us
// where three take 1,034).
// 5,000 points, 13 attributes, h = 0.03, 1024^2, linear: 7,890 -> 1,030 us,
// of which the reach gives 6.1x and the rest is this form.  Counters there:
// matrix instructions busy 44% and vector instructions 27% of the SIMDs'
// cycles, 37.2M matrix instructions; 170 MB written, 56 of it the outputs and the
// rest registers that three workgroups a unit spill.  3,001 points, 5 attributes, quadratic,
// 517 x 389, with slopes: 1,500 -> 854 us (930 with a sweep for each output).
#include "mls_fit_f64.h"

namespace mls {
namespace {

template <int DEG, int NT, int QD, int R, int NE>
struct ShapeLayout {
  static constexpr int m = DEG == 1 ? 3 : 6;
  static constexpr int nmom = DEG == 1 ? 6 : 15;
  static constexpr int kRows = kWaves * R;
  static constexpr int kNodes = 16 * kRows;
  static constexpr int kFP1 = DEG == 1 ? 8 : 16;            // moment columns
  static constexpr int kFP2 = QD > 0 ? 4 * QD : 16 * NT;    // attributes per slab
  static constexpr int kFG = kFP1 > kFP2 ? kFP1 : kFP2;
  static constexpr int kValRegs = (KT * kFP2 + kThreads - 1) / kThreads;
  // coordinates of two chunks: x of one, y of it, then the other's
  static constexpr int kU = 0;
  static constexpr int kGx = kU + 4 * KT;
  static constexpr int kGy = kGx + kCols * KS;
  static constexpr int kG = kGy + kRows * KS;
  static constexpr int kChunk = kG + kFG * KS;
  // between the passes: the moments of every node, odd stride
  static constexpr int kEpiStride = kFP1 + 1;
  static constexpr int kEpi = kNodes * kEpiStride;
  // shape coefficients (NE rows: the value's, then the slopes'), odd stride,
  // and degree codes
  static constexpr int kYStride = (NE * m) | 1;
  static constexpr int kY = kChunk > kEpi ? kChunk : kEpi;
  static constexpr int kDoubles = kY + kNodes * kYStride;
  static constexpr int kCode0 = 8 * kDoubles;
  static constexpr int kList0 = kCode0 + kNodes;
  static constexpr int kBytes = kList0 + kListB;
};

// NE: 1 fields, 3 fields and slopes.
template <int DEG, int NT, int QD, int R, int NE>
__global__ __launch_bounds__(kThreads, NT > 1 || NE > 1 ? 2 : 3)
void fit_f64_shape_kernel(F64Params p) {
  using L = ShapeLayout<DEG, NT, QD, R, NE>;
  constexpr int m = L::m;
  extern __shared__ double lds[];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c0 = (blockIdx.x % p.tiles_x) * kCols;
  const int r0 = (blockIdx.x / p.tiles_x) * L::kRows;
  const double cx = p.x0 + (double)(c0 + kCols / 2) * p.dx;
  const double cy = p.y0 + (double)(r0 + L::kRows / 2) * p.dy;
  const int64_t plane = (int64_t)p.W * p.H;
  const int D = p.D;

  // coordinates of chunk c (its number's parity picks the buffer)
  auto ux = [&](int c) { return lds + L::kU + (c & 1) * 2 * KT; };
  auto uy = [&](int c) { return ux(c) + KT; };
  double* gx = lds + L::kGx;
  double* gy = lds + L::kGy;
  double* G = lds + L::kG;
  double* ybuf = lds + L::kY;
  uint8_t* codes = (uint8_t*)lds + L::kCode0;
  char* lds_list = (char*)lds + L::kList0;
  const uint16_t* list = (const uint16_t*)lds_list;

  F64Reach reach = tile_reach<DEG>(p, L::kRows, cx, cy, (float*)lds);
  const double sx = p.dx * p.inv_h, sy = p.dy * p.inv_h;
  const double qx = exp(-2.0 * sx * sx), qy = exp(-2.0 * sy * sy);

  bool fine = false;            // gauss_steps
  int kept = 0, segments = 0;   // the last list; the lists of pass 1
  int64_t base = 0;
  auto next_list = [&](int64_t& pos) {
    base = pos;
    kept = list_points<kThreads, kListCap>(
        p.pts, p.n, pos, (LdsBytes)lds_list, [&](float x, float y) { return in_reach(reach, x, y); });
  };

  // raw data of a chunk, one chunk ahead in registers
  float pf_x = 0.0f, pf_y = 0.0f;
  float pf_v[L::kValRegs];
  auto prefetch_xy = [&](int k0) {
    if (tid < KT && k0 + tid < kept) {
      const int64_t g = base + list[k0 + tid];
      pf_x = p.pts[2 * g];
      pf_y = p.pts[2 * g + 1];
    }
  };
  // tile-frame coordinates of a chunk from the prefetched raw data
  auto put_coords = [&](int c) {
    if (tid < KT) {
      const bool in = c * KT + tid < kept;
      ux(c)[tid] = in ? ((double)pf_x - cx) * p.inv_h : 0.0;
      uy(c)[tid] = in ? ((double)pf_y - cy) * p.inv_h : 0.0;
    }
  };
  // Once over the points in reach; where a node's moments turn out so small
  // that what lies beyond could matter, once more over all points.
  for (;;) {
    // ---- pass 1: moments ----
    doublex4 acc[R];
    double acc4[R][2];
#pragma unroll
    for (int t = 0; t < R; ++t) {
      acc[t] = doublex4{0.0, 0.0, 0.0, 0.0};
      acc4[t][0] = acc4[t][1] = 0.0;
    }
    for (int e = tid; e < (L::kFP1 - L::nmom) * KS; e += kThreads) G[L::nmom * KS + e] = 0.0;
    fine = p.fine && reach.r2 <= kFineReach2;
    segments = 0;
    for (int64_t pos = 0; pos < p.n; ++segments) {
      next_list(pos);
      if (kept == 0) continue;
      prefetch_xy(0);
      put_coords(0);
      __syncthreads();
      for (int c = 0; c * KT < kept; ++c) {
        const int kn = kept - c * KT < KT ? kept - c * KT : KT;
        put_monomials<L::nmom>(ux(c), uy(c), G, lane, wave);
        put_gauss<L::kRows>(fine, ux(c), uy(c), gx, kn, sx, sy, qx, qy, tid);
        prefetch_xy((c + 1) * KT);
        __syncthreads();
        const int i = lane & 15;
        const int kq = (lane >> 4) * 4;
#pragma unroll 1
        for (int kg = 0; kg < KT; kg += 16) {
          double ax[4], ay[R][4], bv[2][4];
          read4(gx + i * KS + kg + kq, ax);
#pragma unroll
          for (int t = 0; t < R; ++t) read4(gy + (wave * R + t) * KS + kg + kq, ay[t]);
          if constexpr (DEG == 1) {
            read4(G + (lane & 3) * KS + kg + kq, bv[0]);
            read4(G + (4 + (lane & 3)) * KS + kg + kq, bv[1]);
          } else {
            read4(G + i * KS + kg + kq, bv[0]);
          }
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int t = 0; t < R; ++t) {
              const double a = ax[j] * ay[t][j];
              if constexpr (DEG == 1) {
                acc4[t][0] = __builtin_amdgcn_mfma_f64_4x4x4f64(a, bv[0][j], acc4[t][0], 0, 0, 0);
                acc4[t][1] = __builtin_amdgcn_mfma_f64_4x4x4f64(a, bv[1][j], acc4[t][1], 0, 0, 0);
              } else {
                acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, bv[0][j], acc[t], 0, 0, 0);
              }
            }
        }
        put_coords(c + 1);
        __syncthreads();
      }
    }
    // moments -> LDS [node][column]; a wave solves its own nodes, one per lane
    double* epi = lds + wave * 16 * R * L::kEpiStride;
#pragma unroll
    for (int t = 0; t < R; ++t) {
      if constexpr (DEG == 1) {
        // f64 4x4x4 result: lane holds node 4 ((lane/4) % 4) + lane/16, column lane%4
        const int node = t * 16 + 4 * ((lane >> 2) & 3) + (lane >> 4);
        epi[node * L::kEpiStride + (lane & 3)] = acc4[t][0];
        epi[node * L::kEpiStride + 4 + (lane & 3)] = acc4[t][1];
      } else {
        // f64 16x16 result: lane holds rows lane/16 + 4r, column lane%16
#pragma unroll
        for (int r = 0; r < 4; ++r)
          epi[(t * 16 + (lane >> 4) + 4 * r) * L::kEpiStride + (lane & 15)] = acc[t][r];
      }
    }
    __syncthreads();
    bool again = false;
    if (lane < 16 * R) {
      const int t = lane / 16, col = lane % 16;
      const int row = wave * R + t;
      const double ex = (double)(col - kCols / 2) * p.dx * p.inv_h;
      const double ey = (double)(row - L::kRows / 2) * p.dy * p.inv_h;
      Ladder<DEG> lad;
      const int code = ladder_solve<DEG>(epi + lane * L::kEpiStride, ex, ey, p.tau, p.floor_w,
                                         1.0, lad);
      const bool in = r0 + row < p.H && c0 + col < p.W;
      again = in && code != 255 && lad.diag < reach.scale * kDiagFloor;
      const int node = row * kCols + col;
#pragma unroll
      for (int j = 0; j < m; ++j) ybuf[node * L::kYStride + j] = code == 255 ? 0.0 : lad.y[j];
      if constexpr (NE == 3) {
#pragma unroll
        for (int e = 1; e < 3; ++e) {
          double ya[m];
          if (code != 255) slope_row<DEG>(lad, e, ya);
#pragma unroll
          for (int j = 0; j < m; ++j)
            ybuf[node * L::kYStride + e * m + j] = code == 255 ? 0.0 : ya[j];
        }
      }
      codes[node] = (uint8_t)code;
      if (p.deg_out && in) p.deg_out[(int64_t)(r0 + row) * p.W + c0 + col] = (uint8_t)code;
    }
    if (!(reach.r2 < __builtin_inf())) break;   // every point was summed
    if (!__syncthreads_or(again)) break;
    reach.r2 = __builtin_inf();
  }
  __syncthreads();

  // ---- pass 2: effective weights x attributes, a slab at a time ----
  // In the 16-column form matrix row i is node column 4 (i % 4) + i / 4, so
  // that a lane ends with four consecutive columns of a node row.
  const int i = lane & 15;
  const int ci = QD > 0 ? i : 4 * (i & 3) + (i >> 2);
  const int kq = (lane >> 4) * 4;
  // Slopes: the three outputs share a sweep's loads and weights (EF = 3; 5,000
  // points, 8 attributes, 1024^2 2,044 -> 1,938 us, quadratic with 4 2,707 ->
  // 2,491) unless their accumulators and coefficients pass the registers.
  constexpr int EF = NE > 1 && DEG == 1 && R == 4 && (QD == 0 || QD == 3) ? 1 : NE;
  double yv[EF][R][m];
  auto load_y = [&](int e0) {
#pragma unroll
    for (int e = 0; e < EF; ++e)
#pragma unroll
      for (int t = 0; t < R; ++t)
#pragma unroll
        for (int j = 0; j < m; ++j)
          yv[e][t][j] = ybuf[((wave * R + t) * kCols + ci) * L::kYStride + (e0 + e) * m + j];
  };
  if (EF == NE) load_y(0);
  for (int d0 = 0; d0 < D; d0 += L::kFP2) {
    const int nv = D - d0 < L::kFP2 ? D - d0 : L::kFP2;
    // element e = tid + it kThreads of a chunk's values: point e / nv
    const int fk0 = tid / nv, fd0 = tid - fk0 * nv;
    const int fks = kThreads / nv, fds = kThreads - fks * nv;
    auto prefetch_values = [&](int k0) {
      int k = fk0, d = fd0;
#pragma unroll
      for (int it = 0; it < L::kValRegs; ++it) {
        // bytes from the list's first point: at most 65,536 rows of 83 floats
        const char* rows = (const char*)(p.vals + base * (int64_t)D + d0);
        pf_v[it] = 0.0f;
        if (k < KT && k0 + k < kept)
          pf_v[it] = *(const float*)(rows + 4u * ((uint32_t)list[k0 + k] * (uint32_t)D +
                                                  (uint32_t)d));
        k += fks;
        d += fds;
        if (d >= nv) {
          d -= nv;
          ++k;
        }
      }
    };
    auto put_values = [&]() {
      int k = fk0, d = fd0;
#pragma unroll
      for (int it = 0; it < L::kValRegs; ++it) {
        if (k < KT) G[d * KS + k] = (double)pf_v[it];
        k += fks;
        d += fds;
        if (d >= nv) {
          d -= nv;
          ++k;
        }
      }
    };
    doublex4 acc[NE][R][NT];
    double acc4[NE][R][QD > 0 ? QD : 1];
#pragma unroll
    for (int e = 0; e < NE; ++e)
#pragma unroll
      for (int t = 0; t < R; ++t) {
#pragma unroll
        for (int q = 0; q < NT; ++q) acc[e][t][q] = doublex4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int q = 0; q < (QD > 0 ? QD : 1); ++q) acc4[e][t][q] = 0.0;
      }
    for (int e = tid; e < (L::kFP2 - nv) * KS; e += kThreads) G[nv * KS + e] = 0.0;
    for (int64_t pos = 0; pos < p.n;) {
      if (segments == 1) pos = p.n;   // the list of pass 1 is still there
      else next_list(pos);
      if (kept == 0) continue;
      prefetch_xy(0);
      prefetch_values(0);
      put_coords(0);
      __syncthreads();
      for (int c = 0; c * KT < kept; ++c) {
        const int kn = kept - c * KT < KT ? kept - c * KT : KT;
        put_values();
        put_gauss<L::kRows>(fine, ux(c), uy(c), gx, kn, sx, sy, qx, qy, tid);
        prefetch_xy((c + 1) * KT);
        prefetch_values((c + 1) * KT);
        __syncthreads();
#pragma unroll
        for (int e0 = 0; e0 < NE; e0 += EF) {
        if (EF < NE) load_y(e0);
#pragma unroll 1
        for (int kg = 0; kg < KT; kg += 16) {
          double ax[4], ay[R][4], bx[4], by[4], bv[QD > 0 ? QD : NT][4];
          read4(gx + ci * KS + kg + kq, ax);
          read4(ux(c) + kg + kq, bx);
          read4(uy(c) + kg + kq, by);
#pragma unroll
          for (int t = 0; t < R; ++t) read4(gy + (wave * R + t) * KS + kg + kq, ay[t]);
          if constexpr (QD > 0) {
#pragma unroll
            for (int q = 0; q < QD; ++q) read4(G + (q * 4 + (lane & 3)) * KS + kg + kq, bv[q]);
          } else {
#pragma unroll
            for (int q = 0; q < NT; ++q) read4(G + (q * 16 + i) * KS + kg + kq, bv[q]);
          }
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int t = 0; t < R; ++t) {
              const double w = ax[j] * ay[t][j];
#pragma unroll
              for (int e = 0; e < EF; ++e) {
                const double* y = yv[e][t];
                double sh;
                if constexpr (DEG == 1) {
                  sh = fma(y[2], by[j], fma(y[1], bx[j], y[0]));
                } else {
                  const double s1 = fma(y[3], bx[j], fma(y[4], by[j], y[1]));
                  const double s2 = fma(y[5], by[j], y[2]);
                  sh = fma(bx[j], s1, fma(by[j], s2, y[0]));
                }
                const double a = w * sh;
                if constexpr (QD > 0) {
#pragma unroll
                  for (int q = 0; q < QD; ++q)
                    acc4[e0 + e][t][q] = __builtin_amdgcn_mfma_f64_4x4x4f64(
                        a, bv[q][j], acc4[e0 + e][t][q], 0, 0, 0);
                } else {
#pragma unroll
                  for (int q = 0; q < NT; ++q)
                    acc[e0 + e][t][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                        a, bv[q][j], acc[e0 + e][t][q], 0, 0, 0);
                }
              }
            }
        }
        }
        put_coords(c + 1);
        __syncthreads();
      }
    }
    // fields: the accumulators are the values; slopes: over h
#pragma unroll
    for (int e = 0; e < NE; ++e) {
    // attribute d's plane of this output
    auto out_plane = [&](int d) {
      return e == 0 ? p.fields + (int64_t)(d0 + d) * plane
                    : p.grads + (int64_t)(2 * (d0 + d) + e - 1) * plane;
    };
    const double unit = e == 0 ? 1.0 : p.inv_h;
#pragma unroll
    for (int t = 0; t < R; ++t) {
      const int row = wave * R + t, rg = r0 + row;
      if (rg >= p.H) continue;
      if constexpr (QD > 0) {
        const int col = 4 * ((lane >> 2) & 3) + (lane >> 4), cg = c0 + col;
        const bool und = codes[row * kCols + col] == 255;
#pragma unroll
        for (int q = 0; q < QD; ++q) {
          const int d = 4 * q + (lane & 3);
          if (d < nv && cg < p.W)
            out_plane(d)[(int64_t)rg * p.W + cg] =
                und ? __builtin_nanf("") : (float)(acc4[e][t][q] * unit);
        }
      } else {
        const int col = 4 * (lane >> 4), cg = c0 + col;
        const uint8_t* code = codes + row * kCols + col;
#pragma unroll
        for (int q = 0; q < NT; ++q) {
          const int d = 16 * q + i;
          if (d >= nv) continue;
          float* out = out_plane(d) + (int64_t)rg * p.W + cg;
          float v[4];
#pragma unroll
          for (int r = 0; r < 4; ++r)
            v[r] = code[r] == 255 ? __builtin_nanf("") : (float)(acc[e][t][q][r] * unit);
          if (p.vec4) {
            if (cg < p.W) *(float4*)out = make_float4(v[0], v[1], v[2], v[3]);
          } else {
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (cg + r < p.W) out[r] = v[r];
          }
        }
      }
    }
    }
  }
}

template <int DEG, int NT, int QD, int R, int NE>
hipError_t launch_impl(const F64Params& prm, hipStream_t s) {
  using L = ShapeLayout<DEG, NT, QD, R, NE>;
  F64Params p = prm;
  p.tiles_x = (p.W + kCols - 1) / kCols;
  const int64_t blocks = (int64_t)p.tiles_x * ((p.H + L::kRows - 1) / L::kRows);
  const void* fn = (const void*)fit_f64_shape_kernel<DEG, NT, QD, R, NE>;
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, L::kBytes);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((fit_f64_shape_kernel<DEG, NT, QD, R, NE>), dim3((unsigned)blocks),
                     dim3(kThreads), L::kBytes, s, p);
  return hipGetLastError();
}

template <int DEG, int NT, int QD, int NE>
hipError_t launch_tiles(const F64Params& p, hipStream_t s) {
  // (the slopes do not enter: the tiles' frames are those of a call without, and
  // so are the fields' bits)
  const int attrs = p.D < 48 ? p.D : 48;
  const int cycles = f64_pair_cycles(moment_terms(DEG), DEG == 1) +
                     f64_pair_cycles(attrs, true) + (DEG == 1 ? 12 : 24);
  switch (f64_tile_strips(p.W, p.H, DEG == 1 ? 4 : 2, 2, cycles)) {
    case 1: return launch_impl<DEG, NT, QD, 1, NE>(p, s);
    case 2: return launch_impl<DEG, NT, QD, 2, NE>(p, s);
    default:
      // quadratic fits hold twice the shape coefficients per strip: with two
      // strips a wave keeps them all in registers (2,500 points, 5
      // attributes, 700 x 500: 760 us with four strips, 702 with two; 5,000
      // points, 13 attributes, 1000 x 300: 784 and 662)
      if constexpr (DEG == 1) return launch_impl<DEG, NT, QD, 4, NE>(p, s);
      else return hipErrorInvalidValue;
  }
}

// Attributes go in slabs of up to 48 (16 with slopes, whose accumulators are
// three times as many).
template <int DEG, int NE>
hipError_t launch_deg(const F64Params& p, hipStream_t s) {
  if (p.D <= 4) return launch_tiles<DEG, 1, 1, NE>(p, s);
  if (p.D <= 8) return launch_tiles<DEG, 1, 2, NE>(p, s);
  if (p.D <= 12) return launch_tiles<DEG, 1, 3, NE>(p, s);
  if constexpr (NE == 1) {
    if (p.D > 32) return launch_tiles<DEG, 3, 0, NE>(p, s);
    if (p.D > 16) return launch_tiles<DEG, 2, 0, NE>(p, s);
  }
  return launch_tiles<DEG, 1, 0, NE>(p, s);
}

}  // namespace

// Cycles per 64 node-point pairs of the two forms: matrix instructions (64
// per 16 columns, 17 per 4), the weights, and for the second pass its share
// of a chunk's production.  Every quadratic fit and linear fits of 4
// attributes or more take the two-pass form; the slopes do not enter, so that
// the fields of a call with slopes are those of one without.
bool f64_use_shape_form(int degree, int D) {
  if (degree < 1) return false;
  const int F = moment_terms(degree) + basis_terms(degree) * D;
  const int one = degree < 2 && F <= 12 ? 17 * ((F + 3) / 4) : 64 * ((F + 15) / 16);
  const int attrs = D <= 12 ? 17 * ((D + 3) / 4) : 64 * ((D + 15) / 16);
  const int two = (degree == 1 ? 34 + 16 : 64 + 28) + attrs + 16;
  return two < one;
}

hipError_t launch_fit_f64_shape(const F64Params& p, int degree, hipStream_t s) {
  if (p.grads)
    return degree == 1 ? launch_deg<1, 3>(p, s) : launch_deg<2, 3>(p, s);
  return degree == 1 ? launch_deg<1, 1>(p, s) : launch_deg<2, 1>(p, s);
}

}  // namespace mls
