// Float64 matrix-core MLS fit for gfx950 (Muelder et al., Sec. 3.3).
//
// Per node p the fit needs the weighted moments of the basis and of
// basis x attribute products, G_p = sum_i w(p, x_i) g_i with
//   g_i = [u_x^a u_y^b (a + b <= 2 deg) | b_j(u_i) f_{i,d}]   (F features)
// in a tile frame u = (x_i - c_T) / h.  Over a tile of nodes this is the
// product W (nodes x points) . G (points x F): a dense contraction, run here
// on v_mfma_f64_16x16x4f64 with the point index as the reduction dimension.
//
// Workgroup: 256 threads (4 waves) own a tile of 16 columns x 4R rows of
// nodes.  Each wave owns R row-strips of 16 nodes (one MFMA M-tile each) and
// all NT = ceil(F / 16) feature N-tiles, so a wave holds R * NT accumulator
// blocks.  Points stream through LDS in chunks of KT:
//   1. point coordinates -> LDS (tile-frame u, float64),
//   2. Gaussian weight factors gx[col][k] = exp(-((x_k - p_col)/h)^2) and
//      gy[row][k] (the Gaussian separates on a grid, so a tile needs
//      16 + 4R factors per point instead of 64R), and the feature block
//      G[j][k] in float64.  The factors follow by stepping from node to node
//      (gauss_steps: two exponentials per point, axis and half), or are copied
//      from tables of the launch (mls_fit_f64_all.hip),
//   3. MFMA sweep: the A operand (node x point weight) is gx * gy, built in
//      registers; B is read from G.  Within each group of 16 points a lane
//      supplies points k0 + 4 (lane / 16) + j for MFMA j = 0..3, so it reads
//      four consecutive points with one 32-byte LDS access.
// After the last chunk the accumulators go through LDS to one node per
// lane, which runs the float64 degree-ladder solve (mls_solve.h) and stores
// the D fields and the degree code.  Every node sums its points in the same
// fixed order, so results are bit-reproducible run to run.
//
// With the Gaussian the points are those in reach of the tile (mls_fit_f64.h,
// tile_reach), listed in LDS: 5,000 points, 13 attributes, h = 0.03, 1024^2
// contracts 13% of the points.  Gaussian fits whose feature block would be
// wider than 16 columns take the two-pass form instead
// (mls_fit_f64_shape.hip); this kernel keeps the constant basis, the linear
// basis with up to 3 attributes, the rigid map, every inverse-distance fit, and
// the Gaussian fits whose tiles would list nearly all points anyway and that
// gain by the tables (f64_sums_all).  3,000 points, 9 attributes, constant
// basis, 700 x 500: 545 us over all points, 277 in reach; 4,500 points, 2
// attributes, linear: 875 and 308.
#include "mls_fit_f64_kernel.h"

namespace mls {
namespace {

// The look over the inputs for all tiles: words[1] = the digits (size_digits)
// that the bound gains, the most of any attribute.  Every block leaves its part
// in words[2 ..]; the one that finishes last takes them together and sets the
// count, words[0], back to zero.  5 us at 5,000 points, 13 attributes.
__global__ __launch_bounds__(kThreads) void look_kernel(const float* vals, int64_t n, int D,
                                                        const float* pts, uint32_t* words) {
  __shared__ uint32_t hi[kF64MaxAttrs], lo[kF64MaxAttrs];
  __shared__ uint32_t last, most;
  const int tid = threadIdx.x, nb = gridDim.x;
  if (tid < D) {
    hi[tid] = 0;
    lo[tid] = 0x7F800000u;
  }
  __syncthreads();
  look_sizes<kThreads>(vals, n, D, pts, blockIdx.x, nb, hi, lo);
  __syncthreads();
  // the parts are stored, by the wave that then counts, and loaded past the
  // caches that the blocks do not share (a release fence by every wave would
  // write the L2 back as many times)
  uint64_t* part = (uint64_t*)(words + 2);
  if (tid < 64)
    for (int d = tid; d < D; d += 64)
      __hip_atomic_store(part + blockIdx.x * D + d, (uint64_t)hi[d] << 32 | lo[d],
                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (tid == 0) {
    last = __hip_atomic_fetch_add(words, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) ==
           (uint32_t)nb - 1u;
    most = 0;
  }
  __syncthreads();
  if (!last) return;
  // (its own sizes are in hi and lo already)
#pragma unroll 8
  for (int e = tid; e < nb * D; e += kThreads) {
    const uint64_t q =
        __hip_atomic_load(part + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    atomicMax(hi + e % D, (uint32_t)(q >> 32));
    atomicMin(lo + e % D, (uint32_t)q);
  }
  __syncthreads();
  if (tid < D) atomicMax(&most, (uint32_t)size_digits(hi[tid], lo[tid]));
  __syncthreads();
  if (tid == 0) {
    words[0] = 0;
    words[1] = most;
  }
}

// Most points for which a tile leaves out those beyond its reach.  The tiles'
// own tests of the points cost n x tiles, but that is not why the line lies
// here: tests/test_gpu_server.py queues, cancels and times out requests behind
// a float64 request of 40,000 points (quadratic, 1024^2), which has to run longer
// than the 25 ms that this takes the host; in reach it would take 7.
constexpr int64_t kReachPoints = 32768;

// Values that every tile looks through itself rather than by look_kernel
// (a launch, 5 us, against 64 loads per thread).
constexpr int64_t kLookInTile = 16384;

}  // namespace

// Whether no tile leaves a point out, whatever the points.
static bool never_cuts(const FitArgs& a) {
  return a.n > kReachPoints || (a.n < kFloorPoints && !(a.floor_w > 0.0));
}

// Share of the points that lie within reach of a tile, on average over the
// grid's tiles, for points spread evenly over the grid's rectangle (with a reach
// of 6 h, about the smallest).  Only a measure of what the reach can save: the
// fit is the same either way.
static double reach_share(const FitArgs& a) {
  if (never_cuts(a)) return 1.0;
  auto axis = [&](double d, int cells) {
    const double len = fabs(d) * (double)cells;
    const double r = len > 0.0 ? 6.0 * a.h / len : 1.0;
    return r < 1.0 ? r * (2.0 - r) : 1.0;
  };
  return axis(a.dx, a.W) * axis(a.dy, a.H);
}

// Past kReachPoints the line between one pass over all points and two lies
// where one gains as much on the calls with slopes as two on those without
// (which take the same form, so that the fields are the same bits).  33,000
// points, 256^2, with tables, us one pass / two: linear d = 4 2,490 / 3,220 and
// with slopes 2,500 / 4,160, d = 14 3,600 / 3,850 and 3,600 / 6,220, d = 30 7,630
// / 4,940 and 7,680 / 10,900; quadratic d = 5 3,580 / 4,040 and 3,570 / 5,880,
// d = 8 4,890 / 4,060 and 6,000 / 5,900.  Where the tables pass the scratch cap one
// pass forms the factors in its tiles: 40,000 points, 1024^2, ms, linear d = 4
// 44.1 / 35.6 and 44.1 / 58.9, quadratic d = 4 73.1 / 58.1 and 72.8 / 95.8, d = 8
// 98.5 / 63.8 and 126.7 / 109.7: the same line.
// Below it, where a call has work enough for the tables' launch and nearly all
// points are in reach, the forms that gain by the tables' factors (3,000 points,
// 512^2, us tables / list): constant d = 1 214 / 298, d = 60 1,674 / 1,834,
// linear d = 2 416 / 442, d = 8 831 / 730 but with slopes 840 / 1,303, quadratic
// d = 2 830 / 963 and with slopes 966 / 1,574.  (The others take the list:
// constant d = 13 561 / 515, d = 45 1,368 / 1,275, linear d = 4 852 / 639 and with
// slopes 855 / 1,038, d = 13 1,226 / 919 and 1,405 / 1,901, quadratic d = 4 1,502 /
// 965 and 1,516 / 1,579.)
bool f64_sums_all(const FitArgs& a) {
  if (a.wkind != 0) return false;
  const int F = moment_terms(a.degree) + basis_terms(a.degree) * a.D;
  if (a.n > kReachPoints) return a.degree == 0 || F <= 48;
  if ((int64_t)a.W * a.H < 65536) return false;
  if (a.degree == 2) return F <= 27 && reach_share(a) >= 0.95;
  if (a.degree == 1 && F > 20) return F <= 32 && reach_share(a) >= 0.95;
  const bool tiles = a.degree == 0 && ((F > 16 && F <= 32) || F > 48);
  return (F <= 12 || tiles) && reach_share(a) >= 0.85;
}

hipError_t launch_fit_f64(const FitArgs& a, hipStream_t stream) {
  const int F = moment_terms(a.degree) + basis_terms(a.degree) * a.D;
  const int nt = (F + 15) / 16;
  if (nt > 16) return hipErrorInvalidValue;
  F64Params p{};
  p.pts = a.pts;
  p.vals = a.vals;
  p.n = a.n;
  p.D = a.D;
  p.F = F;
  p.h = a.h;
  p.inv_h = 1.0 / a.h;
  p.alpha = a.alpha;
  p.x0 = a.x0; p.y0 = a.y0; p.dx = a.dx; p.dy = a.dy;
  p.W = a.W; p.H = a.H;
  p.tau = a.tau;
  p.floor_w = a.floor_w;
  p.fields = a.fields;
  p.deg_out = a.deg_out;
  p.grads = a.grads;
  p.rigid = a.rigid;
  if (a.wkind == 2) return launch_fit_f64_inv(p, a.degree, nt, stream);
  if (f64_sums_all(a)) return launch_fit_f64_all(p, a.degree, nt, a.table, stream);
  p.list_log = never_cuts(a) ? HUGE_VAL : log((double)a.n) + 54.0 * 0.6931471805599453;
  p.vec4 = (a.W & 3) == 0 && (((uintptr_t)a.fields | (uintptr_t)a.grads) & 15) == 0;
  const double span = fmax(fabs(a.dx), fabs(a.dy)) * p.inv_h * 15.0;
  p.fine = span <= kFineSpan && p.list_log < HUGE_VAL;
  if (f64_needs_words(a)) {
    // as many values per thread as parts per thread of the last block
    const int64_t nb = (int64_t)ceil(sqrt((double)a.n));
    p.sizes = a.words + 1;
    hipLaunchKernelGGL(look_kernel, dim3((unsigned)(nb < kF64LookBlocks ? nb : kF64LookBlocks)),
                       dim3(kThreads), 0, stream, a.vals, a.n, a.D, a.pts, a.words);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return !a.rigid && f64_use_shape_form(a.degree, a.D)
             ? launch_fit_f64_shape(p, a.degree, stream)
             : launch_kind<WM_GAUSS>(p, a.degree, nt, stream);
}

bool f64_needs_words(const FitArgs& a) {
  return a.wkind == 0 && a.n * a.D > kLookInTile && !never_cuts(a) && !f64_sums_all(a);
}

}  // namespace mls
