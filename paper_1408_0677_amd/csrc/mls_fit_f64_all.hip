// Float64 Gaussian fits over all points, in one pass (mls_fit_f64_kernel.h).
// The factors are copied from tables of every grid column and row, built once
// per launch where they fit the scratch cap, or else formed by the tiles, which
// costs vector instructions that do not overlap the matrix cores.
#include "mls_fit_f64_kernel.h"

namespace mls {
namespace {

// Row r < cols is exp(-((x_k - (x0 + r dx)) / h)^2) over the points k, row cols +
// r the same with y and y0 + r dy; zero for k >= n.  Rows past the grid serve
// the padding nodes of edge tiles.
__global__ __launch_bounds__(256) void gauss_table_kernel(const float* __restrict__ pts, int64_t n,
                                                          int64_t tab_n, int cols, int rows,
                                                          double x0, double dx, double y0,
                                                          double dy, double inv_h,
                                                          double* __restrict__ tab) {
  for (int row = blockIdx.y; row < rows; row += gridDim.y) {
    const bool xr = row < cols;
    const double c = xr ? x0 + (double)row * dx : y0 + (double)(row - cols) * dy;
    for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < tab_n;
         k += (int64_t)gridDim.x * 256) {
      double v = 0.0;
      if (k < n) {
        const double u = ((double)pts[2 * k + (xr ? 0 : 1)] - c) * inv_h;
        v = exp(-(u * u));
      }
      tab[row * tab_n + k] = v;
    }
  }
}

int64_t table_points(int64_t n) { return (n + KT - 1) / KT * KT; }
int table_rows(int cells) { return (cells + kCols - 1) / kCols * kCols; }

}  // namespace

size_t f64_table_bytes(int64_t n, int32_t W, int32_t H) {
  const double bytes = 8.0 * (double)table_points(n) * (double)(table_rows(W) + table_rows(H));
  return bytes <= (double)kF64TableCap ? (size_t)bytes : 0;
}

hipError_t launch_fit_f64_all(const F64Params& prm, int degree, int nt, double* tab,
                              hipStream_t s) {
  F64Params p = prm;
  if (!tab) return launch_kind<WM_STEP>(p, degree, nt, s);
  p.tab = tab;
  p.tab_n = table_points(p.n);
  p.tab_cols = table_rows(p.W);
  const int rows = p.tab_cols + table_rows(p.H);
  const int64_t per_row = (p.tab_n + 255) / 256;
  hipLaunchKernelGGL(gauss_table_kernel,
                     dim3((unsigned)(per_row < 64 ? per_row : 64),
                          (unsigned)(rows < 65535 ? rows : 65535)),
                     dim3(256), 0, s, p.pts, p.n, p.tab_n, p.tab_cols, rows, p.x0, p.dx, p.y0,
                     p.dy, p.inv_h, tab);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? launch_kind<WM_TABLE>(p, degree, nt, s) : e;
}

}  // namespace mls
