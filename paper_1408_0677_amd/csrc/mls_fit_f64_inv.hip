// Float64 fits with the inverse-distance weight (mls_fit_f64_kernel.h).
#include "mls_fit_f64_kernel.h"

namespace mls {

hipError_t launch_fit_f64_inv(const F64Params& p, int degree, int nt, hipStream_t s) {
  if (nt <= 2 && p.alpha == 1.0) return launch_kind<WM_INV1>(p, degree, nt, s);
  if (nt <= 2 && p.alpha == 2.0) return launch_kind<WM_INV2>(p, degree, nt, s);
  return launch_kind<WM_INV>(p, degree, nt, s);
}

}  // namespace mls
