// Two-pass (shape-function) bfloat16 fits: instantiations.
#include "mls_fit_lp.h"

namespace mls {

hipError_t launch_lp_shape(const LPParams& p, int deg, int ntv, int terms, hipStream_t s) {
  switch (terms) {
    case 1: return launch_shape_deg<1>(p, deg, ntv, s);
    case 2: return launch_shape_deg<2>(p, deg, ntv, s);
    default: return launch_shape_deg<3>(p, deg, ntv, s);
  }
}

}  // namespace mls
