// Two-pass (shape-function) 16-bit fits: float16 instantiations.
#include "mls_fit_lp.h"

namespace mls {

hipError_t launch_shape_fp16(const LPParams& p, int deg, int ntv, int terms, hipStream_t s) {
  return launch_shape_terms<_Float16>(p, deg, ntv, terms, s);
}

}  // namespace mls
