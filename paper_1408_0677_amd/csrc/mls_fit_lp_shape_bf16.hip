// Two-pass (shape-function) 16-bit fits: bfloat16 instantiations.
#include "mls_fit_lp.h"

namespace mls {

hipError_t launch_shape_bf16(const LPParams& p, int deg, int ntv, int terms, hipStream_t s) {
  return launch_shape_terms<__bf16>(p, deg, ntv, terms, s);
}

}  // namespace mls
