// One-pass 16-bit fits with the Gaussian weight: float16 instantiations.
#include "mls_fit_lp.h"

namespace mls {

hipError_t launch_lp_fp16(const LPParams& p, int deg, int nts, int terms, hipStream_t s) {
  return launch_lp_terms<_Float16, false>(p, deg, nts, terms, s);
}

}  // namespace mls
