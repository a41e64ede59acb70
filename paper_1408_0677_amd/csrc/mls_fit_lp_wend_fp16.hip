// One-pass 16-bit fits with the Wendland weight: float16 instantiations.
#include "mls_fit_lp.h"

namespace mls {

hipError_t launch_lp_wend_fp16(const LPParams& p, int deg, int nts, int terms, hipStream_t s) {
  return launch_lp_terms<_Float16, true>(p, deg, nts, terms, s);
}

}  // namespace mls
