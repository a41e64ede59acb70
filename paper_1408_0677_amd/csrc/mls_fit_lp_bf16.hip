// One-pass 16-bit fits with the Gaussian weight: bfloat16 instantiations.
#include "mls_fit_lp.h"

namespace mls {

hipError_t launch_lp_bf16(const LPParams& p, int deg, int nts, int terms, hipStream_t s) {
  return launch_lp_terms<__bf16, false>(p, deg, nts, terms, s);
}

}  // namespace mls
