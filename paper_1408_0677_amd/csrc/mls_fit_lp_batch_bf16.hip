// Served batches of 16-bit fits: bfloat16 instantiations.
#include "mls_fit_lp.h"

namespace mls {

hipError_t launch_batch_bf16(const LPBatch& b, int deg, int nts, int grid, hipStream_t s) {
  return launch_batch_deg<3, __bf16>(b, deg, nts, grid, s);
}

}  // namespace mls
