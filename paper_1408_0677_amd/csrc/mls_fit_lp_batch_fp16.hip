// Served batches of 16-bit fits: float16 instantiations.
#include "mls_fit_lp.h"

namespace mls {

hipError_t launch_batch_fp16(const LPBatch& b, int deg, int nts, int grid, hipStream_t s) {
  return launch_batch_deg<2, _Float16>(b, deg, nts, grid, s);
}

}  // namespace mls
