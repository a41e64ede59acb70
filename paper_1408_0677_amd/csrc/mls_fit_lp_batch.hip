// Served batches of one-pass 16-bit fits: instantiations.
#include "mls_fit_lp.h"

namespace mls {

hipError_t launch_lp_batch(const LPBatch& b, bool fp16, int deg, int nts, int grid,
                           hipStream_t s) {
  return fp16 ? launch_batch_deg<2, _Float16>(b, deg, nts, grid, s)
              : launch_batch_deg<3, __bf16>(b, deg, nts, grid, s);
}

}  // namespace mls
