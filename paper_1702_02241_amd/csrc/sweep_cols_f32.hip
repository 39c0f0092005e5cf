// Instantiations of the objective/gradient sweep split by columns: FP32 products,
// plain and trial evaluations.
#include "sweep_cols.h"

namespace rpca {
hipError_t launch_cols_f32(const SweepArgs& sa, bool trial, bool masked, hipStream_t s) {
  using namespace rpca_cols;
  if (masked)
    return trial ? launch_cols<true, true, false>(sa, s) : launch_cols<true, false, false>(sa, s);
  return trial ? launch_cols<false, true, false>(sa, s) : launch_cols<false, false, false>(sa, s);
}
}  // namespace rpca
