// Instantiations of the objective/gradient sweep split by columns: FP32 products, elastic-net marginal,
// plain and trial evaluations.
#include "sweep_cols.h"

namespace rpca {
hipError_t launch_cols_f32_elastic(const SweepArgs& sa, bool trial, bool masked, hipStream_t s) {
  using namespace rpca_cols;
  if (masked)
    return trial ? launch_cols<true, true, false, true>(sa, s) : launch_cols<true, false, false, true>(sa, s);
  return trial ? launch_cols<false, true, false, true>(sa, s) : launch_cols<false, false, false, true>(sa, s);
}
}  // namespace rpca
