// Instantiations of the objective/gradient sweep split by columns: BF16 products,
// plain and trial evaluations.
#include "sweep_cols.h"

namespace rpca {
hipError_t launch_cols_bf16(const SweepArgs& sa, bool trial, bool masked, hipStream_t s) {
  using namespace rpca_cols;
  if (masked)
    return trial ? launch_cols<true, true, true>(sa, s) : launch_cols<true, false, true>(sa, s);
  return trial ? launch_cols<false, true, true>(sa, s) : launch_cols<false, false, true>(sa, s);
}
}  // namespace rpca
