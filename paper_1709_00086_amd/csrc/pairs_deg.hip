// The degenerate-triangle pass on its own.
#include "pair_kernel.h"

namespace g3 {
hipError_t launch_pair_distinct(const PairArgs& a, int fp64, hipStream_t st) {
  return fp64 ? launch_one<double, kBasisDeg, false, kDeg>(a, st)
              : launch_one<float, kBasisDeg, false, kDeg>(a, st);
}
}  // namespace g3
