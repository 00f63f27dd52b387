// Cartesian pair kernels, FP64.
#include "pair_kernel.h"

namespace g3 {
hipError_t launch_pair_cart64(const PairArgs& a, hipStream_t st) {
  return launch_one<double, G3PCF_BASIS_CARTESIAN, false, kDeg>(a, st);
}
}  // namespace g3
