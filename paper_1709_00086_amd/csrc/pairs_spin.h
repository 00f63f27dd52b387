// The spin pair kernels of a degree; included after pair_kernel.h by the file
// that instantiates them.
#pragma once

namespace g3 {

template <int DEG>
hipError_t launch_pair_spin(const PairArgs& a, int fp64, int what, hipStream_t st) {
  if (fp64) {
    if (what == kSpinAdjoint) return launch_one<double, G3PCF_BASIS_SPIN, true, DEG>(a, st);
    if (what == kSpinForwardDeg) return launch_one<double, kBasisSpinDeg, false, DEG>(a, st);
    return launch_one<double, G3PCF_BASIS_SPIN, false, DEG>(a, st);
  }
  if (what == kSpinAdjoint) return launch_one<float, G3PCF_BASIS_SPIN, true, DEG>(a, st);
  if (what == kSpinForwardDeg) return launch_one<float, kBasisSpinDeg, false, DEG>(a, st);
  return launch_one<float, G3PCF_BASIS_SPIN, false, DEG>(a, st);
}

}  // namespace g3
