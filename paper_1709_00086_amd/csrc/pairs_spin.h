// The spin pair kernels of one degree and kind, for the files that instantiate
// them.
#pragma once

#include "pair_kernel.h"

namespace g3 {

template <int DEG, int WHAT>
hipError_t launch_pair_spin(const PairArgs& a, int fp64, hipStream_t st) {
  constexpr int kBasis = WHAT == kSpinForwardDeg ? kBasisSpinDeg : int(G3PCF_BASIS_SPIN);
  constexpr bool kAdjoint = WHAT == kSpinAdjoint;
  return fp64 ? launch_one<double, kBasis, kAdjoint, DEG>(a, st)
              : launch_one<float, kBasis, kAdjoint, DEG>(a, st);
}

}  // namespace g3
