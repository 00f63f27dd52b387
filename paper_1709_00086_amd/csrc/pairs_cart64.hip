// Cartesian pair kernels, FP64.
#include "pair_kernel.h"

namespace g3 {
hipError_t launch_pair_cart64(const PairArgs& a, hipStream_t st) {
  return launch_one<double, G3PCF_BASIS_CARTESIAN, false, kDeg>(a, st);
}

const short* cart_order64() {
  static short order[kTermsCart];
  int at = 0;
  for_each_chunk(Chunks<double, G3PCF_BASIS_CARTESIAN, kDeg>::type{}, [&](auto* tag) {
    using Chunk = std::remove_pointer_t<decltype(tag)>;
    for (int i = 0; i < Chunk::NT; ++i) order[Chunk::term_of(i)] = short(at++);
  });
  return order;
}
}  // namespace g3
