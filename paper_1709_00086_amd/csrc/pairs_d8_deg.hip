// Spin pair kernels of degree 8: forward with degenerate sums.
#include "pairs_spin.h"

namespace g3 {
template hipError_t launch_pair_spin<8, kSpinForwardDeg>(const PairArgs&, int, hipStream_t);
}  // namespace g3
