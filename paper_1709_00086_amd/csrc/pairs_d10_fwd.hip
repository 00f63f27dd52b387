// Spin pair kernels of degree 10: forward.
#include "pairs_spin.h"

namespace g3 {
template hipError_t launch_pair_spin<10, kSpinForward>(const PairArgs&, int, hipStream_t);
}  // namespace g3
