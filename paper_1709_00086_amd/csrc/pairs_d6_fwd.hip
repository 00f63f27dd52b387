// Spin pair kernels of degree 6: forward.
#include "pairs_spin.h"

namespace g3 {
template hipError_t launch_pair_spin<6, kSpinForward>(const PairArgs&, int, hipStream_t);
}  // namespace g3
