// Spin pair kernels of degree 6: adjoint.
#include "pairs_spin.h"

namespace g3 {
template hipError_t launch_pair_spin<6, kSpinAdjoint>(const PairArgs&, int, hipStream_t);
}  // namespace g3
