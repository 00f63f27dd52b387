// Spin pair kernels of degree 8.
#include "pair_kernel.h"
#include "pairs_spin.h"

namespace g3 {
template hipError_t launch_pair_spin<8>(const PairArgs&, int, int, hipStream_t);
}  // namespace g3
