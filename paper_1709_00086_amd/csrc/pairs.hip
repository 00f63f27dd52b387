// The pair kernels' conversion tables on the device and the choice of kernel for a
// problem (the kernels themselves are compiled in the other pairs_*.hip).
#include "internal.h"

namespace g3 {

__device__ CartTable g_cart[2];  // FP32, FP64
__device__ SpinTable g_spin[kNumDegrees];

hipError_t upload_cart_tables() {
  static CartTable host[2];
  static bool built = false;
  if (!built) {
    if (!build_cart_table(cart_order32(), &host[0]) || !build_cart_table(cart_order64(), &host[1]))
      return hipErrorInvalidValue;
    built = true;
  }
  return hipMemcpyToSymbol(HIP_SYMBOL(g_cart), host, sizeof(host), 0, hipMemcpyHostToDevice);
}

hipError_t upload_spin_tables() {
  static SpinTable host[kNumDegrees];
  static bool built = false;
  if (!built) {
    for (int d : kDegrees) build_spin_table(d, &host[spin_table_of(d)]);
    built = true;
  }
  return hipMemcpyToSymbol(HIP_SYMBOL(g_spin), host, sizeof(host), 0, hipMemcpyHostToDevice);
}

hipError_t table_addresses(int fp64, const CartTable** cart, const SpinTable** spin) {
  void* p = nullptr;
  hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(g_cart));
  if (e != hipSuccess) return e;
  *cart = static_cast<const CartTable*>(p) + (fp64 ? 1 : 0);
  if ((e = hipGetSymbolAddress(&p, HIP_SYMBOL(g_spin))) != hipSuccess) return e;
  *spin = static_cast<const SpinTable*>(p);
  return hipSuccess;
}

namespace {

// The smallest degree that holds l_max.
template <int WHAT>
hipError_t launch_spin(const PairArgs& a, int fp64, hipStream_t st) {
  if (a.lmax <= 4) return launch_pair_spin<4, WHAT>(a, fp64, st);
  if (a.lmax <= 6) return launch_pair_spin<6, WHAT>(a, fp64, st);
  if (a.lmax <= 8) return launch_pair_spin<8, WHAT>(a, fp64, st);
  return launch_pair_spin<10, WHAT>(a, fp64, st);
}

}  // namespace

hipError_t launch_pair_forward(const PairArgs& a, int fp64, int basis, bool distinct,
                               hipStream_t st) {
  if (basis == G3PCF_BASIS_SPIN)
    return distinct ? launch_spin<kSpinForwardDeg>(a, fp64, st)
                    : launch_spin<kSpinForward>(a, fp64, st);
  return fp64 ? launch_pair_cart64(a, st) : launch_pair_cart32(a, st);
}

// The per-pair polynomial represents sum_lm H_lm conj(Y_lm(u)) whatever
// monomial basis the forward pass accumulated in: the adjoint always evaluates
// it in the spin-Chebyshev basis.
hipError_t launch_pair_adjoint(const PairArgs& a, int fp64, hipStream_t st) {
  return launch_spin<kSpinAdjoint>(a, fp64, st);
}

}  // namespace g3
