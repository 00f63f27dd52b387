// The pair kernels' conversion tables on the device, the choice of kernel for a
// problem, and the cartesian kernels (the spin kernels are compiled by degree
// in pairs_d*.hip).
#include "pair_kernel.h"

namespace g3 {

__device__ ConvTable g_conv;
__device__ SpinTable g_spin[kNumDegrees];

hipError_t upload_conv_table() {
  static ConvTable host;
  static bool built = false;
  if (!built) {
    build_conv_table(G3PCF_BASIS_CARTESIAN, &host);
    built = true;
  }
  return hipMemcpyToSymbol(HIP_SYMBOL(g_conv), &host, sizeof(host), 0, hipMemcpyHostToDevice);
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

hipError_t table_addresses(const ConvTable** conv, const SpinTable** spin) {
  void* p = nullptr;
  hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(g_conv));
  if (e != hipSuccess) return e;
  *conv = static_cast<const ConvTable*>(p);
  if ((e = hipGetSymbolAddress(&p, HIP_SYMBOL(g_spin))) != hipSuccess) return e;
  *spin = static_cast<const SpinTable*>(p);
  return hipSuccess;
}

namespace {

// The smallest degree that holds l_max.
hipError_t launch_spin(const PairArgs& a, int fp64, int what, hipStream_t st) {
  if (a.lmax <= 4) return launch_pair_spin<4>(a, fp64, what, st);
  if (a.lmax <= 6) return launch_pair_spin<6>(a, fp64, what, st);
  if (a.lmax <= 8) return launch_pair_spin<8>(a, fp64, what, st);
  return launch_pair_spin<10>(a, fp64, what, st);
}

}  // namespace

hipError_t launch_pair_forward(const PairArgs& a, int fp64, int basis, bool distinct,
                               hipStream_t st) {
  if (basis == G3PCF_BASIS_SPIN)
    return launch_spin(a, fp64, distinct ? kSpinForwardDeg : kSpinForward, st);
  return fp64 ? launch_one<double, G3PCF_BASIS_CARTESIAN, false, kDeg>(a, st)
              : launch_one<float, G3PCF_BASIS_CARTESIAN, false, kDeg>(a, st);
}

hipError_t launch_pair_distinct(const PairArgs& a, int fp64, hipStream_t st) {
  return fp64 ? launch_one<double, kBasisDeg, false, kDeg>(a, st)
              : launch_one<float, kBasisDeg, false, kDeg>(a, st);
}

// The per-pair polynomial represents sum_lm H_lm conj(Y_lm(u)) whatever
// monomial basis the forward pass accumulated in: the adjoint always evaluates
// it in the spin-Chebyshev basis.
hipError_t launch_pair_adjoint(const PairArgs& a, int fp64, hipStream_t st) {
  return launch_spin(a, fp64, kSpinAdjoint, st);
}

}  // namespace g3
