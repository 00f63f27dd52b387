// Device helpers of the pair kernels: wave-uniform broadcasts, DPP wave sums
// and the two monomial bases with their register-resident accumulators.
//
// Included by pair_kernel.h only (it opens an anonymous namespace).
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

#include "internal.h"

namespace g3 {
namespace {

// ---------------------------------------------------------------- utilities
template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

template <typename Real>
struct V4;
template <>
struct V4<float> {
  using T = float4;
};
template <>
struct V4<double> {
  using T = double4;
};

// Copies of a wave-uniform value in scalar registers.  The value passes
// through an empty asm statement first: the compiler drops readfirstlane of a
// value it already knows to be uniform, and such values then stay in (and
// spill from) vector registers.
__device__ __forceinline__ int uniform_int(int v) {
  asm("" : "+v"(v));
  return __builtin_amdgcn_readfirstlane(v);
}
__device__ __forceinline__ float uniform_real(float v) {
  return __int_as_float(uniform_int(__float_as_int(v)));
}

__device__ __forceinline__ double uniform_double(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = uniform_int(int(b & 0xffffffffll));
  const int hi = uniform_int(int(b >> 32));
  return __longlong_as_double((static_cast<long long>(hi) << 32) |
                              (static_cast<unsigned int>(lo)));
}
__device__ __forceinline__ double uniform_real(double v) { return uniform_double(v); }

// DPP move with compile-time controls (old value 0 where the row is masked).
// With bound_ctrl set and full masks the compiler folds the move into the add.
template <int CTRL, int ROW, int BANK>
__device__ __forceinline__ int dpp_i(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, ROW, BANK, true);
}

// Sum over the 64 lanes; the total is valid in lanes 48..63.
// quad_perm [1,0,3,2], quad_perm [2,3,0,1], row_ror 4, row_ror 8 give every
// lane its row sum; row_bcast 15 and row_bcast 31 then fold rows 0-2 into 3.
__device__ __forceinline__ float wave_sum(float v) {
  v += __int_as_float(dpp_i<0xB1, 0xF, 0xF>(__float_as_int(v)));
  v += __int_as_float(dpp_i<0x4E, 0xF, 0xF>(__float_as_int(v)));
  v += __int_as_float(dpp_i<0x124, 0xF, 0xF>(__float_as_int(v)));
  v += __int_as_float(dpp_i<0x128, 0xF, 0xF>(__float_as_int(v)));
  v += __int_as_float(dpp_i<0x142, 0xA, 0xF>(__float_as_int(v)));
  v += __int_as_float(dpp_i<0x143, 0xC, 0xF>(__float_as_int(v)));
  return v;
}

template <int CTRL, int ROW, int BANK>
__device__ __forceinline__ double dpp_d(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = dpp_i<CTRL, ROW, BANK>(int(b & 0xffffffffll));
  const int hi = dpp_i<CTRL, ROW, BANK>(int(b >> 32));
  return __longlong_as_double((static_cast<long long>(hi) << 32) |
                              (static_cast<unsigned int>(lo)));
}

__device__ __forceinline__ double wave_sum(double v) {
  v += dpp_d<0xB1, 0xF, 0xF>(v);
  v += dpp_d<0x4E, 0xF, 0xF>(v);
  v += dpp_d<0x124, 0xF, 0xF>(v);
  v += dpp_d<0x128, 0xF, 0xF>(v);
  v += dpp_d<0x142, 0xA, 0xF>(v);
  v += dpp_d<0x143, 0xC, 0xF>(v);
  return v;
}

// Sum over the 16 lanes of each row (every lane gets its row's sum).
__device__ __forceinline__ float row_sum(float v) {
  v += __int_as_float(dpp_i<0xB1, 0xF, 0xF>(__float_as_int(v)));
  v += __int_as_float(dpp_i<0x4E, 0xF, 0xF>(__float_as_int(v)));
  v += __int_as_float(dpp_i<0x124, 0xF, 0xF>(__float_as_int(v)));
  v += __int_as_float(dpp_i<0x128, 0xF, 0xF>(__float_as_int(v)));
  return v;
}
__device__ __forceinline__ double row_sum(double v) {
  v += dpp_d<0xB1, 0xF, 0xF>(v);
  v += dpp_d<0x4E, 0xF, 0xF>(v);
  v += dpp_d<0x124, 0xF, 0xF>(v);
  v += dpp_d<0x128, 0xF, 0xF>(v);
  return v;
}

// Fold four values a, e, b, f across rows: lane i of row 0 of the result
// holds a summed over lanes i, i + 16, i + 32 and i + 48, row 1 the same for
// e, row 2 for b, row 3 for f, so a row sum of the result gives the four
// totals (and given row sums as inputs, the result holds the totals):
// permlane32_swap exchanges the upper half of its first operand with the
// lower half of its second, permlane16_swap the odd rows of its first with the
// even rows of its second.
__device__ __forceinline__ unsigned pl32(unsigned& x, unsigned y) {
  const auto r = __builtin_amdgcn_permlane32_swap(x, y, false, false);
  x = r[0];
  return r[1];
}
__device__ __forceinline__ unsigned pl16(unsigned& x, unsigned y) {
  const auto r = __builtin_amdgcn_permlane16_swap(x, y, false, false);
  x = r[0];
  return r[1];
}
__device__ __forceinline__ float fold4(float a, float e, float b, float f) {
  unsigned ua = __float_as_uint(a), ue = __float_as_uint(e);
  const unsigned ub = pl32(ua, __float_as_uint(b));
  const unsigned uf = pl32(ue, __float_as_uint(f));
  const float c = __uint_as_float(ua) + __uint_as_float(ub);
  const float d = __uint_as_float(ue) + __uint_as_float(uf);
  unsigned uc = __float_as_uint(c);
  const unsigned ud = pl16(uc, __float_as_uint(d));
  return __uint_as_float(uc) + __uint_as_float(ud);
}
__device__ __forceinline__ double swap32_d(double& x, double y) {
  const long long bx = __double_as_longlong(x), by = __double_as_longlong(y);
  unsigned xl = unsigned(bx), xh = unsigned(bx >> 32);
  const unsigned yl = pl32(xl, unsigned(by)), yh = pl32(xh, unsigned(by >> 32));
  x = __longlong_as_double((static_cast<long long>(xh) << 32) | xl);
  return __longlong_as_double((static_cast<long long>(yh) << 32) | yl);
}
__device__ __forceinline__ double swap16_d(double& x, double y) {
  const long long bx = __double_as_longlong(x), by = __double_as_longlong(y);
  unsigned xl = unsigned(bx), xh = unsigned(bx >> 32);
  const unsigned yl = pl16(xl, unsigned(by)), yh = pl16(xh, unsigned(by >> 32));
  x = __longlong_as_double((static_cast<long long>(xh) << 32) | xl);
  return __longlong_as_double((static_cast<long long>(yh) << 32) | yl);
}
__device__ __forceinline__ double fold4(double a, double e, double b, double f) {
  const double b2 = swap32_d(a, b);
  const double f2 = swap32_d(e, f);
  double c = a + b2;
  const double d = e + f2;
  const double d2 = swap16_d(c, d);
  return c + d2;
}

// Fold two values across neighbouring rows: rows 0 and 2 of the result hold a
// summed over rows 0-1 and 2-3, rows 1 and 3 the same for b.
__device__ __forceinline__ float fold2(float a, float b) {
  unsigned ua = __float_as_uint(a);
  const unsigned ub = pl16(ua, __float_as_uint(b));
  return __uint_as_float(ua) + __uint_as_float(ub);
}
__device__ __forceinline__ double fold2(double a, double b) {
  const double b2 = swap16_d(a, b);
  return a + b2;
}
// Sums over each row of 16 lanes of four values at once: two values share a
// register after each halving of the row, so that the last steps add all four
// together (11 instructions instead of 16).
__device__ __forceinline__ float dpp_ror8(float v) {
  return __int_as_float(dpp_i<0x128, 0xF, 0xF>(__float_as_int(v)));
}
__device__ __forceinline__ double dpp_ror8(double v) { return dpp_d<0x128, 0xF, 0xF>(v); }
__device__ __forceinline__ float dpp_half_mirror(float v) {
  return __int_as_float(dpp_i<0x141, 0xF, 0xF>(__float_as_int(v)));
}
__device__ __forceinline__ double dpp_half_mirror(double v) { return dpp_d<0x141, 0xF, 0xF>(v); }
__device__ __forceinline__ float quad_sum(float v) {
  v += __int_as_float(dpp_i<0xB1, 0xF, 0xF>(__float_as_int(v)));
  v += __int_as_float(dpp_i<0x4E, 0xF, 0xF>(__float_as_int(v)));
  return v;
}
__device__ __forceinline__ double quad_sum(double v) {
  v += dpp_d<0xB1, 0xF, 0xF>(v);
  v += dpp_d<0x4E, 0xF, 0xF>(v);
  return v;
}
// The lanes of quad 0 of a row return the row's sum of a, those of quad 1 of c,
// of quad 2 of b and of quad 3 of d.
template <typename Real>
__device__ __forceinline__ Real row_sums4(Real a, Real b, Real c, Real d, int lane) {
  const bool hi = (lane & 8) != 0, odd = (lane & 4) != 0;
  const Real ab = (hi ? b : a) + dpp_ror8(hi ? a : b);
  const Real cd = (hi ? d : c) + dpp_ror8(hi ? c : d);
  return quad_sum((odd ? cd : ab) + dpp_half_mirror(odd ? ab : cd));
}

__device__ __forceinline__ float fma_r(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_r(double a, double b, double c) { return __builtin_fma(a, b, c); }

// ---------------------------------------------------------------- monomial bases
// Canonical cartesian index (q outermost, then p, then k); must match tables.cpp.
__host__ __device__ constexpr int cart_index_c(int k, int p, int q) {
  int t = 0;
  for (int qq = 0; qq < q; ++qq) t += (kDeg - qq + 1) * (kDeg - qq + 2) / 2;
  for (int pp = 0; pp < p; ++pp) t += kDeg - q - pp + 1;
  return t + k;
}
__host__ __device__ constexpr int cart_count(unsigned qmask) {
  int c = 0;
  for (int q = 0; q <= kDeg; ++q)
    if ((qmask >> q) & 1u) c += (kDeg - q + 1) * (kDeg - q + 2) / 2;
  return c;
}
// local index of (k, p, q) inside a chunk holding the q's of qmask
__host__ __device__ constexpr int cart_local(unsigned qmask, int k, int p, int q) {
  int t = 0;
  for (int qq = 0; qq < q; ++qq)
    if ((qmask >> qq) & 1u) t += (kDeg - qq + 1) * (kDeg - qq + 2) / 2;
  for (int pp = 0; pp < p; ++pp) t += kDeg - q - pp + 1;
  return t + k;
}

// Global term index of the i-th accumulator of a cartesian chunk.
__host__ __device__ constexpr int cart_term_of(unsigned qmask, int i) {
  int t = 0;
  for (int q = 0; q <= kDeg; ++q) {
    if (!((qmask >> q) & 1u)) continue;
    for (int p = 0; p + q <= kDeg; ++p)
      for (int k = 0; k + p + q <= kDeg; ++k) {
        if (t == i) return cart_index_c(k, p, q);
        ++t;
      }
  }
  return -1;
}

// Cartesian chunk: the monomials u_x^k u_y^p u_z^q whose z power q is in QMASK.
// Per pair: P = w u_y^p u_z^q by running products, then acc += u_x^k * P
// (one FMA per monomial).
template <typename Real, unsigned QMASK>
struct CartChunk {
  static constexpr int NT = cart_count(QMASK);
  Real acc[NT];
  static __host__ __device__ constexpr int term_of(int i) { return cart_term_of(QMASK, i); }

  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int i = 0; i < NT; ++i) acc[i] = Real(0);
  }

  __device__ __forceinline__ void add(Real x, Real y, Real z, Real w) {
    Real xp[kDeg + 1];
    xp[0] = Real(1);
#pragma unroll
    for (int k = 1; k <= kDeg; ++k) xp[k] = xp[k - 1] * x;
    Real wz = w;
    static_for<kDeg + 1>([&](auto qc) {
      constexpr int q = decltype(qc)::value;
      if constexpr (q > 0) wz = wz * z;
      if constexpr (((QMASK >> q) & 1u) != 0) {
        Real P = wz;
        static_for<kDeg + 1 - q>([&](auto pc) {
          constexpr int p = decltype(pc)::value;
          if constexpr (p > 0) P = P * y;
          static_for<kDeg + 1 - q - p>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            constexpr int t = cart_local(QMASK, k, p, q);
            if constexpr (k == 0)
              acc[t] += P;
            else
              acc[t] = fma_r(xp[k], P, acc[t]);
          });
        });
      }
    });
  }
};

// Term index of Re / Im S_{m,n} among the sums of degree at most D
// ((D + 1)^2 of them): the D + 1 real ones of m = 0, then (Re, Im) pairs.
template <int D>
__host__ __device__ constexpr int spin_pair_c(int m, int n) {  // pair (m >= 1, n)
  return (m - 1) * (D + 1) - (m - 1) * m / 2 + n;
}
template <int D>
__host__ __device__ constexpr int spin_term_c(int m, int n, int part) {
  return m == 0 ? n : D + 1 + 2 * spin_pair_c<D>(m, n) + part;
}

// Exchange of half waves: on return a holds the lower halves of both inputs
// ([a.lo | b.lo]) and b the upper ones ([a.hi | b.hi]).
__device__ __forceinline__ void swap_halves(float& a, float& b) {
  unsigned ua = __float_as_uint(a);
  const unsigned ub = pl32(ua, __float_as_uint(b));
  a = __uint_as_float(ua);
  b = __uint_as_float(ub);
}
__device__ __forceinline__ void swap_halves(double& a, double& b) { b = swap32_d(a, b); }

// T_1..T_N of z, given 2 z too, by their three-term recurrence
// T_{n+1} = 2 z T_n - T_{n-1} (one FMA each).  In this basis the
// coefficients of the spherical harmonics do not cancel: those of the powers
// z^n do, by up to three orders of magnitude at l = 10 (for m = 0 they are
// the power-basis coefficients of the Legendre polynomials), which costs
// FP32 sums as many digits.
template <int N, typename Real, int D>
__device__ __forceinline__ void chebyshev_z2(Real z, Real z2, Real (&tn)[D]) {
  tn[1] = z;
  if constexpr (N >= 2) tn[2] = fma_r(z2, z, Real(-1));
  static_for<(N > 2 ? N - 2 : 0)>([&](auto nc) {
    constexpr int n = decltype(nc)::value + 2;
    tn[n + 1] = fma_r(z2, tn[n], -tn[n - 1]);
  });
}

// c = (x - i y) c, two multiply-adds and two products.  The power's real part
// alone follows 2 x c_m - (x^2 + y^2) c_{m-1} with half the operations, but the
// rounding errors of that recurrence grow with m (random directions, FP32: 2.0
// times those of the product at m = 3, 3.6 at 6, 5.7 at 10).
template <typename Real>
__device__ __forceinline__ void times_xy(Real& re, Real& im, Real x, Real y) {
  const Real r = fma_r(re, x, im * y);
  im = fma_r(im, x, -(re * y));
  re = r;
}

// Degenerate-triangle sums that ride along with the spin sums: deg[n] += w^2
// T_n(z), n <= 2 D, given T_1..T_D.
template <int D, typename Real, int N>
__device__ __forceinline__ void add_degenerate(Real (&deg)[N], const Real (&t)[D + 1], Real z,
                                               Real w) {
  const Real w2 = w * w, z2 = z + z;
  deg[0] += w2;
  static_for<D>([&](auto nc) {
    constexpr int n = decltype(nc)::value + 1;
    deg[n] = fma_r(w2, t[n], deg[n]);
  });
  Real p0 = t[D - 1], p1 = t[D];
  static_for<D>([&](auto nc) {
    constexpr int n = decltype(nc)::value + D + 1;
    const Real p2 = fma_r(z2, p1, -p0);
    deg[n] = fma_r(w2, p2, deg[n]);
    p0 = p1;
    p1 = p2;
  });
}

// Spin sums S_{m,n} = sum w (u_x - i u_y)^m T_n(u_z), m + n <= D, with T_n the
// Chebyshev polynomials (the conversion to a_lm uses the spin-Chebyshev table).
// Every lane carries all (D + 1)^2 sums of its own pairs, in term order.
// (Real and imaginary parts in either half of a wave, as in FP64 at D = 10 below, fit
// four FP32 waves a SIMD at D = 10 instead of three, but a lane then sums twice as many pairs:
// the errors of S_{m,0}, m = 1..3, over 20,000 pairs were 1.4 to 1.5 times these.  The
// fourth wave is worth 11 to 13% where the search counts, 16 catalogues of 8192
// in 3.66 against 4.18 ms, and nothing on dense catalogues.  Degrees 4, 6 and 8 have
// four waves either way and are up to 8% faster unsplit, in FP64 up to 7%, sparse
// catalogues at D = 8 4% slower.)
template <typename Real, int D, bool DISTINCT>
struct SpinSums {
  static constexpr int NT = (D + 1) * (D + 1);
  static constexpr int ND = DISTINCT ? 2 * D + 1 : 1;
  Real acc[NT];
  Real deg[ND];            // sum w^2 T_n(u_z), n <= 2 D (degenerate triangles)

  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int i = 0; i < NT; ++i) acc[i] = Real(0);
#pragma unroll
    for (int i = 0; i < ND; ++i) deg[i] = Real(0);
  }

  __device__ __forceinline__ void add(Real x, Real y, Real z, Real w) {
    Real t[D + 1];
    chebyshev_z2<D>(z, z + z, t);
    acc[0] += w;
    static_for<D>([&](auto nc) {
      constexpr int n = decltype(nc)::value + 1;
      acc[n] = fma_r(w, t[n], acc[n]);
    });
    if constexpr (DISTINCT) add_degenerate<D>(deg, t, z, w);
    Real cr = w * x, ci = -(w * y);  // w (x - i y)^m
    static_for<D>([&](auto mc) {
      constexpr int m = decltype(mc)::value + 1;
      if constexpr (m > 1) times_xy(cr, ci, x, y);
      Real* a = acc + spin_term_c<D>(m, 0, 0);
      a[0] += cr;
      a[1] += ci;
      static_for<D - m>([&](auto nc) {
        constexpr int n = decltype(nc)::value + 1;
        a[2 * n] = fma_r(cr, t[n], a[2 * n]);
        a[2 * n + 1] = fma_r(ci, t[n], a[2 * n + 1]);
      });
    });
  }
};

// Adjoint polynomial (either basis): the sum over (m, n), m + n <= D, of the
// coefficients times the Re / Im parts of (x - i y)^m T_n(z), with Chebyshev
// polynomials T_n in place of z^n.  In this basis the coefficients of the
// spherical harmonics do not cancel (those of z^n do, by two to three orders
// of magnitude at l = 10), so FP32 evaluation keeps close to FP32 accuracy.
// The coefficients are the same for every pair (one set per primary and
// shell) and are held in vector registers: a multiply-add with a scalar-register
// operand issues more slowly than one with three vector registers.
template <typename Real, int D>
struct SpinPoly {
  static constexpr int NT = (D + 1) * (D + 1);
  Real g[NT];

  template <typename Ptr>
  __device__ __forceinline__ void load(Ptr gc, int) {
#pragma unroll
    for (int i = 0; i < NT; ++i) g[i] = gc[i];
  }

  __device__ __forceinline__ Real eval(Real x, Real y, Real z) const {
    Real t[D + 1];
    chebyshev_z2<D>(z, z + z, t);
    Real total = g[0];
    static_for<D>([&](auto nc) {
      constexpr int n = decltype(nc)::value + 1;
      total = fma_r(g[n], t[n], total);
    });
    Real cr = x, ci = -y;  // (x - i y)^m
    static_for<D>([&](auto mc) {
      constexpr int m = decltype(mc)::value + 1;
      if constexpr (m > 1) times_xy(cr, ci, x, y);
      const Real* a = g + spin_term_c<D>(m, 0, 0);
      Real hr = a[0], hi = a[1];
      static_for<D - m>([&](auto nc) {
        constexpr int n = decltype(nc)::value + 1;
        hr = fma_r(a[2 * n], t[n], hr);
        hi = fma_r(a[2 * n + 1], t[n], hi);
      });
      total = fma_r(cr, hr, fma_r(ci, hi, total));
    });
    return total;
  }
};

// The half waves' operands.  For m >= 1 a register holds the real part of
// something in the lower half of the wave and the imaginary part in the upper;
// the 64 pairs are then taken 32 at a time, each by both halves, which need the
// pair's z and powers (x - i y)^m: in LDS every lane leaves what they follow
// from, and reads it for its half's part of a lower pair (lane mod 32) and of
// an upper one.  Each half carries the power's other part too: with s = y in the
// lower half and -y in the upper, both follow
//   own' = own x + other s,   other' = other x - own s.
__device__ __forceinline__ float flip(float v, int lane) {  // -v in the upper half
  return __uint_as_float(__float_as_uint(v) ^ (unsigned(lane & 32) << 26));
}
__device__ __forceinline__ double flip(double v, int lane) {
  return __longlong_as_double(__double_as_longlong(v) ^ ((long long)(lane & 32) << 58));
}
template <typename Real>
struct Half {
  Real z, x, s;
  Real own, other;  // of w (x - i y), or of x - i y
};
// kWeighted: with w.
template <typename Real, bool kWeighted>
struct Exchange {
  static constexpr int kReals = (kWeighted ? 8 : 4) * kWave;  // per wave
  typedef Real V4r __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ void put(Real* s, int lane, Real x, Real y, Real z, Real w) {
    // (the fourth of either is not read)
    reinterpret_cast<V4r*>(s)[lane] = V4r{z, x, y, Real(0)};
    if constexpr (kWeighted)
      reinterpret_cast<V4r*>(s)[kWave + lane] = V4r{w * x, -(w * y), w * x, Real(0)};
  }
  // upper: pairs 32..63 instead of 0..31
  static __device__ __forceinline__ Half<Real> get(const Real* s, int lane, bool upper) {
    const int p = (lane & 31) + (upper ? 32 : 0), half = lane >> 5;
    const V4r a = reinterpret_cast<const V4r*>(s)[p];
    const Real sy = flip(a.z, lane);
    if constexpr (kWeighted) {
      const Real* c = s + 4 * (kWave + p) + half;
      return Half<Real>{a.x, a.y, sy, c[0], c[1]};
    } else {
      return Half<Real>{a.x, a.y, sy, half ? sy : a.y, half ? a.y : -sy};
    }
  }
  static __device__ __forceinline__ void fence() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();
  }
};

// The same sums at D = 10 in FP64, of which a lane holds no 121.  For m >= 1 the lower half of the wave holds the real
// part of S_{m,n} and the upper half the imaginary part, in one register: 66
// accumulators instead of 121 at D = 10, which fit two waves per SIMD at once.
template <int D, bool DISTINCT>
struct SpinSplit {
  static constexpr int ND = DISTINCT ? 2 * D + 1 : 1;
  static constexpr int NP = D * (D + 1) / 2;  // (m >= 1, n) pairs
  double acc0[D + 1];       // m = 0, one pair per lane
  double acc[NP];           // Re | Im
  double deg[ND];           // sum w^2 T_n(u_z), n <= 2 D (degenerate triangles)

  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int i = 0; i <= D; ++i) acc0[i] = 0.0;
#pragma unroll
    for (int i = 0; i < NP; ++i) acc[i] = 0.0;
#pragma unroll
    for (int i = 0; i < ND; ++i) deg[i] = 0.0;
  }

  // 32 pairs, both halves of the wave
  __device__ __forceinline__ void add_half(const Half<double>& h) {
    double t[D + 1];
    chebyshev_z2<D - 1>(h.z, h.z + h.z, t);
    double own = h.own, other = h.other;
    static_for<D>([&](auto mc) {
      constexpr int m = decltype(mc)::value + 1;
      if constexpr (m > 1) times_xy(own, other, h.x, h.s);
      double* a = acc + spin_pair_c<D>(m, 0);
      a[0] += own;
      static_for<D - m>([&](auto nc) {
        constexpr int n = decltype(nc)::value + 1;
        a[n] = fma_r(own, t[n], a[n]);
      });
    });
  }

  __device__ __forceinline__ void add(double x, double y, double z, double w, double* xch,
                                      int lane) {
    Exchange<double, true>::put(xch, lane, x, y, z, w);
    // m = 0 (and the degenerate sums) while the exchange is under way
    double t[D + 1];
    chebyshev_z2<D>(z, z + z, t);
    acc0[0] += w;
    static_for<D>([&](auto nc) {
      constexpr int n = decltype(nc)::value + 1;
      acc0[n] = fma_r(w, t[n], acc0[n]);
    });
    if constexpr (DISTINCT) add_degenerate<D>(deg, t, z, w);
    Exchange<double, true>::fence();
    add_half(Exchange<double, true>::get(xch, lane, false));
    add_half(Exchange<double, true>::get(xch, lane, true));
  }
};

// The same polynomial with the coefficients split as the sums of SpinSplit are (66
// registers instead of 121 at D = 10, so four waves a SIMD in FP32: 100,003 primaries
// of 2640 pairs 5.8 ms, at three waves and unsplit 6.3): each half of the wave evaluates
// its part of all 64 pairs, and one exchange at the end adds the two.
template <typename Real, int D>
struct SplitPoly {
  static constexpr int NP = D * (D + 1) / 2;
  Real g0[D + 1], g[NP];

  // gc: the (D + 1)^2 coefficients in term order
  template <typename Ptr>
  __device__ __forceinline__ void load(Ptr gc, int lane) {
    const int part = lane >> 5;
#pragma unroll
    for (int i = 0; i <= D; ++i) g0[i] = gc[i];
#pragma unroll
    for (int i = 0; i < NP; ++i) g[i] = gc[D + 1 + 2 * i + part];
  }

  __device__ __forceinline__ Real eval_half(const Half<Real>& h) const {
    Real t[D + 1];
    chebyshev_z2<D - 1>(h.z, h.z + h.z, t);
    Real own = h.own, other = h.other, sum = Real(0);
    static_for<D>([&](auto mc) {
      constexpr int m = decltype(mc)::value + 1;
      if constexpr (m > 1) times_xy(own, other, h.x, h.s);
      const Real* a = g + spin_pair_c<D>(m, 0);
      Real v = a[0];
      static_for<D - m>([&](auto nc) {
        constexpr int n = decltype(nc)::value + 1;
        v = fma_r(a[n], t[n], v);
      });
      sum = m == 1 ? own * v : fma_r(own, v, sum);
    });
    return sum;
  }

  // the polynomial of the lane's own pair
  __device__ __forceinline__ Real eval(Real x, Real y, Real z, Real* xch, int lane) {
    Exchange<Real, false>::put(xch, lane, x, y, z, Real(1));
    Real t[D + 1];
    chebyshev_z2<D>(z, z + z, t);
    Real total = g0[0];
    static_for<D>([&](auto nc) {
      constexpr int n = decltype(nc)::value + 1;
      total = fma_r(g0[n], t[n], total);
    });
    Exchange<Real, false>::fence();
    Real sa = eval_half(Exchange<Real, false>::get(xch, lane, false));
    Real sb = eval_half(Exchange<Real, false>::get(xch, lane, true));
    swap_halves(sa, sb);
    return total + (sa + sb);
  }
};

template <class... C>
struct ChunkList {};

// Chunking keeps each chunk's accumulators within the 256 architected VGPRs.
template <typename Real, int BASIS, int DEG>
struct Chunks;
template <>
struct Chunks<float, G3PCF_BASIS_CARTESIAN, kDeg> {
  // z powers {0, 5, 9, 10}, {1, 4, 7, 8}, {2, 3, 6}: 91, 99 and 96 sums, so
  // that each chunk fits three waves per SIMD (two chunks at two waves
  // measured 7% slower)
  using type = ChunkList<CartChunk<float, 0x621u>, CartChunk<float, 0x192u>,
                         CartChunk<float, 0x04Cu>>;
};
template <>
struct Chunks<double, G3PCF_BASIS_CARTESIAN, kDeg> {
  using type = ChunkList<CartChunk<double, 0x601u>, CartChunk<double, 0x182u>,
                         CartChunk<double, 0x00Cu>, CartChunk<double, 0x070u>>;
};
// Degenerate-triangle sums on their own (the cartesian basis): D_n = sum w^2
// T_n(z), n <= 2 kDeg, with the Chebyshev polynomials (bounded by 1 on [-1, 1],
// so FP32 is accurate).  conj(Y_lm) Y_l'm depends on z alone and is a polynomial
// of degree l + l', i.e. a combination of these T_n.
template <typename Real>
struct DegChunk {
  static constexpr int NT = kTermsDeg;
  Real acc[NT];
  static __host__ __device__ constexpr int term_of(int i) { return i; }

  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int i = 0; i < NT; ++i) acc[i] = Real(0);
  }

  __device__ __forceinline__ void add(Real, Real, Real z, Real w) {
    const Real w2 = w * w;
    Real p0 = Real(1), p1 = z;
    const Real z2 = z + z;
    acc[0] += w2;
    acc[1] = fma_r(w2, p1, acc[1]);
    static_for<NT - 2>([&](auto nc) {
      constexpr int n = decltype(nc)::value + 1;  // T_{n+1} from T_n and T_{n-1}
      const Real p2 = fma_r(z2, p1, -p0);
      acc[n + 1] = fma_r(w2, p2, acc[n + 1]);
      p0 = p1;
      p1 = p2;
    });
  }
};
template <typename Real>
struct Chunks<Real, kBasisDeg, kDeg> {
  using type = ChunkList<DegChunk<Real>>;
};
template <typename Real, int DEG, bool DISTINCT>
using SpinOf = std::conditional_t<sizeof(Real) == 4 || DEG != kDeg, SpinSums<Real, DEG, DISTINCT>,
                                  SpinSplit<DEG, DISTINCT>>;
template <typename Real, int DEG>
struct Chunks<Real, G3PCF_BASIS_SPIN, DEG> {
  using type = ChunkList<SpinOf<Real, DEG, false>>;
};
template <typename Real, int DEG>
struct Chunks<Real, kBasisSpinDeg, DEG> {
  using type = ChunkList<SpinOf<Real, DEG, true>>;
};

template <class... C, typename F>
__host__ __device__ __forceinline__ void for_each_chunk(ChunkList<C...>, F&& f) {
  (f(static_cast<C*>(nullptr)), ...);
}

}  // namespace
}  // namespace g3
