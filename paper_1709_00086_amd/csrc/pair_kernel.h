// The pair stage: neighbour gather, line-of-sight rotation, radial binning and
// monomial accumulation (paper, Algorithm 1 and eq. 1), followed by the FP64
// conversion of the monomial sums to a_lm (Sec. 3.1).
//
// One wavefront owns one primary at a time and pulls primaries from a shared
// counter (dynamic scheduling over primaries, as the paper's OpenMP dynamic
// schedule; one counter per XCD over a contiguous share of the primaries, so
// that the primaries an XCD works on at once share candidates in its L2).
// For its primary the wave takes the radial shells one after the other; for
// shell b it
//   1. builds, 64 rows of cells at a time (one lane per (cy, cz) row), the
//      runs of galaxies that can lie in the annulus: per row the x-interval
//      of the outer sphere minus the x-interval of the inner sphere, i.e. at
//      most two contiguous ranges of cells (four where they wrap around a
//      periodic box).  All cell-start lookups of the 64 rows are in flight at
//      once, and the runs go into a table in LDS with their prefix sums;
//   2. streams the runs' galaxies with one candidate per lane (a lane finds
//      its run among the run starts, which the wave keeps in a register; the
//      next window's loads are in flight while one is binned), bins each
//      candidate with the shell's squared edges, and appends the accepted
//      separations to a ring of pairs in LDS -- the GPU form of the paper's
//      per-bin pair buckets;
//   3. whenever the ring holds a full wave of pairs, normalises and rotates
//      them and accumulates them, one pair per lane, into every monomial sum
//      of the shell held in registers (vectorised over pairs, not over
//      monomials, as in the paper's vectorisation section);
//   4. reduces the per-lane partials once per (primary, shell) with DPP and
//      converts the shell's monomial sums to a_lm in FP64.
// Sparse neighbouring shells are searched together: a group of shells that is
// expected to hold few pairs (GroupTable) is searched once, into a list in
// LDS, and steps 2 and 3 then read the list for each of its shells.
// No neighbour list ever leaves the compute unit.  A basis whose sums do not
// fit in registers at once is accumulated in chunks: the first chunk's
// search also writes the shell's secondary indices to the wave's spill list,
// which the later chunks replay (a repeated search if the list overflowed).
//
// The adjoint kernel runs the same search and, per accepted pair, evaluates
// the shell's adjoint polynomial and adds it to the secondary's gradient with one
// atomic (both in FP32 on the FP32 path, in FP64 on the FP64 path).
//
// What bounds it: dense shells, the issue of the accumulation's multiply-adds
// (524,288 primaries of 35135 pairs, FP32 spin: 99 ms at 121 sums a lane and three
// waves per SIMD); the adjoint, the rate of the atomic adds (151.7 -> 144 ms with
// more stripes, see run); sparse shells, the instructions and the waits of a search
// (100,000 primaries of 2640 pairs in 10 shells: 8.9 -> 3.9 ms; 131,072 of 274 pairs
// in 16 catalogues: 5.5 -> 3.0 ms).
//
// Included by the pairs_*.hip files, which instantiate the kernels (it opens an
// anonymous namespace).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <type_traits>
#include <utility>

#include "internal.h"
#include "monomials.h"

namespace g3 {
namespace {

constexpr int kWavesPerBlock = 4;
constexpr int kMaxRuns = 3 * kWave;  // runs of one chunk of 64 rows (<= 3 per row)
constexpr int kRing = 2 * kWave;     // accepted pairs waiting for a full wave
constexpr int kAdjStripes = 64;      // interleaved stripes of an XCD's share (adjoint)
// Run-start marks: one bit per virtual candidate index, for a span of
// kMarkSpan candidates of the run table at a time (64 windows).
constexpr int kMarkSpan = 64 * kWave;
constexpr int kMarkWords = kMarkSpan / 32;

// A run of the table: g0 is the cell-order slot of its first galaxy minus the
// run's first virtual candidate index (so candidate c of the run is slot
// g0 + c).  FP32 keeps the primary's position minus the run's periodic image
// shift (the reference the candidates are measured from).
template <typename Real>
struct RunEntry;
template <>
struct RunEntry<float> {
  float rx, ry, rz;
  int g0;
};
template <>
struct RunEntry<double> {
  int g0;
};

// ---------------------------------------------------------------- per-wave LDS
// FP32 adjoint: (secondary, term) pairs waiting for their atomic add.
constexpr int kOutBuf = 4 * kWave;

// SPILL: the ring keeps the secondaries' indices too (multi-chunk bases), and
// the reduced sums have their own space (a later chunk may search again while
// they wait); otherwise the sums of a shell take the ring's, which is empty by
// then.
// The list: the accepted pairs of a group of sparse shells, found by one search
// (see search).  As many as the LDS of the occupancy target has room for (FP64:
// of a workgroup's 64 KB).
template <typename Real>
constexpr int kList = sizeof(Real) == 4 ? kListMost32 : kListMost64;
constexpr int kOutBufList = 3 * kWave;  // terms that may wait beside the list

template <typename Real, bool SPILL, bool SPINT, bool SPLIT, bool ADJ, bool LISTED>
struct WaveLds {
  using V = typename V4<Real>::T;
  static constexpr int kExchange = SPLIT ? int(Exchange<Real, !ADJ>::kReals * sizeof(Real)) : 0;
  // FP32 adjoints have 10 KB a wave (four waves per SIMD): with the list the
  // exchange and the waiting terms go into the run table, which is not in use
  // while the list is read
  static constexpr bool kInRuns = LISTED && SPINT;
  static constexpr int kOut = SPINT ? (LISTED ? kOutBufList : kOutBuf) : 0;  // waves of terms
  static constexpr int kEntries = kList<Real>;
  static constexpr int kListBytes = LISTED ? kEntries * int(sizeof(V)) : 0;
  static constexpr int kBins = LISTED && sizeof(Real) == 8 ? kEntries * 4 : 0;
  static constexpr int kSums = SPILL ? (kTermsCart + 1) * int(sizeof(Real)) + 4 : 0;  // (+1 padding slot)
  static constexpr int kSpilled = SPILL && !LISTED ? kRing * 4 : 0;
  static constexpr int kMore = kListBytes + kBins + (kInRuns ? 0 : kExchange + kOut * 8) + kSums +
                               kSpilled;

  V ring[kRing];               // (d_x, d_y, d_z, w) forward; (d_x, d_y, d_z, index) adjoint
  alignas(16) RunEntry<Real> run[kMaxRuns + 1];  // (+1: the FP32 search's sentinel run)
  // bit c of the span: a run starts at virtual candidate index mbase + c
  alignas(16) unsigned marks[kMarkWords];
  // the list and (FP64) its entries' shells; what the half waves take each
  // other's pairs from (spin kernels); waiting terms (before the first, the
  // shell's polynomial coefficients); the reduced sums and the secondary
  // indices of the ring's entries (several chunks)
  alignas(16) char more[kMore > 0 ? kMore : 16];
  int pre[kMaxRuns + 1];       // first virtual candidate index of each run

  static_assert(!kInRuns || kExchange + kOut * 8 <= int(sizeof(run)), "the run table holds both");
  __device__ __forceinline__ V* list() { return reinterpret_cast<V*>(more); }
  __device__ __forceinline__ int* bins() { return reinterpret_cast<int*>(more + kListBytes); }
  __device__ __forceinline__ Real* xch() {
    if constexpr (kInRuns)
      return reinterpret_cast<Real*>(run);
    else
      return reinterpret_cast<Real*>(more + kListBytes + kBins);
  }
  __device__ __forceinline__ int2* out() {
    return reinterpret_cast<int2*>(reinterpret_cast<char*>(xch()) + kExchange);
  }
  __device__ __forceinline__ Real* sums() {
    return reinterpret_cast<Real*>(more + kListBytes + kBins + kExchange + kOut * 8);
  }
  __device__ __forceinline__ int* ring_j() {
    return reinterpret_cast<int*>(more + kListBytes + kBins + kExchange + kOut * 8 + kSums);
  }
};

__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
  __builtin_amdgcn_wave_barrier();
}

// Lane index computed in place (the compiler cannot hoist an asm statement),
// so that no lane-dependent address has to stay live, or be spilled, across
// the accumulation loops.
__device__ __forceinline__ int lane_here() {
  int v;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(v));
  return v;
}

// Mask of the lanes where c holds (the compare result itself, without
// materialising the predicate in a vector register first).
__device__ __forceinline__ unsigned long long ballot(bool c) {
  return __builtin_amdgcn_ballot_w64(c);
}

__device__ __forceinline__ int lanes_below(unsigned long long m) {
  return __builtin_amdgcn_mbcnt_hi(unsigned(m >> 32), __builtin_amdgcn_mbcnt_lo(unsigned(m), 0));
}

// Inclusive prefix sum over the 64 lanes with DPP moves only (no lane
// addresses to keep live): row_shr 1, 2, 4 and 8 give every lane the sum of
// its row up to itself (lanes shifted in from outside the row read 0), then
// row_bcast 15 adds the last lane of rows 0 and 2 to rows 1 and 3, and
// row_bcast 31 the last lane of row 1 (rows 0-1 by then) to rows 2 and 3.
__device__ __forceinline__ int wave_incl_scan(int x) {
  x += dpp_i<0x111, 0xF, 0xF>(x);
  x += dpp_i<0x112, 0xF, 0xF>(x);
  x += dpp_i<0x114, 0xF, 0xF>(x);
  x += dpp_i<0x118, 0xF, 0xF>(x);
  x += dpp_i<0x142, 0xA, 0xF>(x);
  x += dpp_i<0x143, 0xC, 0xF>(x);
  return x;
}

// index <-> last component of a ring entry
__device__ __forceinline__ float pack_index(int j, float) { return __int_as_float(j); }
__device__ __forceinline__ double pack_index(int j, double) { return double(j); }
__device__ __forceinline__ int unpack_index(float v) { return __float_as_int(v); }
__device__ __forceinline__ int unpack_index(double v) { return int(v); }

// ---------------------------------------------------------------- geometry
// Distance range along one axis from the primary to a cell: the nearest and
// farthest points of the cell.  The outer cells of an open box also hold any
// point beyond it, and on a tight periodic axis the nearest distance is taken
// over the images (the farthest is then not used).  t0 is the cell's low side
// measured from the primary in cells (its index minus the primary's, an exact
// integer, minus the primary's fraction of a cell); the result is in length
// units, FP32 throughout.  The rounding (about 1e-5 cells of R_max / 64, 1e-6 of
// R_max / 8) is far inside the search margin of 1e-5 R_max, which enters the
// squared distances as 2 r * margin.
template <bool TIGHT>
__device__ __forceinline__ void axis_range_f(float t0, bool first, bool last, int nc, float s,
                                             int tight, float& dmin, float& dmax) {
  float lo = t0, hi = t0 + 1.0f;
  if constexpr (TIGHT) {
    if (tight) {  // min over the images of wrapped cell c_u
      float best = __builtin_huge_valf();
      for (int k = -1; k <= 1; ++k) {
        const float l = t0 + float(k * nc), h = l + 1.0f;
        best = fminf(best, fmaxf(0.0f, fmaxf(l, -h)));
      }
      dmin = best * s;
      dmax = __builtin_huge_valf();
      return;
    }
  }
  lo = first ? -__builtin_huge_valf() : lo;
  hi = last ? __builtin_huge_valf() : hi;
  dmin = fmaxf(0.0f, fmaxf(lo, -hi)) * s;
  dmax = fmaxf(fabsf(lo), fabsf(hi)) * s;
}

// floor to int, clamped first so that far-away coordinates cannot overflow
__device__ __forceinline__ int cell_of(float c) {
  return int(fminf(fmaxf(floorf(c), -1e9f), 1e9f));
}

// Periodic wrap of an unwrapped cell index c in [-n, 2n) (a search window on a
// non-tight axis spans less than one box): c -> c - k n with k in {-1, 0, 1}.
__device__ __forceinline__ int wrap_cell(int c, int n, int& k) {
  k = (c < 0) ? -1 : (c >= n ? 1 : 0);
  return c - k * n;
}

// q = r / d and r - q d for 0 <= r < 2^24 and a uniform d > 0, from a float
// reciprocal corrected by one step.
__device__ __forceinline__ int div_small(int r, int d, float inv_d, int& rem) {
  int q = int(float(r) * inv_d);
  rem = r - q * d;
  if (rem < 0) {
    --q;
    rem += d;
  } else if (rem >= d) {
    ++q;
    rem -= d;
  }
  return q;
}

// The coordinate for a run k boxes away (by value: a conditional between
// members would select their addresses and put them into memory).
__device__ __forceinline__ float image(int k, float here, float below, float above) {
  const float other = k < 0 ? below : above;
  return k == 0 ? here : other;
}

// ---------------------------------------------------------------- binning
// FP64 shell of a candidate: the same operations, in the same order and
// without contraction, as the plain definition (minimum image by
// nearbyint(d / L), r = sqrt(r^2), shell = floor(r * nbins / R_max)).
// Returns -1 for a rejected candidate.
struct Bin64 {
  double L[3];
  bool minimg;
  double r2max;
  int nbins;
  double rmax;

  __device__ __forceinline__ int classify(const double4& q, const double ref[3], double d[3],
                                          double& r2) const {
    d[0] = __dsub_rn(q.x, ref[0]);
    d[1] = __dsub_rn(q.y, ref[1]);
    d[2] = __dsub_rn(q.z, ref[2]);
    if (minimg) {
      // L * k is exact for k in {-1, 0, 1}, so one rounding as in the definition
      for (int c = 0; c < 3; ++c)
        d[c] = __dsub_rn(d[c], __dmul_rn(L[c], rint(__ddiv_rn(d[c], L[c]))));
    }
    r2 = __dadd_rn(__dadd_rn(__dmul_rn(d[0], d[0]), __dmul_rn(d[1], d[1])),
                   __dmul_rn(d[2], d[2]));
    if (!(r2 > 0.0) || !(r2 < r2max)) return -1;
    const double r = sqrt(r2);
    const int b = int(floor(__ddiv_rn(__dmul_rn(r, double(nbins)), rmax)));
    return b < nbins ? b : nbins - 1;
  }
};

// Occupancy target per kernel (waves per SIMD); the register budget is
// 512 / target per lane, so every accumulator chunk must fit: four waves for the 81
// FP32 sums (or coefficients) of degree 8 and below, three for the 121 sums of degree
// 10 and for the cartesian chunks of 91 to 99, two for FP64.  kSplit: sums or
// coefficients in the halves of a wave: the sums only where they fit no other way (FP64,
// degree 10: see SpinSums), the coefficients where that is faster (FP32 of degree 10,
// which then also runs at four waves; FP64 of degrees 8 and 10: 30,003 primaries of
// 2383 pairs at l_max 8 2.5 against 3.0 ms, at l_max 6 2.1 against 2.0 unsplit).
template <typename Real, int BASIS, bool ADJOINT, int DEG>
struct Occ {
  static constexpr bool kF32 = std::is_same<Real, float>::value;
  static constexpr bool kSpinT = ADJOINT && kF32;
  static constexpr bool kSplit = (BASIS == G3PCF_BASIS_SPIN || BASIS == kBasisSpinDeg) &&
                                 DEG >= (ADJOINT ? (kF32 ? 10 : 8) : (kF32 ? kDeg + 1 : 10));
  static constexpr int value = !kF32                               ? 2
                               : (BASIS == kBasisDeg)              ? 4
                               : (BASIS == G3PCF_BASIS_CARTESIAN) ? 3
                               : DEG == kDeg && !kSplit            ? 3
                                                                   : 4;
};

template <class... C>
constexpr int n_chunks(ChunkList<C...>) {
  return int(sizeof...(C));
}

// ---------------------------------------------------------------- the kernel
// DEG: degree the sums are carried to (at least l_max).
// kRot: line of sight towards the observer (every separation is rotated);
// kMin: a periodic axis where the search window can wrap onto itself (FP32: the
// minimum image per candidate).  All are fixed per launch, so each kernel holds
// the code and the live values of one mode only.
// KIND: kKindSingle, every group of shells is one shell, whose pairs are
// accumulated as its search finds them; kKindListed, the launch's groups are
// searched into the list; kKindAfter, as the first, after a launch of the
// second: also the shells that did not fit the list.  (A kernel that does more
// than the first needs registers for it: 4 to 7% slower on a large catalogue.)
enum { kKindSingle, kKindListed, kKindAfter };
template <typename Real, int BASIS, bool ADJOINT, int DEG, bool kRot, bool kMin, int KIND>
struct PairKernel {
  static constexpr bool kListed = KIND == kKindListed;
  using V = typename V4<Real>::T;
  // (constant memory: read into scalar registers)
  using Groups = const __attribute__((address_space(4))) GroupTable*;
  static constexpr bool kF32 = std::is_same<Real, float>::value;
  // FP32 adjoint: terms wait in LDS for their atomic additions
  static constexpr bool kSpinT = Occ<Real, BASIS, ADJOINT, DEG>::kSpinT;
  static constexpr bool kSpin = BASIS == G3PCF_BASIS_SPIN || BASIS == kBasisSpinDeg;
  // real and imaginary parts in the halves of a wave
  static constexpr bool kSplit = Occ<Real, BASIS, ADJOINT, DEG>::kSplit;
  using CL = typename Chunks<Real, BASIS, DEG>::type;
  static constexpr bool kMulti = !ADJOINT && n_chunks(CL{}) > 1;
  using Lds = WaveLds<Real, kMulti, kSpinT, kSplit, ADJOINT, kListed>;
  // the waves of the occupancy target fit a CU's LDS (the waves' first items are
  // dealt out in advance, so all of them have to run at once)
  static_assert(sizeof(Lds) * 4 * Occ<Real, BASIS, ADJOINT, DEG>::value <= 160 * 1024, "LDS");

  // Per-primary state shared by the shell searches.
  struct Primary {
    double p[3];
    Real pref[3];  // primary position in the working precision
    float ref[3][2];  // FP32: the position from the images below and above (p + L, p - L)
    double invLd[3];
    int ic[3];     // the primary's cell (unwrapped)
    float fc[3];   // its place in the cell, in cells
    float sf[3], isf[3];  // cell sides and their inverses
    Real L[3], invL[3];
    Real Rm[9];    // line-of-sight rotation (kRot)
    bool minimg;   // minimum image per candidate (else the run's image shift)
    Bin64 bin64;
  };

  // Runs of the rows [rb, rb + 64) of the window for the annulus
  // r0 <= r < r1 (given as r0^2, r1^2) into the LDS table; returns the number
  // of runs and sets `total` to their summed length.  One row of cells per
  // lane: the x-interval of the outer sphere minus the inner sphere's, i.e. two
  // intervals of cells (one where they meet), and on a periodic axis the part
  // of one of them beyond the box, so at most three runs.  All geometry in FP32
  // relative to the primary's cell, no branches that differ between lanes but
  // the one around a row out of reach, and the cell starts of all runs in
  // flight together: the wave waits for memory once per 64 rows.
  static __device__ __forceinline__ int build_runs(const PairArgs& a, const int* __restrict__ cs,
                                                   const Primary& P, float r0sq, float r1sq,
                                                   const int c0[3], int nyr, float inv_nyr,
                                                   int rb, int nrows, Lds& W, int& total) {
    const int lane = lane_here();
    const int nx = a.nc[0], ny = a.nc[1], nz = a.nc[2];
    int lo1 = 0, hi1 = -1, lo2 = 0, hi2 = -1, loe = 0, hie = -1;
    int k1 = 0, k2 = 0, ke = 0, ky = 0, kz = 0, row = 0;
    const int r = rb + lane;
    if (r < nrows) {
      int ry;
      int cz = c0[2] + div_small(r, nyr, inv_nyr, ry), cy = c0[1] + ry;
      float dzmin, dzmax, dymin, dymax;
      axis_range_f<kMin>(float(cz - P.ic[2]) - P.fc[2], !a.periodic && cz == 0,
                         !a.periodic && cz == nz - 1, nz, P.sf[2], a.tight[2], dzmin, dzmax);
      axis_range_f<kMin>(float(cy - P.ic[1]) - P.fc[1], !a.periodic && cy == 0,
                         !a.periodic && cy == ny - 1, ny, P.sf[1], a.tight[1], dymin, dymax);
      const float d2min = fma_r(dymin, dymin, dzmin * dzmin);
      const float d2max = fma_r(dymax, dymax, dzmax * dzmax);
      if (d2min < r1sq) {
        if (a.periodic) {
          if (!kMin || !a.tight[2]) cz = wrap_cell(cz, nz, kz);
          if (!kMin || !a.tight[1]) cy = wrap_cell(cy, ny, ky);
        }
        row = (cz * ny + cy) * nx;
        if (kMin && a.tight[0]) {
          hi1 = nx - 1;
        } else {
          // half-chords in cells, widened by a relative 2e-6 (inside the
          // margin); no inner one where the row's far side is out of the inner
          // sphere (or unknown: the nearest image on a tight axis)
          const float h1 = __builtin_amdgcn_sqrtf(r1sq - d2min) * P.isf[0] * (1.0f + 2e-6f) + 1e-6f;
          const float q0 = fmaxf(0.0f, r0sq - d2max);
          const float h0 =
              fmaxf(0.0f, __builtin_amdgcn_sqrtf(q0) * P.isf[0] * (1.0f - 2e-6f) - 1e-6f);
          lo1 = P.ic[0] + cell_of(P.fc[0] - h1);
          hi1 = P.ic[0] + cell_of(P.fc[0] - h0);
          lo2 = P.ic[0] + cell_of(P.fc[0] + h0);
          hi2 = P.ic[0] + cell_of(P.fc[0] + h1);
          if (!a.periodic) {
            lo1 = min(max(lo1, 0), nx - 1);
            hi1 = min(max(hi1, 0), nx - 1);
            lo2 = min(max(lo2, 0), nx - 1);
            hi2 = min(max(hi2, 0), nx - 1);
          }
          const bool one = lo2 <= hi1 + 1;
          hi1 = one ? hi2 : hi1;
          lo2 = one ? 0 : lo2;
          hi2 = one ? -1 : hi2;
          if (a.periodic) {
            // a window spans less than the box, so at most one interval crosses
            // one of its ends: its part beyond becomes the extra run
            const bool below = lo1 < 0 && hi1 >= 0;
            const bool above1 = hi1 >= nx && lo1 < nx, above2 = hi2 >= nx && lo2 < nx;
            // the second interval can also cross the lower end
            const bool below2 = lo2 < 0 && hi2 >= 0;
            const bool cross_lo = below || below2, cross_hi = above1 || above2;
            loe = below ? lo1 + nx : below2 ? lo2 + nx : 0;
            hie = cross_lo ? nx - 1 : above1 ? hi1 - nx : above2 ? hi2 - nx : -1;
            ke = cross_lo ? -1 : cross_hi ? 1 : 0;
            lo1 = below ? 0 : lo1;
            lo2 = below2 ? 0 : lo2;
            hi1 = above1 ? nx - 1 : hi1;
            hi2 = above2 ? nx - 1 : hi2;
            k1 = hi1 < 0 ? -1 : lo1 >= nx ? 1 : 0;
            k2 = hi2 < 0 ? -1 : lo2 >= nx ? 1 : 0;
            k2 = hi2 < lo2 ? 0 : k2;  // empty
            lo1 -= k1 * nx;
            hi1 -= k1 * nx;
            lo2 -= k2 * nx;
            hi2 -= k2 * nx;
          }
        }
      }
    }
    // an empty interval is [0, -1]: two reads of the same cell start
    const int g1 = cs[row + lo1], g2 = cs[row + lo2];
    int len1 = cs[row + hi1 + 1] - g1, len2 = cs[row + hi2 + 1] - g2;
    int ge = 0, lene = 0;
    if (a.periodic) {
      ge = cs[row + loe];
      lene = cs[row + hie + 1] - ge;
    }
    // table slots: a lane's runs follow those of the lower lanes
    const unsigned long long m1 = ballot(len1 > 0), m2 = ballot(len2 > 0), me = ballot(lene > 0);
    const int at1 = lanes_below(m1) + lanes_below(m2) + lanes_below(me);
    const int tot = len1 + len2 + lene;
    const int incl = wave_incl_scan(tot);
    const int v1 = incl - tot, v2 = v1 + len1, ve = v2 + len2;
    const int at2 = at1 + (len1 > 0 ? 1 : 0), ate = at2 + (len2 > 0 ? 1 : 0);
    float ry = 0.0f, rz = 0.0f;
    if constexpr (kF32) {
      ry = image(ky, P.pref[1], P.ref[1][0], P.ref[1][1]);
      rz = image(kz, P.pref[2], P.ref[2][0], P.ref[2][1]);
    }
    auto put = [&](int len, int at, int v, int g, int k) {
      if (len > 0) {
        W.pre[at] = v;
        RunEntry<Real> e;
        e.g0 = g - v;  // galaxy slot of virtual candidate index c: e.g0 + c
        if constexpr (kF32) {
          e.rx = image(k, P.pref[0], P.ref[0][0], P.ref[0][1]);
          e.ry = ry;
          e.rz = rz;
        }
        W.run[at] = e;
      }
    };
    put(len1, at1, v1, g1, k1);
    put(len2, at2, v2, g2, k2);
    if (a.periodic) put(lene, ate, ve, ge, ke);
    total = uniform_int(__builtin_amdgcn_readlane(incl, kWave - 1));
    const int nrun = __popcll(m1) + __popcll(m2) + __popcll(me);
    if constexpr (kF32) {
      // the sentinel run after the last one: the lanes of a window past the
      // last candidate map onto the NaN entries after the catalogue
      if (lane == 0) {
        W.pre[nrun] = total;
        RunEntry<Real> e;
        e.g0 = a.sentinel - total;
        e.rx = e.ry = e.rz = 0.0f;
        W.run[nrun] = e;
      }
    }
    // marks of the first span [0, kMarkSpan)
    clear_marks(W);
    if (len1 > 0 && v1 < kMarkSpan) set_mark(W, v1);
    if (len2 > 0 && v2 < kMarkSpan) set_mark(W, v2);
    if (lene > 0 && ve < kMarkSpan) set_mark(W, ve);
    if (kF32 && lane == 0 && total < kMarkSpan) set_mark(W, total);
    wave_lds_fence();
    return nrun;
  }

  static __device__ __forceinline__ void clear_marks(Lds& W) {
    const int lane = threadIdx.x % kWave;
    static_assert(kMarkWords == 2 * kWave, "two mark words per lane");
    reinterpret_cast<unsigned long long*>(W.marks)[lane] = 0ull;
    // LDS operations of one wave complete in order; the empty statement keeps
    // the compiler from moving the marks' updates above the clear
    asm volatile("" ::: "memory");
  }
  static __device__ __forceinline__ void set_mark(Lds& W, int c) {
    __hip_atomic_fetch_or(&W.marks[c >> 5], 1u << (c & 31), __ATOMIC_RELAXED,
                          __HIP_MEMORY_SCOPE_WAVEFRONT);
  }
  // The 64 marks from offset c (a multiple of 64) of the span, wave-uniform.
  static __device__ __forceinline__ unsigned long long window_marks(const Lds& W, int c) {
    const unsigned long long w = reinterpret_cast<const unsigned long long*>(W.marks)[c >> 6];
    return (static_cast<unsigned long long>(uniform_int(int(w >> 32))) << 32) |
           static_cast<unsigned>(uniform_int(int(unsigned(w))));
  }
  // The marks of two adjacent windows from offset c (a multiple of 128) of
  // the span, wave-uniform, in one LDS read.
  static __device__ __forceinline__ void window_marks2(const Lds& W, int c,
                                                       unsigned long long& m0,
                                                       unsigned long long& m1) {
    const uint4 q = reinterpret_cast<const uint4*>(W.marks)[c >> 7];
    m0 = (static_cast<unsigned long long>(uniform_int(int(q.y))) << 32) |
         static_cast<unsigned>(uniform_int(int(q.x)));
    m1 = (static_cast<unsigned long long>(uniform_int(int(q.w))) << 32) |
         static_cast<unsigned>(uniform_int(int(q.z)));
  }
  // Marks of the span starting at mbase, from the run starts in LDS (and the
  // FP32 search's sentinel run).
  static __device__ __forceinline__ void span_marks(Lds& W, int nrun, int mbase) {
    const int lane = threadIdx.x % kWave;
    wave_lds_fence();
    clear_marks(W);
    const int nr = kF32 ? nrun + 1 : nrun;
    for (int r = lane; r < nr; r += kWave) {
      const int c = W.pre[r] - mbase;
      if (c >= 0 && c < kMarkSpan) set_mark(W, c);
    }
    wave_lds_fence();
  }

  // Candidate of each lane in the window [v0, v0 + 64) of the chunk's runs.
  // Lanes past the end: FP32, one of the NaN entries after the catalogue
  // (through the sentinel run, whose start at `total` is marked like the
  // others); FP64, the last candidate again.  Windows come in order:
  // kb is the run holding v0 - 1 on entry (-1 before the first window) and the
  // run holding the window's last candidate on return.  The run starts inside
  // the window are the window's 64 bits of the marks (runs are never empty, so
  // starts are distinct positions), and a lane's run is kb plus the marks at or
  // below its position.  mbase is the first index of the span the marks hold.
  // Windows come in pairs, an even one (v0 a multiple of 128) and the odd one
  // after it, in the same span: the even one reads both windows' marks and
  // leaves the odd one's in nextm.
  template <bool ODD>
  static __device__ __forceinline__ int map_window(Lds& W, int nrun, int total, int v0, int& kb,
                                                   int& mbase, Real ref[3],
                                                   unsigned long long& nextm) {
    const int lane = threadIdx.x % kWave;
    int vc = kF32 ? v0 + lane : min(v0 + lane, total - 1);
    // the window's 64 marks; one test on the common path, where v0 is below
    // both the end and the end of the marked span
    unsigned long long pm = 0;
    if (__builtin_expect(v0 < min(total, mbase + kMarkSpan), 1)) {
      if constexpr (ODD) {
        pm = nextm;
      } else {
        window_marks2(W, v0 - mbase, pm, nextm);
      }
    } else if (v0 < total) {
      // a new span starts at an even window (spans hold 64 windows), so an
      // odd window below the end is always in its even window's span
      mbase = v0 & ~(kMarkSpan - 1);
      span_marks(W, nrun, mbase);
      if constexpr (ODD) {
        pm = window_marks(W, v0 - mbase);
      } else {
        window_marks2(W, v0 - mbase, pm, nextm);
      }
    } else if constexpr (kF32) {
      // a window past the end: every lane on the sentinel run's entries
      kb = nrun;
      vc = total + lane;
    }
    // the lane's own mark as the count's starting value (the mask itself
    // selects it, one instruction)
    int f;
    asm("v_cndmask_b32_e64 %0, 0, 1, %1" : "=v"(f) : "s"(pm));
    const int k = kb + __builtin_amdgcn_mbcnt_hi(unsigned(pm >> 32),
                                                 __builtin_amdgcn_mbcnt_lo(unsigned(pm), f));
    kb += __popcll(pm);
    const RunEntry<Real> e = W.run[k];
    if constexpr (kF32) {
      ref[0] = e.rx;
      ref[1] = e.ry;
      ref[2] = e.rz;
    }
    return e.g0 + vc;
  }

  // Galaxy j of the cell-ordered catalogue through a 32-bit byte offset from
  // the scalar base address (the catalogue is below 4 GiB: n < 2^27).
  static __device__ __forceinline__ V load_galaxy(const V* __restrict__ pos4, int j) {
    return *reinterpret_cast<const V*>(reinterpret_cast<const char*>(pos4) +
                                       (unsigned(j) * unsigned(sizeof(V))));
  }

  // Unit separation (rotated into the line-of-sight frame) of a ring entry.
  static __device__ __forceinline__ void unit(const Primary& P, const V& e, Real& ux, Real& uy,
                                              Real& uz) {
    Real inv;
    if constexpr (kF32) {
      inv = __builtin_amdgcn_rsqf(fma_r(e.z, e.z, fma_r(e.y, e.y, e.x * e.x)));
    } else {
      inv = 1.0 / sqrt(e.x * e.x + e.y * e.y + e.z * e.z);
    }
    const Real dx = e.x * inv, dy = e.y * inv, dz = e.z * inv;
    if constexpr (kRot) {
      const Real* R = P.Rm;
      ux = R[0] * dx + R[1] * dy + R[2] * dz;
      uy = R[3] * dx + R[4] * dy + R[5] * dz;
      uz = R[6] * dx + R[7] * dy + R[8] * dz;
    } else {
      ux = dx;
      uy = dy;
      uz = dz;
    }
  }

  // One search of the shells b..b_last over the annulus [r0, r1).
  // kListed: the accepted pairs are written to the list; a search that finds more
  // than it holds ends early, and `whole` is then about how many pairs there are.
  // Else b = b_last, and every one is
  // appended to the LDS ring as (separation, weight or index), and every full
  // wave of pairs is handed to consume(entry, index, valid) (one pair per
  // lane; the index only with SPILL); the
  // remainder at the end.  The position loads of the next window are issued
  // before the current window is binned.
  template <bool MINIMG, bool SPILL, typename Consume>
  static __device__ __forceinline__ unsigned search(const PairArgs& a, Lds& W,
                                                    const V* __restrict__ pos4, const Primary& P,
                                                    int b, int b_last, double r0, double r1,
                                                    float& whole, Consume&& consume) {
    const int lane = threadIdx.x % kWave;
    const int* __restrict__ cs = a.cell_start;
    int c0[3] = {0, 0, 0}, c1[3] = {0, 0, 0};
    const float r1f = float(r1);
    for (int ax = 1; ax < 3; ++ax) {
      if (kMin && a.tight[ax]) {
        c0[ax] = 0;
        c1[ax] = a.nc[ax] - 1;
      } else {
        // in cells from the primary's own (see axis_range_f for the rounding)
        const float h = r1f * P.isf[ax];
        c0[ax] = P.ic[ax] + cell_of(P.fc[ax] - h);
        c1[ax] = P.ic[ax] + cell_of(P.fc[ax] + h);
        if (!a.periodic) {
          c0[ax] = min(max(c0[ax], 0), a.nc[ax] - 1);
          c1[ax] = min(max(c1[ax], 0), a.nc[ax] - 1);
        }
      }
    }
    // uniform per shell: kept in scalar registers across the window loops
    for (int ax = 1; ax < 3; ++ax) c0[ax] = uniform_int(c0[ax]);
    const int nyr = uniform_int(c1[1] - c0[1] + 1), nzr = uniform_int(c1[2] - c0[2] + 1);
    const int nrows = nyr * nzr;
    const float inv_nyr = uniform_real(1.0f / float(nyr));
    const float r0sq = uniform_real(float(r0 * r0)), r1sq = uniform_real(float(r1 * r1));
    float lo2 = 0.0f, hi2 = 0.0f;
    if constexpr (kF32) {
      lo2 = a.r2_lo[b];
      hi2 = a.r2_hi[b_last];
    }
    int cnt = 0;
    unsigned accepted = 0;
    // Wave priority: the search (run tables, window mapping, binning) is a
    // chain of dependent LDS reads, position loads and compares, the
    // accumulation independent arithmetic; a search at priority 1 over
    // accumulations at 0 issues first when both are ready on a SIMD, and
    // its next loads start sooner (the adjoint also raises the mapping and
    // load issue to 2 over its binning).
    __builtin_amdgcn_s_setprio(1);
    for (int rb = 0; rb < nrows; rb += kWave) {
      int total = 0;
      const int nrun = build_runs(a, cs, P, r0sq, r1sq, c0, nyr, inv_nyr, rb, nrows, W, total);
      if (total == 0) continue;
      int kb = -1, mbase = 0;
      // bin one window and append its accepted pairs to the ring; consume a
      // full wave of pairs when there is one
      auto step = [&](const V& q, const Real* rref, int j, int v0) {
        Real d[3];
        bool acc;
        unsigned long long m;
        int bin = 0;
        if constexpr (kF32) {
          const float* ref = MINIMG ? P.pref : rref;
          float dx = __fsub_rn(q.x, ref[0]), dy = __fsub_rn(q.y, ref[1]),
                dz = __fsub_rn(q.z, ref[2]);
          if constexpr (MINIMG) {
            dx = fma_r(-P.L[0], __builtin_rintf(__fmul_rn(dx, P.invL[0])), dx);
            dy = fma_r(-P.L[1], __builtin_rintf(__fmul_rn(dy, P.invL[1])), dy);
            dz = fma_r(-P.L[2], __builtin_rintf(__fmul_rn(dz, P.invL[2])), dz);
          }
          const float r2 = fma_r(dz, dz, fma_r(dy, dy, __fmul_rn(dx, dx)));
          d[0] = dx;
          d[1] = dy;
          d[2] = dz;
          // no short circuit: no branches; lanes past the end hold NaN and
          // fail both tests.  The mask from the two compares' own lane masks
          // (a ballot of their conjunction would first materialise it)
          acc = (r2 > lo2) & (r2 < hi2);
          m = ballot(r2 > lo2) & ballot(r2 < hi2);
        } else {
          double r2;
          bin = P.bin64.classify(q, P.p, d, r2);
          acc = (v0 + lane < total) && bin >= b && bin <= b_last;
          m = ballot(acc);
        }
        if (acc) {
          V ent;
          ent.x = d[0];
          ent.y = d[1];
          ent.z = d[2];
          if constexpr (ADJOINT) {
            ent.w = pack_index(j, Real(0));
          } else {
            ent.w = q.w;
          }
          const int slot = cnt + lanes_below(m);  // ring: below kRing, as cnt < kWave here
          if constexpr (kListed) {
            if (slot < Lds::kEntries) {
              W.list()[slot] = ent;
              if constexpr (!kF32) W.bins()[slot] = bin;
            }
          } else {
            W.ring[slot] = ent;
            if constexpr (SPILL) W.ring_j()[slot] = j;
          }
        }
        const int got = __popcll(m);
        cnt += got;
        accepted += unsigned(got);
        if (!kListed && cnt >= kWave) {
          // the first wave of pairs out, the rest (fewer than kWave) moved to
          // the front, so that slots need no wrap-around
          wave_lds_fence();
          const V ent = W.ring[lane];
          const V rest = W.ring[kWave + lane];
          int jj = 0;
          if constexpr (SPILL) {
            jj = W.ring_j()[lane];
            W.ring_j()[lane] = W.ring_j()[kWave + lane];
          }
          W.ring[lane] = rest;
          __builtin_amdgcn_s_setprio(0);
          consume(ent, jj, true);
          __builtin_amdgcn_s_setprio(1);
          cnt -= kWave;
        }
      };
      // two windows in flight: while one is binned the other's loads are
      // outstanding (the buffers alternate, so no copy waits on a load).
      // Windows past the end accept nothing (FP32: every lane on a NaN
      // entry; FP64: on the last candidate, rejected by the index test).
      Real refa[3] = {P.pref[0], P.pref[1], P.pref[2]};
      Real refb[3] = {P.pref[0], P.pref[1], P.pref[2]};
      unsigned long long nextm = 0;
      int ja = map_window<false>(W, nrun, total, 0, kb, mbase, refa, nextm);
      V qa = load_galaxy(pos4, ja);
      for (int v0 = 0; v0 < total; v0 += 2 * kWave) {
        if constexpr (ADJOINT) __builtin_amdgcn_s_setprio(2);
        const int jb = map_window<true>(W, nrun, total, v0 + kWave, kb, mbase, refb, nextm);
        const V qb = load_galaxy(pos4, jb);
        if constexpr (ADJOINT) __builtin_amdgcn_s_setprio(1);
        step(qa, refa, ja, v0);
        if constexpr (ADJOINT) __builtin_amdgcn_s_setprio(2);
        ja = map_window<false>(W, nrun, total, v0 + 2 * kWave, kb, mbase, refa, nextm);
        qa = load_galaxy(pos4, ja);
        if constexpr (ADJOINT) __builtin_amdgcn_s_setprio(1);
        step(qb, refb, jb, v0 + kWave);
        if constexpr (kListed) {
          if (accepted > unsigned(Lds::kEntries)) {
            // the rows go through the sphere from its lowest z up: at a fraction q of
            // them, 3 q^2 - 2 q^3 of its volume
            const float rows = float(rb) + float(min(nrows - rb, kWave)) *
                                               (float(min(v0 + 2 * kWave, total)) / float(total));
            const float q = fminf(rows / float(nrows), 1.0f);
            whole = float(accepted) / (q * q * (3.0f - 2.0f * q));
            rb = nrows;
            break;
          }
        }
      }
      wave_lds_fence();
    }
    __builtin_amdgcn_s_setprio(0);
    if (!kListed && cnt > 0) {
      wave_lds_fence();
      V ent;
      int jj = 0;
      if (lane < cnt) {
        ent = W.ring[lane];
        if constexpr (SPILL) jj = W.ring_j()[lane];
      } else {
        ent.x = Real(0);
        ent.y = Real(0);
        ent.z = Real(1);
        ent.w = ADJOINT ? pack_index(0, Real(0)) : Real(0);
      }
      consume(ent, jj, lane < cnt);
      wave_lds_fence();
    }
    return accepted;
  }

  // The pairs of shell b among the list's n entries, a wave at a time to
  // consume, as search does (the same test on the same separations).
  template <typename Consume>
  static __device__ __forceinline__ void list_shell(const PairArgs& a, Lds& W, int b, int n,
                                                    Consume&& consume) {
    const int lane = threadIdx.x % kWave;
    float lo2 = 0.0f, hi2 = 0.0f;
    if constexpr (kF32) {
      lo2 = a.r2_lo[b];
      hi2 = a.r2_hi[b];
    }
    int cnt = 0;
    wave_lds_fence();
    for (int at = 0; at < n; at += kWave) {
      const int i = at + lane;
      const V e = W.list()[min(i, n - 1)];
      bool acc = i < n;
      if constexpr (kF32) {
        const float r2 = fma_r(e.z, e.z, fma_r(e.y, e.y, __fmul_rn(e.x, e.x)));
        acc = acc & (r2 > lo2) & (r2 < hi2);
      } else {
        acc = acc & (W.bins()[min(i, n - 1)] == b);
      }
      const unsigned long long m = ballot(acc);
      if (acc) W.ring[cnt + lanes_below(m)] = e;
      cnt += __popcll(m);
      if (cnt >= kWave) {
        wave_lds_fence();
        const V ent = W.ring[lane];
        W.ring[lane] = W.ring[kWave + lane];
        consume(ent, 0, true);
        cnt -= kWave;
      }
    }
    if (cnt > 0) {
      wave_lds_fence();
      V ent;
      if (lane < cnt) {
        ent = W.ring[lane];
      } else {
        ent.x = Real(0);
        ent.y = Real(0);
        ent.z = Real(1);
        ent.w = ADJOINT ? pack_index(0, Real(0)) : Real(0);
      }
      consume(ent, 0, lane < cnt);
      wave_lds_fence();
    }
  }

  // Separation of secondary j from the primary exactly as the search forms
  // it (same reference point or minimum image, same rounding).
  template <bool MINIMG>
  static __device__ __forceinline__ void separation(const PairArgs& a, const Primary& P,
                                                    const V& q, Real d[3]) {
    if constexpr (kF32) {
      float ref[3] = {P.pref[0], P.pref[1], P.pref[2]};
      if (!MINIMG && a.periodic) {
        // the run's image shift: the unique k with |q - p + k L| < L / 2
        const double qq[3] = {double(q.x), double(q.y), double(q.z)};
        // |q - p + k L| stays far from L / 2 on a non-tight axis, so the
        // product with 1/L rounds to the same k as the quotient would
        for (int c = 0; c < 3; ++c) {
          const double k = -rint((qq[c] - P.p[c]) * P.invLd[c]);
          ref[c] = float(P.p[c] - k * a.L[c]);
        }
      }
      float dx = __fsub_rn(q.x, ref[0]), dy = __fsub_rn(q.y, ref[1]), dz = __fsub_rn(q.z, ref[2]);
      if constexpr (MINIMG) {
        dx = fma_r(-P.L[0], __builtin_rintf(__fmul_rn(dx, P.invL[0])), dx);
        dy = fma_r(-P.L[1], __builtin_rintf(__fmul_rn(dy, P.invL[1])), dy);
        dz = fma_r(-P.L[2], __builtin_rintf(__fmul_rn(dz, P.invL[2])), dz);
      }
      d[0] = dx;
      d[1] = dy;
      d[2] = dz;
    } else {
      double r2;
      P.bin64.classify(q, P.p, d, r2);
    }
  }

  // Stream `count` spilled secondaries of a shell, one per lane, into
  // body(unit vector, weight; 0 past the end).  Two batches alternate so that
  // the next batch's gathers and the batch after that's indices are in flight
  // while one batch is used.
  template <bool MINIMG, typename Body>
  static __device__ __forceinline__ void replay(const PairArgs& a, const V* __restrict__ pos4,
                                                const Primary& P, const int* __restrict__ sp,
                                                int count, Body&& body) {
    if (count <= 0) return;
    const int lane = threadIdx.x % kWave;
    const int last = count - 1;
    auto use = [&](const V& q, int base) {
      const bool valid = base + lane < count;
      Real d[3];
      separation<MINIMG>(a, P, q, d);
      V e;
      e.x = valid ? d[0] : Real(0);
      e.y = valid ? d[1] : Real(0);
      e.z = valid ? d[2] : Real(1);
      Real ux, uy, uz;
      unit(P, e, ux, uy, uz);
      body(ux, uy, uz, valid ? q.w : Real(0));
    };
    int ja = sp[min(lane, last)];
    int jb = sp[min(kWave + lane, last)];
    V qa = load_galaxy(pos4, ja);
    for (int base = 0; base < count; base += 2 * kWave) {
      const V qb = load_galaxy(pos4, jb);
      ja = sp[min(base + 2 * kWave + lane, last)];
      use(qa, base);
      qa = load_galaxy(pos4, ja);
      jb = sp[min(base + 3 * kWave + lane, last)];
      use(qb, base + kWave);
    }
  }

  // The pairs of shell b to consume: by a search of its own, or (kListed) from
  // the list, which holds the group's `found` pairs.
  template <bool MINIMG, typename Consume>
  static __device__ __forceinline__ unsigned pairs_of(const PairArgs& a, Lds& W,
                                                      const V* __restrict__ pos4,
                                                      const Primary& P, int b, double r0,
                                                      double r1, int found, Consume&& consume) {
    if constexpr (kListed) {
      list_shell(a, W, b, found, consume);
      return 0;
    } else {
      float whole;
      return search<MINIMG, false>(a, W, pos4, P, b, b, r0, r1, whole, consume);
    }
  }

  // All chunks (forward) or the adjoint of shell b; returns the pairs its search
  // accepted (kListed: found pairs are counted by the caller).  With several
  // chunks and no list, the first search also writes the shell's secondaries to
  // the wave's spill list, and the later chunks replay it instead of searching
  // again (unless it overflowed).
  static __device__ __forceinline__ unsigned shell(const PairArgs& a, Lds& W,
                                                   const V* __restrict__ pos4, const Primary& P,
                                                   int b, double r0, double r1, int found,
                                                   long long row, double w_prim,
                                                   int* __restrict__ sp) {
    constexpr bool MINIMG = kF32 && kMin;
    const int lane = threadIdx.x % kWave;
    unsigned got = 0;
    if constexpr (!ADJOINT) {
      const int cap = a.spill_cap;
      bool first = true;
      bool replayable = false;
      int base = 0;
      for_each_chunk(CL{}, [&](auto* tag) {
        using Chunk = std::remove_pointer_t<decltype(tag)>;
        Chunk ch;
        ch.zero();
        auto add_unit = [&](Real ux, Real uy, Real uz, Real w) {
          if constexpr (kSplit)
            ch.add(ux, uy, uz, w, W.xch(), lane);
          else
            ch.add(ux, uy, uz, w);
        };
        auto add = [&](const V& e) {
          Real ux, uy, uz;
          unit(P, e, ux, uy, uz);
          add_unit(ux, uy, uz, e.w);
        };
        if (kMulti && !kListed && first && cap > 0) {
          int nsp = 0;
          float whole;
          got = search<MINIMG, kMulti && !kListed>(
              a, W, pos4, P, b, b, r0, r1, whole, [&](const V& e, int j, bool valid) {
                if (valid && nsp + lane < cap) sp[nsp + lane] = j;
                nsp += __popcll(ballot(valid));
                add(e);
              });
          replayable = got <= unsigned(cap);
        } else if (kMulti && !kListed && !first && replayable) {
          replay<MINIMG>(a, pos4, P, sp, int(got), add_unit);
        } else {
          const unsigned g = pairs_of<MINIMG>(a, W, pos4, P, b, r0, r1, found,
                                              [&](const V& e, int, bool) { add(e); });
          if (first) got = g;
        }
        first = false;
        if constexpr (kSplit) {
          reduce_split(W, ch);
        } else {
          // a chunk's sums after the last's
          const int wl = lane_here();
          const int row = wl >> 4, grp = ((wl >> 3) & 1) | ((wl >> 1) & 2);
          const bool leader = (wl & 3) == 0;
          fold_plain<Chunk::NT>(sums(W) + base, ch.acc, row, grp, leader, wl);
          if constexpr (BASIS == kBasisSpinDeg)
            fold_plain<Chunk::ND>(sums(W) + kSpinTerms, ch.deg, row, grp, leader, wl);
          base += Chunk::NT;
        }
      });
      wave_lds_fence();
      if constexpr (BASIS == kBasisDeg) {
        store_deg(a, sums(W), b, a.A + row * a.lay.W);
      } else if constexpr (kSpin) {
        convert_spin(a, sums(W), b, row);
        if constexpr (BASIS == kBasisSpinDeg) {
          store_deg(a, sums(W) + kSpinTerms, b, a.deg + row * (a.nbins * (2 * a.lmax + 1)));
        }
      } else {
        convert(a, sums(W), b, row);
      }
      wave_lds_fence();
    } else {
      // the shell's polynomial: its coefficients, formed from the H row and
      // staged through LDS, in vector registers
      Real* coef = coef_stage(W);
      shell_coefficients(a, W, coef, row, b);
      wave_lds_fence();
      std::conditional_t<kSplit, SplitPoly<Real, DEG>, SpinPoly<Real, DEG>> poly;
      poly.load(coef, lane);
      wave_lds_fence();
      if constexpr (kSpinT) {
        // FP32 polynomial and FP32 atomics.
        const float wp = float(w_prim);
        // Each wave of terms goes to the LDS buffer and the buffer to the
        // atomics every few waves: a wait for the candidate loads then finds
        // atomics outstanding (and has to wait for them, vmcnt counting both)
        // once per flush instead of after every wave of pairs.  A full buffer
        // is flushed before the next wave's polynomial, which then runs while
        // the atomics complete.
        int nout = 0;
        got = pairs_of<MINIMG>(a, W, pos4, P, b, r0, r1, found,
                               [&](const V& e, int, bool valid) {
                                 if (nout == Lds::kOut) {
                                   flush_terms(a, W, nout);
                                   nout = 0;
                                 }
                                 Real ux, uy, uz;
                                 unit(P, e, ux, uy, uz);
                                 float v;
                                 if constexpr (kSplit)
                                   v = poly.eval(ux, uy, uz, W.xch(), lane_here());
                                 else
                                   v = poly.eval(ux, uy, uz);
                                 W.out()[nout + lane_here()] = make_int2(
                                     valid ? unpack_index(e.w) : -1, __float_as_int(wp * v));
                                 nout += kWave;
                               });
        if (nout > 0) flush_terms(a, W, nout);
      } else {
        got = pairs_of<MINIMG>(a, W, pos4, P, b, r0, r1, found,
                               [&](const V& e, int, bool valid) {
                                 Real ux, uy, uz;
                                 unit(P, e, ux, uy, uz);
                                 double v;
                                 if constexpr (kSplit)
                                   v = poly.eval(ux, uy, uz, W.xch(), lane_here());
                                 else
                                   v = poly.eval(ux, uy, uz);
                                 if (valid)
                                   unsafeAtomicAdd(&a.grad_w[unpack_index(e.w)], w_prim * v);
                               });
      }
      wave_lds_fence();
    }
    return got;
  }

  // Where a shell's reduced sums (forward) and its coefficients (adjoint) wait.
  static __device__ __forceinline__ Real* sums(Lds& W) {
    if constexpr (kMulti)
      return W.sums();
    else
      return reinterpret_cast<Real*>(W.ring);
  }
  static __device__ __forceinline__ Real* coef_stage(Lds& W) {
    if constexpr (kSpinT)
      return reinterpret_cast<Real*>(W.out());
    else  // FP64: behind the staged H values in the ring
      return reinterpret_cast<Real*>(W.ring) + kSpinTerms;
  }
  static constexpr int kSpinTerms = (DEG + 1) * (DEG + 1);
  static_assert(kMulti || sizeof(Lds::ring) >= (2 * kTermsSpin + 1) * sizeof(Real),
                "the ring holds a shell's sums, or its H values and coefficients");

  static __device__ __forceinline__ void run(const PairArgs& a) {
    extern __shared__ char smem_raw[];
    Lds* lds = reinterpret_cast<Lds*>(smem_raw);
    // wave index made uniform so that per-wave pointers live in scalar registers
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = threadIdx.x % kWave;
    Lds& W = lds[wid];
    const V* __restrict__ pos4 = static_cast<const V*>(a.pos4);
    const long long NP = min(a.p_count, (long long)(*a.nprim) - a.p_begin);
    const int nb = a.nbins;
    const double margin = a.rmax_search - a.rmax;
    // this wave's spill list (multi-chunk bases)
    int* sp = a.spill + size_t(blockIdx.x * kWavesPerBlock + wid) * size_t(a.spill_cap);
    unsigned long long my_pairs = 0;

    // The pair-block's primaries (in cell order) are split into kQueues
    // contiguous shares, one per XCD: a wave takes primaries from its own XCD's
    // share first, so the candidates of the primaries an XCD works on at once
    // are neighbours in its L2, then helps the other shares.  Where there are
    // few primaries a wave takes one group of shells of one primary at a time,
    // the outer (larger) shells first.  A wave's first item is its own number in its
    // share (the launch holds no more waves than run at once), the further ones
    // come from the share's counter; a wave whose share is used up looks at all
    // counters in one load before it adds to another's (4096 waves that each
    // tried all eight counters in turn took 60 us to end).
    // groups of this launch: the searched together, or the single shells; then,
    // where a shell of some primary did not fit the list, also all groups again (for
    // those shells)
    int mine = nb, nsingle = nb;
    bool terms = true;  // adjoint: this launch adds the primaries' own terms
    const Groups table = (Groups)(a.groups);
    if constexpr (KIND != kKindSingle) {
      const int ngroup = table->ngroup;
      mine = nsingle = table->nsingle;
      if constexpr (kListed) {
        mine = ngroup - nsingle;
      } else {
        bool any = false;
        if (lane < kQueues) any = a.queue[lane * kQueueStride + kQueueOverflow] != 0;
        if (ballot(any) != 0) mine = ngroup;
        terms = nsingle == ngroup;  // (else the launch of groups did)
      }
    }
    if (mine == 0) return;
    const int g_first = kListed ? nsingle : 0;
    const int per = NP < kSplitBelow ? mine : 1;  // items of a primary
    const int grid = int(gridDim.x);
    const long long share = (NP + kQueues - 1) / kQueues;
    auto share_waves = [&](int x) { return (grid - x + kQueues - 1) / kQueues * kWavesPerBlock; };
    auto share_items = [&](int x) {
      return int(max(min(NP, (x + 1) * share) - x * share, 0ll)) * per;
    };
    int x = int(blockIdx.x % kQueues);
    int t = int(blockIdx.x / kQueues) * kWavesPerBlock + wid;
    int items = share_items(x), seen = 0;
    while (true) {
      if (t >= items) {
        // the first share from the next one on that still has items to hand out
        if (++seen > 2 * kQueues) break;
        int y = x + 1 + lane;
        y = y >= kQueues ? y - kQueues : y;
        bool open = false;
        if (lane < kQueues)
          open = share_waves(y) + __hip_atomic_load(a.queue + y * kQueueStride, __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT) <
                 share_items(y);
        const unsigned long long m = ballot(open);
        if (m == 0) break;
        x = (x + 1 + __builtin_ctzll(m)) % kQueues;
        items = share_items(x);
        int got = 0;
        if (lane == 0) got = atomicAdd(a.queue + x * kQueueStride, 1);
        t = share_waves(x) + uniform_int(__shfl(got, 0));
        continue;
      }
      seen = 0;
      const long long lo = x * share;
      int item = 0;
      long long tt = t;
      if (per > 1) {
        const int np = items / per;
        item = t / np;
        tt = t - item * np;
      }
      if constexpr (ADJOINT) {
        // the adjoint hands out its share in kAdjStripes interleaved
        // stripes: the waves of an XCD then work on primaries in
        // kAdjStripes places at once, and their atomic adds into the
        // secondaries' gradient meet on the same cache lines far less
        // often than when all of them work on neighbouring primaries
        // (2^18 galaxies, 13494 pairs a primary: 42.3 ms with 4 stripes, 37.4
        // with 16, 35.4 with 64 and no less with more; 25.6 without the atomic
        // adds, whose rate in the L2 is the bound: 27.7 with as many to
        // consecutive addresses, and no change with a gradient per XCD)
        const long long q = (items / per) / kAdjStripes;
        if (tt < kAdjStripes * q) tt = (tt % kAdjStripes) * q + tt / kAdjStripes;
      }
      const long long qi = lo + tt;
      // groups of shells of this item, from the outermost in: all, or one
      const int g_hi = g_first + (per > 1 ? per - 1 - item : mine - 1);
      const int g_lo = per > 1 ? g_hi : g_first;
      const int slot = uniform_int(a.plist[a.p_begin + qi]);
      const V pv = pos4[slot];
      Primary P;
      P.p[0] = uniform_double(double(pv.x));
      P.p[1] = uniform_double(double(pv.y));
      P.p[2] = uniform_double(double(pv.z));
      const long long row = qi;  // row of A within this pair-block
      if (!(isfinite(P.p[0]) && isfinite(P.p[1]) && isfinite(P.p[2]))) {
        // no separation from a non-finite position is accepted: no neighbours,
        // a zero row of sums (forward), no secondary terms (adjoint)
        if constexpr (!ADJOINT) {
          if (item == 0) {
            double* out = a.A + row * a.lay.W;
            for (int k = lane; k < a.lay.W; k += kWave) out[k] = 0.0;
            if constexpr (BASIS == kBasisSpinDeg) {
              const int nd = nb * (2 * a.lmax + 1);
              for (int k = lane; k < nd; k += kWave) a.deg[row * nd + k] = 0.0;
            }
          }
        }
        int next = items;
        if (items > share_waves(x) && lane == 0)
          next = share_waves(x) + atomicAdd(a.queue + x * kQueueStride, 1);
        t = uniform_int(__shfl(next, 0));
        continue;
      }
      if constexpr (kRot) {
        frame(a, P);
        // uniform per primary: held in scalar registers
        for (int i = 0; i < 9; ++i) P.Rm[i] = uniform_real(P.Rm[i]);
      }
      for (int c = 0; c < 3; ++c) {
        P.L[c] = uniform_real(Real(a.L[c]));
        P.invL[c] = uniform_real(Real(a.inv_L[c]));
        P.pref[c] = uniform_real(Real(P.p[c]));
        P.ref[c][0] = uniform_real(float(P.p[c] + a.L[c]));
        P.ref[c][1] = uniform_real(float(P.p[c] - a.L[c]));
        P.invLd[c] = a.inv_L[c];
        const double rel = fmin(fmax((P.p[c] - a.lo[c]) * a.inv_s[c], -1e9), 1e9);
        const double cell = floor(rel);
        P.ic[c] = uniform_int(int(cell));
        P.fc[c] = uniform_real(float(rel - cell));
        P.sf[c] = uniform_real(float(a.s[c]));
        P.isf[c] = uniform_real(float(a.inv_s[c]));
        P.bin64.L[c] = a.L[c];
      }
      // FP64 always measures from the primary with the minimum image (the
      // plain definition); FP32 only where a search window can wrap onto
      // itself (kMin)
      P.minimg = kF32 ? kMin : (a.periodic != 0);
      P.bin64.minimg = P.minimg;
      P.bin64.r2max = a.rmax * a.rmax;
      P.bin64.nbins = nb;
      P.bin64.rmax = a.rmax;

      double w_prim = 0.0;
      if constexpr (ADJOINT) {
        w_prim = a.wsort[slot];
        if (item == 0 && terms) primary_term(a, row, slot);
      }

      // annulus of a shell, widened by the search margin on both sides
      auto inner = [&](int b) { return uniform_double(fmax(0.0, b * a.rmax / nb - margin)); };
      auto outer = [&](int b) {
        return uniform_double((b + 1 == nb) ? a.rmax_search : (b + 1) * a.rmax / nb + margin);
      };
      int next = items;
      const int first = share_waves(x);
      unsigned over = 0;  // shells left to the launch of the single shells
      // pairs of this primary per dr^3 of volume: the catalogue's mean, until a search
      // finds more
      float dens = kListed ? table->density : 0.0f;
      if constexpr (KIND == kKindAfter) {
        if (mine > nsingle) over = unsigned(uniform_int(int(a.overflow[a.p_begin + qi])));
      }
      for (int g = g_hi; g >= g_lo; --g) {
        // every shell is a group of its own where none are searched together
        const int range = KIND == kKindSingle ? g | g << 8 : uniform_int(table->range[g]);
        const int b0 = range & 255, b1 = range >> 8;
        if constexpr (KIND == kKindAfter) {
          // the mask is left clear for the next kernel: which shells overflow depends on
          // the windows in which a search that ends early took its candidates
          const unsigned mask = over & ((2u << b1) - (1u << b0));
          if (g >= nsingle && mask && lane == 0) atomicAnd(a.overflow + a.p_begin + qi, ~mask);
        }
        // the wave's next item is asked for before its last group
        if (g == g_lo && items > first && lane == 0)
          next = first + atomicAdd(a.queue + x * kQueueStride, 1);
        // KIND == kKindListed: the group's outermost shells that the list is expected
        // to hold, or one, then the next ones
        for (int top = b1; top >= b0;) {
          int low = b0, found = 0;
          if constexpr (kListed) {
            auto volume = [&](int c) {  // of the shells c..top, in dr^3
              const float u = float(top + 1), v = float(c);
              return u * u * u - v * v * v;
            };
            auto expected = [&](int c) {
              return dens * volume(c) + (c == 0 ? table->excess : 0.0f);
            };
            low = top;
            while (low > b0 && expected(low - 1) <= a.list_mean) --low;
            low = uniform_int(low);
            found = Lds::kEntries + 1;
            if (expected(low) <= float(Lds::kEntries)) {
              float whole = 0.0f;
              found = int(search<kF32 && kMin, false>(a, W, pos4, P, low, top, inner(low),
                                                      outer(top), whole,
                                                      [](const V&, int, bool) {}));
              if (found > Lds::kEntries) {
                dens = fmaxf(dens, uniform_real(
                                       (whole - (low == 0 ? table->excess : 0.0f)) / volume(low)));
                if (low < top) continue;
              }
            }
            if (found > Lds::kEntries) {
              // left to the launch of the single shells
              over |= 1u << top;
              --top;
              continue;
            }
            my_pairs += unsigned(found);
          }
          for (int bb = top; bb >= low; --bb) {
            const int b = uniform_int(bb);  // in a scalar register throughout the shell
            if constexpr (KIND == kKindAfter) {
              if (g >= nsingle && ((over >> b) & 1u) == 0) continue;
            }
            my_pairs += shell(a, W, pos4, P, b, inner(b), outer(b), found, row, w_prim, sp);
          }
          top = low - 1;
        }
      }
      if constexpr (kListed) {
        if (over && lane == 0) {
          // (in a launch of single groups, another wave may hold the primary too)
          atomicOr(a.overflow + a.p_begin + qi, over);
          a.queue[x * kQueueStride + kQueueOverflow - kQueueListed] = 1;
        }
      }
      t = uniform_int(__shfl(next, 0));
    }

    // counted only where the caller asked for it, on its XCD's line (4096 waves
    // adding to one address take 140 us to end)
    if (a.pairs && lane == 0 && my_pairs)
      atomicAdd(a.pairs + blockIdx.x % kQueues * (kQueueStride / 2), my_pairs);
  }

  // Line-of-sight frame of the primary: the Rodrigues rotation taking the
  // direction from the observer to +z (the identity for a primary on the
  // observer, which has no line of sight).
  static __device__ __forceinline__ void frame(const PairArgs& a, Primary& P) {
    for (int i = 0; i < 9; ++i) P.Rm[i] = Real((i % 4 == 0) ? 1 : 0);
    const double* p = P.p;
    double n[3] = {p[0] - a.obs[0], p[1] - a.obs[1], p[2] - a.obs[2]};
    const double nn = sqrt(n[0] * n[0] + n[1] * n[1] + n[2] * n[2]);
    if (!(nn > 0.0)) return;
    for (int c = 0; c < 3; ++c) n[c] /= nn;
    const double c = n[2];
    if (c < -1.0 + 1e-12) {
      P.Rm[4] = Real(-1);
      P.Rm[8] = Real(-1);
      return;
    }
    const double vx = n[1], vy = -n[0];  // v = n x z
    const double f = 1.0 / (1.0 + c);
    const double vv = vx * vx + vy * vy;
    // R = I + [v]x + (v v^T - |v|^2 I) / (1 + c), v_z = 0
    P.Rm[0] = Real(1.0 + (vx * vx - vv) * f);
    P.Rm[1] = Real(vx * vy * f);
    P.Rm[2] = Real(vy);
    P.Rm[3] = Real(vx * vy * f);
    P.Rm[4] = Real(1.0 + (vy * vy - vv) * f);
    P.Rm[5] = Real(-vx);
    P.Rm[6] = Real(-vy);
    P.Rm[7] = Real(vx);
    P.Rm[8] = Real(1.0 - vv * f);
  }

  // Wave sums of the spin sums into sums(W), in term order (the degenerate
  // sums, if any, after them).  A register of m >= 1 holds two sums already
  // (Re in the lower half of the wave, Im in the upper): registers q and q + 1
  // fold into rows Re q, Re q + 1, Im q, Im q + 1; those of m = 0 fold by four.
  // Four such results share the last steps, and one lane of each quad stores.
  static __device__ __forceinline__ void reduce_split(Lds& W,
                                                      SpinSplit<DEG, BASIS == kBasisSpinDeg>& ch) {
    using Chunk = SpinSplit<DEG, BASIS == kBasisSpinDeg>;
    constexpr int NP = Chunk::NP;
    const auto& s = ch.acc;
    Real* M = sums(W);
    const int lane = lane_here();
    const int row = lane >> 4;
    // quads 0..3 of a row hold the results 0, 2, 1, 3 of a group
    const int grp = ((lane >> 3) & 1) | ((lane >> 1) & 2);
    const bool leader = (lane & 3) == 0;
    // all loops have constant bounds and unroll, so the registers stay registers
#pragma unroll
    for (int g = 0; g < NP; g += 8) {
      Real c[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int q = g + 2 * k;
        c[k] = q < NP ? fold2(s[q < NP ? q : 0], q + 1 < NP ? s[q + 1 < NP ? q + 1 : 0] : Real(0))
                      : Real(0);
      }
      const Real tot = row_sums4(c[0], c[1], c[2], c[3], lane);
      // rows 0..3: Re q, Re q + 1, Im q, Im q + 1
      const int q = g + 2 * grp + (row & 1);
      if (leader && q < NP) M[DEG + 1 + 2 * q + (row >> 1)] = tot;
    }
    fold_plain<DEG + 1>(M, ch.acc0, row, grp, leader, lane);
    if constexpr (BASIS == kBasisSpinDeg)
      fold_plain<Chunk::ND>(M + kSpinTerms, ch.deg, row, grp, leader, lane);
  }
  template <int N>
  static __device__ __forceinline__ void fold_plain(Real* M, const Real (&v)[N], int row, int grp,
                                                    bool leader, int lane) {
#pragma unroll
    for (int g = 0; g < N; g += 16) {
      Real c[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int i = g + 4 * k;
        c[k] = i < N ? fold4(v[i < N ? i : 0], i + 1 < N ? v[i + 1 < N ? i + 1 : 0] : Real(0),
                             i + 2 < N ? v[i + 2 < N ? i + 2 : 0] : Real(0),
                             i + 3 < N ? v[i + 3 < N ? i + 3 : 0] : Real(0))
                     : Real(0);
      }
      const Real tot = row_sums4(c[0], c[1], c[2], c[3], lane);
      const int t = g + 4 * grp + row;
      if (leader && t < N) M[t] = tot;
    }
  }

  // Convert the shell's cartesian sums to a_lm (FP64) and write them, four
  // entries of the 64 rows of a round at a time.
  static __device__ __forceinline__ void convert(const PairArgs& a, const Real* M, int b,
                                                 long long row) {
    const int lane = threadIdx.x % kWave;
    const CartTable& t = *a.cart;
    const RowLayout& L = a.lay;
    double* out = a.A + row * L.W;
    for (int r = 0; r < 2; ++r) {
      const int meta = t.meta[r][lane], most = t.most[r];
      const int l = meta & 15, m = (meta >> 4) & 15, part = (meta >> 8) & 1, n = meta >> 9;
      double s = 0.0;
      for (int k0 = 0; k0 < most; k0 += 4) {
        double c[4];
        int k[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          c[i] = t.coef[r][k0 + i][lane];
          k[i] = t.term[r][k0 + i][lane];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (k0 + i < n) s = __builtin_fma(c[i], double(M[k[i]]), s);
      }
      if (l <= L.lmax) out[L.off[m] + part * L.d[m] + L.pos(m, l, b)] = s;
    }
  }

  // The same from the spin sums: a_lm = sum_k c[k] S_{m, n}, n = (l - m) mod 2
  // + 2 k <= l - m, outputs in term order (n standing for l - m), so that an
  // output's loads do not depend on one another.
  static __device__ __forceinline__ void convert_spin(const PairArgs& a, const Real* M, int b,
                                                      long long row) {
    const int lane = threadIdx.x % kWave;
    const SpinTable& t = a.spin[spin_table_of(DEG)];
    const RowLayout& L = a.lay;
    double* out = a.A + row * L.W;
    for (int o = lane; o < kSpinTerms; o += kWave) {
      const int meta = t.meta[o];
      double c[kSpinCoef];
#pragma unroll
      for (int k = 0; k <= DEG / 2; ++k) c[k] = t.c[k][o];
      const int m = meta & 15, j = (meta >> 4) & 15, part = (meta >> 8) & 1, base = meta >> 9;
      const int stride = m ? 2 : 1;
      const Real* S = M + base + part + (j & 1) * stride;
      double s = 0.0;
#pragma unroll
      for (int k = 0; k <= DEG / 2; ++k)
        if (2 * k <= j) s = __builtin_fma(c[k], double(S[2 * k * stride]), s);
      if (m + j <= L.lmax) out[L.off[m] + part * L.d[m] + L.pos(m, m + j, b)] = s;
    }
  }

  // The shell's degenerate-triangle sums D_n, n <= 2 lmax, into a row (FP64,
  // [shell][n]).
  static __device__ __forceinline__ void store_deg(const PairArgs& a, const Real* M, int b,
                                                   double* out) {
    const int lane = threadIdx.x % kWave;
    const int nd = 2 * a.lmax + 1;
    if (lane < nd) out[b * nd + lane] = double(M[lane]);
  }

  // Adjoint, per primary: its term as a primary, Re(a^T H) / 2 in FP64
  // over its A and H rows (the imaginary half of each m >= 1 block with a
  // minus sign), added to its FP64 gradient entry (one wave per primary).
  static __device__ __forceinline__ void primary_term(const PairArgs& a, long long row, int slot) {
    const int lane = threadIdx.x % kWave;
    const double* x = a.A + row * a.lay.W;
    const double* h = a.H + row * a.lay.W;
    double s = 0.0;
    for (int m = 0; m <= a.lay.lmax; ++m) {
      const int off = a.lay.off[m], wm = a.lay.wm[m], dm = a.lay.d[m];
      for (int j = lane; j < wm; j += kWave) {
        const double v = x[off + j] * h[off + j];
        s += (m > 0 && j >= dm) ? -v : v;
      }
    }
    s = wave_sum(s);
    // the FP64 path adds secondary terms to the same array
    if (lane == kWave - 1) unsafeAtomicAdd(&a.grad_w[slot], 0.5 * s);
  }

  // Adjoint, per primary and shell b: the coefficients of the polynomial in
  // (x - i y)^m T_n(z), g_{m,n} = sum over l = m + n + 2 k <= l_max of
  // c_{lm,n} Re H_lm(b) (real parts) or -c_{lm,n} Im H_lm(b) (imaginary parts),
  // formed in FP64 and stored to LDS in the working precision.  The shell's H
  // values are first staged in term order (n standing for l - m), the
  // imaginary parts negated and l > l_max as zero, in the ring's LDS, which is
  // empty between shells (FP32: as much room as the ring's float4s leave,
  // 256 doubles).
  static __device__ __forceinline__ void shell_coefficients(const PairArgs& a, Lds& W, Real* coef,
                                                            long long row, int b) {
    const int lane = threadIdx.x % kWave;
    const double* h = a.H + row * a.lay.W;
    const SpinTable& t = a.spin[spin_table_of(DEG)];
    double* hs = reinterpret_cast<double*>(W.ring);
    static_assert(sizeof(W.ring) >= kTermsSpin * sizeof(double), "staging fits the ring");
    for (int o = lane; o < kSpinTerms; o += kWave) {
      const int meta = t.meta[o];
      const int m = meta & 15, j = (meta >> 4) & 15, part = (meta >> 8) & 1;
      double v = 0.0;
      if (m + j <= a.lay.lmax) {
        v = h[a.lay.off[m] + a.lay.pos(m, m + j, b) + part * a.lay.d[m]];
        if (part) v = -v;
      }
      hs[o] = v;
    }
    wave_lds_fence();
    for (int o = lane; o < kSpinTerms; o += kWave) {
      const int meta = t.meta[o];
      double c[kSpinCoef];
#pragma unroll
      for (int k = 0; k <= DEG / 2; ++k) c[k] = t.ct[k][o];
      const int m = meta & 15, n = (meta >> 4) & 15, part = (meta >> 8) & 1, base = meta >> 9;
      const int stride = m ? 2 : 1;
      const double* S = hs + base + part + n * stride;
      double s = 0.0;
#pragma unroll
      for (int k = 0; k <= DEG / 2; ++k)
        if (m + n + 2 * k <= DEG) s = __builtin_fma(c[k], S[2 * k * stride], s);
      coef[o] = Real(s);
    }
  }

  // The buffered secondary terms of the FP32 adjoint into the FP32
  // gradient (n: a multiple of the wave size; index -1 marks an empty lane).
  static __device__ __forceinline__ void flush_terms(const PairArgs& a, Lds& W, int n) {
    wave_lds_fence();
    for (int k = 0; k < n; k += kWave) {
      const int2 o = W.out()[k + lane_here()];
      if (o.x >= 0) unsafeAtomicAdd(&a.grad_w32[o.x], __int_as_float(o.y));
    }
    wave_lds_fence();
  }
};

template <typename Real, int BASIS, bool ADJOINT, int DEG, bool ROT, bool MIN, int KIND>
__global__ __launch_bounds__(kWave* kWavesPerBlock)
    __attribute__((amdgpu_waves_per_eu(Occ<Real, BASIS, ADJOINT, DEG>::value))) void k_pairs(
        PairArgs a) {
  PairKernel<Real, BASIS, ADJOINT, DEG, ROT, MIN, KIND>::run(a);
}

template <typename Real, int BASIS, bool ADJOINT, int DEG, bool ROT, bool MIN, int KIND>
hipError_t launch_groups(const PairArgs& a, hipStream_t st) {
  // a wave per primary, or per primary and group where they may be handed out so;
  // no more than run at once (the waves' first items are dealt out in advance)
  const long long items = a.p_count < kSplitBelow ? a.p_count * a.nbins : a.p_count;
  const long long want = (items + kWavesPerBlock - 1) / kWavesPerBlock;
  constexpr int kWaves = Occ<Real, BASIS, ADJOINT, DEG>::value * kSimds;
  static_assert(kWaves <= kPairWaves, "spill lists of every wave");
  const unsigned blocks = unsigned(std::min<long long>(want, kWaves / kWavesPerBlock));
  const size_t lds =
      sizeof(typename PairKernel<Real, BASIS, ADJOINT, DEG, ROT, MIN, KIND>::Lds) *
      kWavesPerBlock;
  static_assert(sizeof(typename PairKernel<Real, BASIS, ADJOINT, DEG, ROT, MIN, KIND>::Lds) *
                        kWavesPerBlock <= 64 * 1024, "LDS of a workgroup");
  hipLaunchKernelGGL((k_pairs<Real, BASIS, ADJOINT, DEG, ROT, MIN, KIND>),
                     dim3(blocks > 0 ? blocks : 1), dim3(kWave * kWavesPerBlock), lds, st, a);
  return hipGetLastError();
}

// The groups of sparse shells, then the single shells (a tight box has no groups:
// see shell_plan in cells.hip).
template <typename Real, int BASIS, bool ADJOINT, int DEG, bool ROT, bool MIN>
hipError_t launch_mode(const PairArgs& a, hipStream_t st) {
  if constexpr (!MIN) {
    if (a.lists) {
      PairArgs listed = a;
      listed.queue += kQueueListed;
      const hipError_t e =
          launch_groups<Real, BASIS, ADJOINT, DEG, ROT, MIN, kKindListed>(listed, st);
      if (e != hipSuccess) return e;
      return launch_groups<Real, BASIS, ADJOINT, DEG, ROT, MIN, kKindAfter>(a, st);
    }
  }
  return launch_groups<Real, BASIS, ADJOINT, DEG, ROT, MIN, kKindSingle>(a, st);
}

// The kernel of the problem's mode: rotation (observer line of sight) and tight
// periodic axes.
template <typename Real, int BASIS, bool ADJOINT, int DEG>
hipError_t launch_one(const PairArgs& a, hipStream_t st) {
  const bool rot = a.los == G3PCF_LOS_OBSERVER;
  const bool mi = a.periodic && (a.tight[0] || a.tight[1] || a.tight[2]);
  if (rot)
    return mi ? launch_mode<Real, BASIS, ADJOINT, DEG, true, true>(a, st)
              : launch_mode<Real, BASIS, ADJOINT, DEG, true, false>(a, st);
  return mi ? launch_mode<Real, BASIS, ADJOINT, DEG, false, true>(a, st)
            : launch_mode<Real, BASIS, ADJOINT, DEG, false, false>(a, st);
}

}  // namespace
}  // namespace g3
