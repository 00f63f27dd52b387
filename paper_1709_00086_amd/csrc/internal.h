// Internal declarations shared by the g3pcf HIP sources (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <string>

#include "../../include/g3pcf.h"

namespace g3 {

// Largest total degree of the pair kernels' sums.  The cartesian kernels always
// carry it (a smaller lmax only drops coefficients at conversion time); the
// spin kernels come in the degrees of kDegrees, and a problem takes the
// smallest that holds its lmax: a degree D has (D + 1)^2 sums a pair, so at
// lmax = 4 a quarter of the work of degree 10.
constexpr int kDeg = 10;
constexpr int kDegrees[] = {4, 6, 8, 10};
constexpr int kNumDegrees = 4;
constexpr int kSpinCoef = kDeg / 2 + 1;  // most entries of a spin conversion row
constexpr int kTermsCart = (kDeg + 1) * (kDeg + 2) * (kDeg + 3) / 6;  // 286
constexpr int kTermsSpin = (kDeg + 1) * (kDeg + 1);                   // 121 real sums
// Conversion tables: G3PCF_BASIS_CARTESIAN, G3PCF_BASIS_SPIN and
// G3PCF_BASIS_SPIN_T (the spin terms with T_n(u_z) in place of u_z^n).
constexpr int kConvTables = 3;
// Internal "basis" of the pass that collects the degenerate (j = k) triangles:
// per shell the sums w_j^2 T_n(u_z) of Chebyshev polynomials, n <= 2 kDeg; and
// of the spin pass that collects them beside its own sums.
constexpr int kBasisDeg = 3;
constexpr int kBasisSpinDeg = 4;
constexpr int kTermsDeg = 2 * kDeg + 1;                               // 21
constexpr int kMaxBins = 32;
constexpr int kWave = 64;
// Entries after the catalogue in the cell-ordered position array, every
// coordinate NaN: the FP32 pair search maps the lanes of a window past the
// end of its candidates onto them, and no shell test accepts a NaN distance.
constexpr int kSentinel = kWave;
constexpr int kOutPerBin = (kDeg + 1) * (kDeg + 1);  // real a_lm outputs per shell (121)

// Rows of A (primaries) reduced per Gram block: at most (one list part), and
// (where few rows would leave CUs idle) at least.
constexpr int kZetaBlock = 4096;
constexpr int kZetaRowsMin = 128;
// Parts of the primary list that one launch of the Gram products takes at most.
constexpr int kZetaLists = 32;
// Primary queues of the pair kernel: one per XCD (workgroups are dispatched to
// the 8 XCDs round-robin), each counter on its own 64-byte line.
constexpr int kQueues = 8;
constexpr int kQueueStride = 16;
// further words on the same line: the counter of either kernel's groups of shells
// searched together, whether any of their shells overflowed, and all three of the adjoint
constexpr int kQueueListed = 1, kQueueOverflow = 2, kQueueAdjoint = 3, kQueueKinds = 6;
// Persistent waves of the pair kernel: as many as its occupancy lets run at
// once on the 256 CUs' SIMDs, at most kPairWaves.
constexpr int kSimds = 4 * 256;
constexpr int kPairWaves = 4 * kSimds;
// Pair-blocks of fewer primaries hand out single groups of shells: whole
// primaries leave the chip idle behind the last of them (kPairWaves waves run
// at once).
constexpr long long kSplitBelow = 4 * kPairWaves;
// Pairs the list of a group of shells searched together holds (LDS decides, see
// WaveLds), and pairs expected in a group: about five standard deviations fewer.  Where
// a primary has still more, the search ends early and fewer shells are searched
// together, at the density it found; a shell that does not fit by itself is left to the
// launch of the single shells.  (16 catalogues of 8192, FP32: 4.74 ms a call at a mean
// of 70, 4.12 at 130, 4.10 at 150, 4.08 at 180, where a few lists overflow even in
// a uniform catalogue; FP64 step of 4096: 0.61 ms at 70 and at 85, 0.62 at 100, 0.66
// at 130.  Longer lists for the cartesian kernels, 368 pairs at a mean of 275, were no
// gain: 3.24 against 2.85 ms for 40,000 galaxies.)
constexpr int kListMost32 = 224, kListMost64 = 128;
constexpr double kListMean32 = 150.0, kListMean64 = 85.0;
constexpr double kListSlack = 1.06;  // over the mean, in the measured density's favour
constexpr float kListClusters = 25.0f;  // size of clusters above which nothing is listed
// Searches a primary that the groups have to save: where every shell fits a list, and
// where some do not and a second launch searches them.  (100,000 primaries of 818 pairs,
// four saved and five dense shells, l_max 4: 1517 us forward and 2600 the adjoint,
// against 1575 and 2216 shell by shell; 16384 of 274 in a fifth of the box, four saved:
// 450 against 411.  100,003 of 503 in 20 shells, eight saved and ten dense ones: 3.5 ms
// against 3.7.)
constexpr int kListSaves = 3, kListSavesDense = 5;
// Spill-list entries per wave: a shell's secondaries kept for the later
// accumulator chunks of a multi-chunk basis.
constexpr int kSpillCap = 1 << 14;
// Maximum pair-block (primaries whose a_lm rows are held at once).
constexpr int kPairBlockMax = 524288;

// Sparse monomial -> a_lm conversion table (host), one row per real output of a
// shell.  Output o = (m, part, l) with part 0 = Re, 1 = Im (m >= 1 only).
struct ConvTable {
  int nout;            // 121
  int nnz;
  short out_m[kOutPerBin], out_l[kOutPerBin], out_part[kOutPerBin];
  int rowptr[kOutPerBin + 1];
  short term[4096];
  double coef[4096];
};

// The cartesian conversion on the device: lane i of a wave forms output i of
// each round, entry by entry, so that a wave's loads are contiguous (an entry of
// every row at a time; with a row per lane each load touched 64 lines).  Rows in
// the order of their length, the longest 64 in the first round.  Terms count in
// the order in which the kernel's chunks hold their sums (one table for each
// precision).
constexpr int kCartLen = 24;  // room for a row (the longest has 21 entries)
struct CartTable {
  int meta[2][64];            // l | m << 4 | part << 8 | entries << 9 of the output
  int most[2];                // entries of the round's longest row
  double coef[2][kCartLen][64];
  short term[2][kCartLen][64];
};
// order: [kTermsCart] place of each canonical term among the chunks' sums.
// False if a row is too long.
bool build_cart_table(const short* order, CartTable* t);  // host
const short* cart_order32();
const short* cart_order64();

// The spin-Chebyshev conversion a_lm = sum_n c_{lm,n} S_{m,n} of one degree D,
// over the term order of its sums (the D + 1 real ones of m = 0, then pairs of
// real and imaginary parts, n running to D - m); output o has l - m in n's
// place.
struct SpinTable {
  // c[k][o]: coefficient of output o = (m, l - m = j) for n = j mod 2 + 2 k <= j
  double c[kSpinCoef][128];
  // ct[k][o]: coefficient of term o = (m, n) in the output l = m + n + 2 k <= D
  double ct[kSpinCoef][128];
  int meta[128];  // m | j << 4 | part << 8 | (term index of (m, 0, 0)) << 9
};
__host__ __device__ constexpr int spin_table_of(int deg) { return (deg - kDegrees[0]) / 2; }
void build_spin_table(int deg, SpinTable* t);  // host

// Host: build the conversion table for a basis (0 cartesian, 1 spin with
// powers u_z^n, 2 spin with Chebyshev polynomials T_n(u_z)).
void build_conv_table(int basis, ConvTable* t);
// Degenerate-triangle table G[m][l][l'][n]: Pbar_lm Pbar_l'm = sum_n G T_n.
constexpr int kDegTable = (kDeg + 1) * (kDeg + 1) * (kDeg + 1) * kTermsDeg;
__host__ __device__ inline int deg_index(int m, int l, int lp, int n) {
  return ((m * (kDeg + 1) + l) * (kDeg + 1) + lp) * kTermsDeg + n;
}
void build_deg_table(double* G);  // host

// Cell grid of the sorted catalogue.
struct Grid {
  double rsearch;      // search radius: R_max plus a margin for FP32 rounding
  int nc[3];
  double s[3], inv_s[3];
  double lo[3], L[3];
  int periodic;
  int tight[3];        // periodic axis where the search window can exceed the box
  int64_t ncell;
};

Grid make_grid(const g3pcf_problem& p);

// Layout of the real outputs of a primary inside an A row: block m holds the
// real parts, then (m >= 1) the imaginary parts, of a_lm(b) for l >= m; within
// a half, shell-major (one shell's l values are adjacent, so the pair kernel
// writes each shell's outputs as short contiguous runs).
struct RowLayout {
  int lmax, nb;
  int W;               // total row width
  int off[kDeg + 2];   // column offset of each m block
  int d[kDeg + 1];     // (lmax + 1 - m) * nb
  int wm[kDeg + 1];    // block width: d for m = 0, 2d for m >= 1
  // column of (l, shell b) within a half of block m
  __host__ __device__ int pos(int m, int l, int b) const { return b * (lmax + 1 - m) + (l - m); }
};

RowLayout make_layout(int lmax, int nb);

// Groups of neighbouring shells: first the nsingle ones of a shell of its own, then
// those searched together.
struct GroupTable {
  int ngroup, nsingle;
  float density;             // pairs expected per dr^3 of volume (dr: width of a shell),
  float excess;              // and besides them in the innermost shells
  int range[kMaxBins];       // first shell of the group | last << 8
};
// How a catalogue's table is formed (host part).
struct ShellPlan {
  int lists;                 // 0: no table
  int nbins;
  int cart;
  float density;             // at the catalogue's mean over the declared box
  float most;                // pairs expected in a group at most
  // blocks of cells of about R_max, and runs of cells along x of about R_max / 8: from
  // the galaxies that share one with a galaxy follows the density around galaxies
  int nc[3];                 // cells along each axis
  int side[3], count[3];     // cells of a block and blocks along each axis
  int blocks, rows;          // blocks, and rows of cells whose runs are counted
  int run;                   // cells of a run
  float n;                   // galaxies
  float in_block, in_run;    // others that share a galaxy's in a uniform catalogue
};
constexpr int kCrowdBlocks = 2048;
constexpr int kCrowdWords = 3 * kCrowdBlocks;  // counts, and two sums a row
ShellPlan shell_plan(const g3pcf_problem& p, const Grid& g);

// Arguments of the pair kernels (forward accumulation and adjoint scatter).
struct PairArgs {
  const void* pos4;          // [n + kSentinel] (x, y, z, w) in cell order, float4 or double4
  int sentinel;              // slot of the first NaN entry (n)
  const int* cell_start;     // [ncell + 1]
  const int* plist;          // [*nprim] primary slots in cell order
  const long long* nprim;    // device scalar: number of primaries
  int* spill;                // per-wave lists of a shell's secondaries
  int spill_cap;             // entries per wave (0: no spill lists: one search per shell and chunk)
  int* queue;                // kQueues counters (stride kQueueStride): next primary of each XCD's share
  unsigned long long* pairs; // accepted pairs, a count per XCD (stride kQueueStride / 2); NULL: not counted
  long long p_begin;         // first primary of this pair-block
  long long p_count;         // primaries in this pair-block (upper bound)
  // geometry (double, used for the candidate search)
  int nc[3];
  double s[3], inv_s[3], lo[3], L[3], inv_L[3];
  int periodic;
  int tight[3];
  double rmax, rmax_search;
  // FP32 shell test: shell b holds r^2 with r2_lo[b] < r^2 < r2_hi[b] (floats
  // next to the squared shell edges, so the shells partition the floats)
  float r2_lo[kMaxBins], r2_hi[kMaxBins];
  // whether shells may be searched together: which are is in the table (device);
  // without, every shell is a group of its own
  int lists;
  const GroupTable* groups;
  float list_mean;           // pairs expected in shells searched together, at most
  unsigned* overflow;        // [*nprim] per primary the shells (bits) that did not fit the
                             // list, from the launch of groups to the one after it
  int nbins;
  int lmax;
  int los;                   // 0 z, 1 observer
  double obs[3];
  // outputs
  double* A;                 // [p_count][W] a_lm rows (forward)
  RowLayout lay;
  double* deg;               // [p_count][nbins (2 lmax + 1)] degenerate-triangle sums (kBasisSpinDeg)
  const CartTable* cart;     // cartesian conversion of the kernel's precision (device)
  const SpinTable* spin;     // [kNumDegrees] spin conversions (device)
  // adjoint
  const double* H;           // [p_count][W] H rows (converted per shell in the kernel)
  const int* perm;           // [n] slot -> original index
  double* grad_w;            // [n] cell order: FP64 pair path (secondary terms added atomically)
  float* grad_w32;           // [n] cell order: FP32 pair path (secondary terms added atomically)
  const double* wsort;       // [n] weights in cell order (FP64)
};

// ---- launchers (each returns hipGetLastError after the launch) ----
// Buffers of the cell-list stage (all device, n = galaxies).
struct CellBufs {
  void* pos4;          // [n + kSentinel] out: cell-order (x, y, z, w), float4 or double4, then NaN
  void* stage4;        // [n] scratch: the same values in input order
  int* cell_start;     // [ncell + 1] out
  int* cell_count;     // [ncell + 1] scratch
  int* key_a;          // [n] scratch: cell ids (radix keys)
  int* key_b;          // [n] scratch
  int* val_a;          // [n] scratch: radix values
  int* perm;           // [n] out: cell-order slot -> input index
  int* hist;           // [2 radix_hist_ints(n)] scratch: digit counts and offsets
  double* wsort;       // [n] out: FP64 weights in cell order
  int* blocks;         // [kCrowdWords] scratch (n > kSmallN): see ShellPlan
  GroupTable* groups;  // out, where a ShellPlan asks for it
  void* scan_tmp;      // scan scratch for max(ncell + 1, n + 1, radix_hist_ints(n)) entries
  size_t scan_bytes;
};
size_t radix_hist_ints(int64_t n);
// Buffers a pass starts from zero, cleared in one launch (32-bit words).
struct Clears {
  int count = 0;
  int* at[5];
  int64_t words[5];
  void add(void* p, int64_t n) {
    at[count] = static_cast<int*>(p);
    words[count++] = n;
  }
};
hipError_t launch_clears(const Clears& z, hipStream_t st);
// The primary list of the cell stage (flags NULL: none) and its counters.
struct Primaries {
  const uint8_t* mask;       // [n] or NULL: every galaxy
  int* flags;                // [2 (n + 1)] scratch; left zero in its first half
  int* plist;                // [n] out
  long long* nprim;          // out
  int* counters;             // cleared
  int counter_words;
};
// Galaxies up to which the cell stage runs in one workgroup: 11 us at 300, 13 at
// 700, 40 at 4096, 52 at 6000 and 66 at 8192 galaxies, against 56 us for the
// general path's launches at any of these sizes.
constexpr int kSmallN = 6144;
static_assert(kCrowdWords <= kSmallN + 2, "half of the flags of a larger catalogue");
// Catalogues of a batch of at most kBatchN galaxies take the cell stage together,
// a workgroup each (16 of about 8192: 1160 us of kernels one after the other, 104 us
// in one launch), and their Gram products (see ZetaArgs::cats): the call 5.02 and
// 4.07 ms.  Cell ids of 16 bits (the grid has at most 4 n cells) and the workgroup's
// LDS, 104 KB here, set the limit.
constexpr int kBatchN = 16384;
constexpr int kBatchGroup = 16;
// Head of a catalogue of a group: kCatStride 8-byte words, the first its primaries,
// word kCatFirst its first row in the group and kCatParts the Gram blocks a call of its
// own has room for, from kCatGroups on its GroupTable; the rest its pair kernels'
// counters.
constexpr int kCatStride = 88;  // (whole lines of 64 bytes)
constexpr int kCatFirst = 2, kCatParts = 3, kCatGroups = 4;
struct BatchCat {
  Grid grid;
  ShellPlan plan;
  int64_t first, n;          // galaxies first..first + n - 1 of the call's catalogue
  int64_t cells_at;          // its cell_start in b.cell_start
  int parts;                 // see kCatParts
};
hipError_t launch_cells_batch(const g3pcf_problem& p, const BatchCat* cats, int ncat,
                              const CellBufs& b, int* flags, int* plist, long long* head,
                              int fp64, hipStream_t st);
// The cell list, the table of groups of shells, the primary list and the pass's clears.
hipError_t launch_cells(const g3pcf_problem& p, const Grid& g, const ShellPlan& sp,
                        const CellBufs& b, const Primaries& pr, Clears z, int fp64,
                        hipStream_t st);
// Primary list for the galaxies with region0 <= region[i] < region0 + nregions, by
// region and within one in cell order: region r's are plist[starts[r - region0]] to
// plist[starts[r - region0 + 1] - 1].  nregions <= n; starts shares flags' second
// half.
hipError_t launch_region_primaries(const uint8_t* mask, const int32_t* region, int region0,
                                   int nregions, const CellBufs& b, int64_t n, int* flags,
                                   int* starts, int* plist, long long* nprim, hipStream_t st);
// *out += order-independent hash of the cell-order catalogue (slot -> index,
// stored position words, weight) and the primary list, keyed by `seed` (a hash
// of the settings); *out must be cleared first.
hipError_t launch_fingerprint(const void* pos4, int fp64, const double* wsort, const int* perm,
                              const int* plist, const long long* nprim, int64_t n,
                              unsigned long long seed, unsigned long long* out, hipStream_t st);
hipError_t launch_fill_int(int* p, int64_t count, int value, hipStream_t st);
hipError_t launch_fill_double(double* p, int64_t count, double value, hipStream_t st);
// Forward pass (distinct: the spin kernels also collect the degenerate sums
// into a.deg), adjoint pass (either basis), and the degenerate-triangle pass on
// its own: per primary and shell the sums w_j^2 T_n(u_z), n <= 2 lmax, into
// A[row][shell * (2 lmax + 1) + n] (FP64).
hipError_t launch_pair_forward(const PairArgs& a, int fp64, int basis, bool distinct,
                               hipStream_t st);
hipError_t launch_pair_adjoint(const PairArgs& a, int fp64, hipStream_t st);
hipError_t launch_pair_distinct(const PairArgs& a, int fp64, hipStream_t st);
hipError_t launch_pair_cart32(const PairArgs& a, hipStream_t st);
hipError_t launch_pair_cart64(const PairArgs& a, hipStream_t st);
// The spin kernels of one degree: forward, forward with degenerate sums, adjoint,
// each compiled in its own file.
enum { kSpinForward, kSpinForwardDeg, kSpinAdjoint };
template <int DEG, int WHAT>
hipError_t launch_pair_spin(const PairArgs& a, int fp64, hipStream_t st);
hipError_t upload_cart_tables();
hipError_t upload_spin_tables();
hipError_t table_addresses(int fp64, const CartTable** cart, const SpinTable** spin);

struct ZetaArgs {
  const double* A;           // [rows][W]
  const double* wsort;       // weights in cell order
  const int* plist;
  const long long* nprim;
  const int* range;          // parts of the list that are summed (device, `lists` + 1 of them), or NULL
  const long long* cats;     // or heads of the catalogues whose rows, lists and weights follow each other
  int lists;                 // parts of the list (1 without `range` or `cats`), at most kZetaLists
  long long row_begin;       // global primary index of A row 0
  long long K;               // rows of the pair-block (upper bound)
  RowLayout lay;
  double* C64;               // [parts][sum W_m^2] per-block Gram products (FP64)
  int parts;                 // blocks the partials have room for (>= K / kZetaBlock and `lists`);
                             // with `cats` the sum of theirs
  double* zeta;              // one a list part
  int prec;
  int* queue;                // the pair kernel's primary counters, cleared for its next launch
};
// Every block of a pair-block.
hipError_t launch_zeta_pairblock(const ZetaArgs& z, hipStream_t st);
// Blocks (partial Gram products) of a pair-block of at most PB primaries.
int zeta_parts(const RowLayout& L, long long PB);
// Partials that a workspace holds for a pair-block of at most PB primaries.
int zeta_room(const RowLayout& L, long long PB);

// Adjoint helpers
struct AdjArgs {
  const double* A;           // [rows][W]
  const long long* nprim;
  long long p_begin;
  long long p_count;
  RowLayout lay;
  const double* MHt;         // adjoint matrices M_H^m, transposed
  double* H;                 // [p_count][W] H rows
  int* queue;                // primary counters of both pair kernels, cleared for their next launch
};
size_t adj_matrix_doubles(const RowLayout& L);
hipError_t launch_adj_matrix(const double* gz, const RowLayout& L, double* MHt, hipStream_t st);
// H = X M_H^T (k_h_gemm); the adjoint pair kernel forms the primary terms and the
// per-shell coefficients from H itself.
hipError_t launch_h_gemm(const AdjArgs& a, hipStream_t st);
// grad[perm[s]] (=|+=) gs[s] (+ gs32[s] when gs32 is not null); NaN instead
// when fp_saved is not null and *fp_saved != *fp_now
hipError_t launch_unpermute(const double* gs, const float* gs32, const int* perm, int64_t n,
                            int accumulate, const unsigned long long* fp_saved,
                            const unsigned long long* fp_now, double* grad, hipStream_t st);
size_t scan_tmp_bytes(int64_t count);
hipError_t launch_scan(const int* in, int* out, int64_t count, void* tmp, size_t tmp_bytes,
                       hipStream_t st);

int sum_wm2(const RowLayout& lay);

// Degenerate triangles (distinct secondaries): table upload, the weighted sum
// over a pair-block's rows X[r][b (2 lmax + 1) + n] into D (FP64, in order; it
// clears the pair kernel's primary counters), and the correction of
// zeta^m_{ll'}(b, b).
hipError_t upload_deg_table();
size_t deg_partial_doubles(long long PB, int nb, int lmax);
hipError_t launch_deg_reduce(const double* X, int rowW, int nb, int lmax, const double* wsort,
                             const int* plist, const long long* nprim, const int* range,
                             long long p_begin, long long p_count, double* partial, double* D,
                             int* queue, hipStream_t st);
hipError_t launch_deg_apply(const double* D, int lmax, int nb, double* zeta, hipStream_t st);
// Isotropic multipoles from zeta (addition theorem).
hipError_t launch_isotropic(const double* zeta, int lmax, int nb, double* iso, hipStream_t st);

}  // namespace g3
