// The zeta stage: sum over primaries of w_i a_lm(b1) conj(a_l'm(b2)).
//
// The paper adds the per-primary products a_lm(r1) a*_l'm(r2) (Sec. 3.1) and
// combines per-thread partial multipoles at the end of the loop over primaries
// (single-node optimisations section).  Here the per-primary coefficients of a
// block of K primaries are the rows of A, and for every m the block's
// contribution is a Gram product on the matrix cores:
//   B_m = [Re A^m | Im A^m]  (K x W_m),   C_m = (diag(w) B_m)^T B_m,
//   Re zeta^m = C_pp + C_qq,   Im zeta^m = C_qp - C_pq.
// For m = 0 every a_l0 is real and B_0 = Re A^0.  The blocks' C_m (FP32 or
// FP64 accumulation on the matrix cores) are added into zeta in FP64, in
// block order.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "internal.h"

namespace g3 {

namespace {

typedef float float4_t __attribute__((ext_vector_type(4)));
typedef double double4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

// Rows of the pair-block [begin, begin + count) that are summed: its primaries,
// or those of the list's part range[0]..range[1] - 1; the first of them in `first`.
__device__ __forceinline__ long long valid_rows(const long long* nprim, const int* range,
                                                long long begin, long long count,
                                                long long& first) {
  const long long lo = range ? max((long long)range[0], begin) : begin;
  const long long hi = min(range ? (long long)range[1] : (long long)*nprim, begin + count);
  first = lo - begin;
  return max(hi - lo, 0ll);
}
// The Gram blocks of a launch: the valid rows of its list parts spread over the
// workspace's partials, every block within one part, `rows` of them (a multiple
// of kZetaRowsMin).  Only the device knows how many primaries there are (a mask
// may leave few of the rows the launch covers, a region's part may hold any number
// of them), so the blocks are dealt out here, one list part a lane; the workgroups
// past the last block leave at once.  The catalogues of a batch are each cut as in a
// call of their own.
struct GramBlocks {
  int first, count;  // rows of the lane's list part
  int rows;          // rows of a block of the lane's list part
  int begin, end;    // blocks of the lane's list part
};
static_assert(kZetaLists <= kWave, "a lane per list part");

__device__ __forceinline__ GramBlocks gram_blocks(const ZetaArgs& z) {
  const int lane = threadIdx.x % kWave;
  GramBlocks g{};
  // blocks that `all` rows are cut into
  int share = z.parts - z.lists + 1, all;
  if (z.cats) {
    if (lane < z.lists) {
      g.count = int(z.cats[lane * kCatStride]);
      g.first = int(z.cats[lane * kCatStride + kCatFirst]);
      share = int(z.cats[lane * kCatStride + kCatParts]);
    }
    all = g.count;
  } else {
    if (lane < z.lists) {
      long long first;
      g.count =
          int(valid_rows(z.nprim, z.range ? z.range + lane : nullptr, z.row_begin, z.K, first));
      g.first = int(first);
    }
    // sum of ceil(count / rows) <= ceil(all / rows) + lists - 1 <= parts
    all = g.count;
#pragma unroll
    for (int o = 1; o < kWave; o *= 2) all += __shfl_xor(all, o);
  }
  auto whole = [](int r) {
    return max(r + kZetaRowsMin - 1, kZetaRowsMin) / kZetaRowsMin * kZetaRowsMin;
  };
  const int most = whole((all + share - 1) / share);
  int n = (g.count + most - 1) / most;
  g.rows = whole(n ? (g.count + n - 1) / n : 0);
  n = (g.count + g.rows - 1) / g.rows;
  g.end = n;
#pragma unroll
  for (int o = 1; o < kWave; o *= 2) {
    const int v = __shfl_up(g.end, o);
    if (lane >= o) g.end += v;
  }
  g.begin = g.end - n;
  return g;
}

// ---- One workgroup per (m, 128 x 128 macro tile of C_m on or above the diagonal,
// Gram block of rows).  Each step puts kStep rows of the macro tile's two column
// panels in LDS (weights applied to the left operand, FP64 rows converted to the
// working precision on the way), and the eight waves share out its units: two
// 16 x 16 tiles below each other, so that a right operand is read from LDS once for
// two tiles.  In FP32 and BF16x3 the MFMA accumulators are added into FP64 ones
// every kFlush rows, so the block's partial is FP64 like the sum across blocks.
//
// What bounds it: the staging, that is the reads of the FP64 rows and the vector
// instructions that convert and split them (BF16x3, 2^19 rows of 1210: 7.9 GB staged
// in 2.6 ms, 3.0 TB/s; the MFMAs alone 0.55 ms).  With 64 x 64 macro tiles every
// column was staged in up to five workgroups; 128-wide panels stage it in at most
// three, and tiles below the diagonal or past the last column are left out (438 of
// 16 x 16 a block at lmax 10 and 10 shells instead of 688).  The rows of a step are
// read two steps ahead and its row numbers three, without a branch around a load:
// with a wait for the weights (row number, then weight, then lane reads) in every
// step one took 3.2 us, now 2.2.  50001 primaries BF16x3 555 -> 290 us, 40000 FP32
// 375 -> 253, 50021 FP64 577 -> 415.
constexpr int kPanel = 128;        // columns of a panel
constexpr int kTile = 16;
constexpr int kPT = kPanel / kTile;  // tiles of a panel
constexpr int kGramThreads = 512;
constexpr int kGramWaves = kGramThreads / kWave;
constexpr int kUnits = kPT / 2 * kPT / kGramWaves;  // units a wave holds at most
// Rows per FP32 accumulation before the FP64 sum: blocks hold whole ones, so
// the FP32 sums do not depend on how many blocks the rows are cut into.
constexpr int kFlush = kZetaRowsMin;

struct MDims {
  int nm;
  int W[kDeg + 1];
  int off[kDeg + 1];
  int cw[kDeg + 2];       // offsets of each C_m in a partial
  int order[kDeg + 1];    // the m's, widest first
  int mt[kDeg + 2];       // cumulative macro tiles of order[]
  int csize;
};

MDims make_mdims(const RowLayout& L) {
  MDims d{};
  d.nm = L.lmax + 1;
  int cw = 0, mt = 0;
  for (int m = 0; m < d.nm; ++m) {
    d.W[m] = L.wm[m];
    d.off[m] = L.off[m];
    d.cw[m] = cw;
    cw += L.wm[m] * L.wm[m];
    d.order[m] = m;
  }
  std::stable_sort(d.order, d.order + d.nm, [&](int a, int b) { return L.wm[a] > L.wm[b]; });
  for (int k = 0; k < d.nm; ++k) {
    d.mt[k] = mt;
    const int t = (L.wm[d.order[k]] + kPanel - 1) / kPanel;
    mt += t * (t + 1) / 2;
  }
  d.cw[d.nm] = cw;
  d.mt[d.nm] = mt;
  d.csize = cw;
  return d;
}

__device__ __forceinline__ void macro_tile_of(const MDims& d, int t, int& m, int& ti, int& tj) {
  int k = 0;
  while (k + 1 < d.nm && t >= d.mt[k + 1]) ++k;
  m = d.order[k];
  int r = t - d.mt[k];
  const int nt = (d.W[m] + kPanel - 1) / kPanel;
  ti = 0;
  while (r >= nt - ti) {
    r -= nt - ti;
    ++ti;
  }
  tj = ti + r;
}

// The operands of a precision: how a step's rows lie in LDS and how a unit's two
// tiles take them.
template <int PREC>
struct Operands;

// FP32 / FP64: [row][column]
template <typename Real, int STEP>
struct PlainOperands {
  using Acc = std::conditional_t<sizeof(Real) == 4, float4_t, double4_t>;
  static constexpr int kStep = STEP;
  static constexpr int kStride = kPanel + (sizeof(Real) == 4 ? 16 : 8);
  Real v[2][kStep][kStride];  // left (weighted), right
  // eight rows from r0 of one column
  static constexpr int kRows = STEP / 4;
  __device__ __forceinline__ void put(int side, int col, int rg, const double* x,
                                      const double* wgt) {
#pragma unroll
    for (int q = 0; q < kRows; ++q)
      v[side][rg * kRows + q][col] = Real(side == 0 ? wgt[q] * x[q] : x[q]);
  }
  __device__ __forceinline__ static Acc mma(Real a, Real b, Acc c) {
    if constexpr (sizeof(Real) == 4)
      return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    else
      return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  // row of register r of lane group g in the result (the FP64 one interleaves
  // rows: measured on gfx950)
  __device__ __forceinline__ static int row(int g, int r) {
    return sizeof(Real) == 4 ? 4 * g + r : g + 4 * r;
  }
  struct Left {
    Real a[2][kStep / 4];
  };
  __device__ __forceinline__ void left(Left& l, int i, int lane) const {
    const int li = lane % 16, g = lane / 16;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int k = 0; k < kStep / 4; ++k) l.a[t][k] = v[0][4 * k + g][i + t * kTile + li];
  }
  __device__ __forceinline__ void unit(const Left& l, int j, int lane, Acc (&acc)[2]) const {
    const int li = lane % 16, g = lane / 16;
#pragma unroll
    for (int k = 0; k < kStep / 4; ++k) {
      const Real b = v[1][4 * k + g][j + li];
      acc[0] = mma(l.a[0][k], b, acc[0]);
      acc[1] = mma(l.a[1][k], b, acc[1]);
    }
  }
};
template <>
struct Operands<G3PCF_PREC_FP32> : PlainOperands<float, 32> {};
template <>
struct Operands<G3PCF_PREC_FP64> : PlainOperands<double, 16> {};

// BF16x3: every FP32 operand x split as x0 + x1 + x2, each xk the
// round-to-nearest-even bfloat16 of what is left, and the six products with
// i + j <= 2 on the bfloat16 matrix cores.  [part][column][row], so that an MFMA
// lane reads its eight rows of a column with one load.
template <>
struct Operands<G3PCF_PREC_BF16X3> {
  using Acc = float4_t;
  static constexpr int kStep = 32;
  static constexpr int kRows = 8;
  static constexpr int kPad = 8;  // bf16 padding of a column's 32 rows (bank spread)
  bf16x8_t v[2][3][kPanel][(kStep + kPad) / 8];
  __device__ __forceinline__ void put(int side, int col, int rg, const double* x,
                                      const double* wgt) {
    bf16x8_t p[3];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      float rem = float(side == 0 ? wgt[q] * x[q] : x[q]);
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const __bf16 h = static_cast<__bf16>(rem);
        p[k][q] = h;
        rem -= float(h);
      }
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) v[side][k][col][rg] = p[k];
  }
  __device__ __forceinline__ static int row(int g, int r) { return 4 * g + r; }
  struct Left {
    bf16x8_t a[2][3];
  };
  __device__ __forceinline__ void left(Left& l, int i, int lane) const {
    const int li = lane % 16, g = lane / 16;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int k = 0; k < 3; ++k) l.a[t][k] = v[0][k][i + t * kTile + li][g];
  }
  __device__ __forceinline__ void unit(const Left& l, int j, int lane, Acc (&acc)[2]) const {
    const int li = lane % 16, g = lane / 16;
    const bf16x8_t y0 = v[1][0][j + li][g], y1 = v[1][1][j + li][g], y2 = v[1][2][j + li][g];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      float4_t c = acc[t];
      c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(l.a[t][2], y0, c, 0, 0, 0);
      c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(l.a[t][1], y1, c, 0, 0, 0);
      c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(l.a[t][0], y2, c, 0, 0, 0);
      c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(l.a[t][1], y0, c, 0, 0, 0);
      c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(l.a[t][0], y1, c, 0, 0, 0);
      acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(l.a[t][0], y0, c, 0, 0, 0);
    }
  }
};

template <int PREC, bool DIAG>
__device__ __forceinline__ void gram_tile(const ZetaArgs& z, const MDims& d, Operands<PREC>* lds,
                                          int m, int ti, int tj, int first, int r0, int r1,
                                          double* __restrict__ C) {
  using Op = Operands<PREC>;
  using Acc = typename Op::Acc;
  constexpr int kStep = Op::kStep, kRows = Op::kRows;
  const int tid = threadIdx.x;
  const int lane = tid % kWave;
  const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int W = d.W[m];
  const double* A = z.A + (long long)first * z.lay.W + d.off[m];
  const int* plist = z.plist + z.row_begin + first;
  const double* wsort = z.wsort + (z.cats ? first : 0);

  // staging: thread -> column tid % 128 of both panels, a quarter of the step's
  // rows (the same for a whole wave, so the rows' weights come by readlane)
  const int col = tid % kPanel, rg = __builtin_amdgcn_readfirstlane(tid / kPanel);
  const int ci = min(ti * kPanel + col, W - 1), cj = min(tj * kPanel + col, W - 1);
  // A step on its way: the thread's rows of both panels, and in lane r the weight
  // of the step's row r.  Rows and columns past the end are read from the last one,
  // so that no load hangs on a branch.
  struct Stage {
    double x[kRows], y[kRows], w;
  };
  auto index = [&](int kb) { return plist[min(kb + min(lane, kStep - 1), r1 - 1)]; };
  auto load = [&](Stage& g, int kb, int idx) {
    g.w = wsort[idx];
#pragma unroll
    for (int q = 0; q < kRows; ++q) {
      const double* row = A + min(kb + kRows * rg + q, r1 - 1) * (long long)z.lay.W;
      g.x[q] = row[ci];
      if constexpr (!DIAG) g.y[q] = row[cj];
    }
  };
  auto store = [&](Stage& g, int kb, int buf) {
    const long long wb = __double_as_longlong(g.w);
    const int wlo = int(wb & 0xffffffffll), whi = int(wb >> 32);
    double wgt[kRows];
#pragma unroll
    for (int q = 0; q < kRows; ++q) {
      const int lo = __builtin_amdgcn_readlane(wlo, kRows * rg + q);
      const int hi = __builtin_amdgcn_readlane(whi, kRows * rg + q);
      wgt[q] = __longlong_as_double((static_cast<long long>(hi) << 32) |
                                    static_cast<unsigned int>(lo));
    }
    if (kb + kStep > r1) {
#pragma unroll
      for (int q = 0; q < kRows; ++q)
        if (kb + kRows * rg + q >= r1) {
          g.x[q] = wgt[q] = 0.0;
          if constexpr (!DIAG) g.y[q] = 0.0;
        }
    }
    lds[buf].put(0, col, rg, g.x, wgt);
    if constexpr (DIAG)
      lds[buf].put(1, col, rg, g.x, wgt);
    else
      lds[buf].put(1, col, rg, g.y, wgt);
  };

  // this wave's units: pairs of tile rows (strips), the tiles of a strip from the
  // diagonal on (diagonal macro tiles) or all
  const int nti = (min(W - ti * kPanel, kPanel) + kTile - 1) / kTile;
  const int ntj = (min(W - tj * kPanel, kPanel) + kTile - 1) / kTile;
  int total = 0;
  for (int i = 0; i < nti; i += 2) total += DIAG ? ntj - i : ntj;
  const int per = (total + kGramWaves - 1) / kGramWaves;  // <= kUnits
  int ui[kUnits], uj[kUnits];
  {
    int i = 0, j = wv * per;  // j: units to skip, then the column within strip i
    while (i < nti && j >= (DIAG ? ntj - i : ntj)) {
      j -= DIAG ? ntj - i : ntj;
      i += 2;
    }
#pragma unroll
    for (int u = 0; u < kUnits; ++u) {
      const bool on = u < per && wv * per + u < total;
      ui[u] = on ? i : -1;
      uj[u] = on ? j + (DIAG ? i : 0) : 0;
      if (on && ++j >= (DIAG ? ntj - i : ntj)) {
        j = 0;
        i += 2;
      }
    }
  }

  Acc acc[kUnits][2];
  double4_t tot[kUnits][2];
#pragma unroll
  for (int u = 0; u < kUnits; ++u)
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      acc[u][t] = Acc{0, 0, 0, 0};
      tot[u][t] = double4_t{0.0, 0.0, 0.0, 0.0};
    }
  auto flush = [&]() {
#pragma unroll
    for (int u = 0; u < kUnits; ++u)
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          tot[u][t][r] += double(acc[u][t][r]);
          acc[u][t][r] = 0;
        }
  };

  auto products = [&](int kb, int buf) {
    if constexpr (PREC != G3PCF_PREC_FP64) {
      if (kb > r0 && (kb - r0) % kFlush == 0) flush();
    }
    typename Op::Left l;
#pragma unroll
    for (int u = 0; u < kUnits; ++u) {
      if (ui[u] < 0) continue;
      if (u == 0 || ui[u] != ui[u > 0 ? u - 1 : 0]) lds[buf].left(l, ui[u] * kTile, lane);
      lds[buf].unit(l, uj[u] * kTile, lane, acc[u]);
    }
  };

  // Two steps in flight besides the one in LDS: `even` and `odd` hold those of
  // their parity, and a step's row numbers are read a step before its rows.
  Stage even, odd;
  const int idx0 = index(r0), idx1 = index(r0 + kStep);
  int idx = index(r0 + 2 * kStep);
  load(even, r0, idx0);
  load(odd, r0 + kStep, idx1);
  store(even, r0, 0);
  __syncthreads();
  for (int kb = r0;; kb += 2 * kStep) {
    const int next = index(kb + 3 * kStep);
    load(even, kb + 2 * kStep, idx);
    products(kb, 0);
    if (kb + kStep >= r1) break;
    store(odd, kb + kStep, 1);
    __syncthreads();
    idx = index(kb + 4 * kStep);
    load(odd, kb + 3 * kStep, next);
    products(kb + kStep, 1);
    if (kb + 2 * kStep >= r1) break;
    store(even, kb + 2 * kStep, 0);
    __syncthreads();
  }
  flush();
  const int li = lane % 16, g = lane / 16;
#pragma unroll
  for (int u = 0; u < kUnits; ++u) {
    if (ui[u] < 0) continue;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = ti * kPanel + (ui[u] + t) * kTile + Op::row(g, r);
        const int j = tj * kPanel + uj[u] * kTile + li;
        if (i < W && j < W) C[i * W + j] = tot[u][t][r];
      }
  }
}

// Workgroups are numbered macro tile by macro tile, widest first, within chunks of
// at most kChunkMost blocks: the last workgroups of a launch are small ones, and the
// macro tiles of one m, which share panels, run close together.
constexpr int kChunkMost = 64;

template <int PREC>
__global__ __launch_bounds__(kGramThreads) void k_gram(ZetaArgs z, MDims d,
                                                       double* __restrict__ Cpart, int chunk) {
  __shared__ Operands<PREC> lds[2];
  const int tiles = d.mt[d.nm];
  const int t = int(blockIdx.x) / chunk;
  const int blk = t / tiles * chunk + int(blockIdx.x) % chunk;
  const GramBlocks g = gram_blocks(z);
  const unsigned long long past = __ballot(g.end > blk);
  if (!past) return;
  const int r = __builtin_ctzll(past);  // the block's list part
  const int rows = __builtin_amdgcn_readlane(g.rows, r);
  const int r0 = (blk - __builtin_amdgcn_readlane(g.begin, r)) * rows;
  const int r1 = min(__builtin_amdgcn_readlane(g.count, r), r0 + rows);
  const int first = __builtin_amdgcn_readlane(g.first, r);
  int m, ti, tj;
  macro_tile_of(d, t % tiles, m, ti, tj);
  double* C = Cpart + (long long)blk * d.csize + d.cw[m];
  if (ti == tj)
    gram_tile<PREC, true>(z, d, lds, m, ti, tj, first, r0, r1, C);
  else
    gram_tile<PREC, false>(z, d, lds, m, ti, tj, first, r0, r1, C);
}

// zeta[m][l][l'][b1][b2] += sum over the pair-block's blocks (in order, FP64)
// of the block Gram products.  Only tiles on or above the diagonal are read;
// C_m is symmetric.  One workgroup per 16 x 16 tile of one m's (l, b1)
// x (l', b2) entries, so that the partials are read in 128-byte pieces whether
// an entry is stored as it is or transposed, and list part; only the part's
// blocks are read.  Reading the partials bounds it: 166,100 doubles per block (lmax 10,
// 10 shells).
constexpr int kAT = 16;

__global__ __launch_bounds__(kAT * kAT) void k_zeta_accum_mt(ZetaArgs z, MDims d,
                                                             double* __restrict__ zeta) {
  const RowLayout& L = z.lay;
  const int nb = L.nb, nm = L.lmax + 1;
  // the pair kernel's next launch starts from cleared counters
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < kQueueAdjoint * kQueues)
    z.queue[threadIdx.x / kQueueAdjoint * kQueueStride + threadIdx.x % kQueueAdjoint] = 0;
  int t = blockIdx.x, m = 0;
  for (; m < nm; ++m) {
    const int nt = (L.d[m] + kAT - 1) / kAT;
    if (t < nt * nt) break;
    t -= nt * nt;
  }
  const int dm = L.d[m], nt = (dm + kAT - 1) / kAT, nl = nm - m;
  const int P = (t / nt) * kAT + int(threadIdx.x) / kAT, Pp = (t % nt) * kAT + int(threadIdx.x) % kAT;
  const GramBlocks g = gram_blocks(z);
  const int begin = __builtin_amdgcn_readlane(g.begin, blockIdx.y);
  const int nsub = __builtin_amdgcn_readlane(g.end, blockIdx.y) - begin;
  if (P >= dm || Pp >= dm || nsub == 0) return;
  const int W = d.W[m];
  auto at = [&](int i, int j) {
    if (i / kTile > j / kTile) {
      const int x = i;
      i = j;
      j = x;
    }
    return d.cw[m] + i * W + j;
  };
  const int Q = dm + P, Qp = dm + Pp;
  const int iPP = at(P, Pp);
  const int iQQ = (m > 0) ? at(Q, Qp) : 0, iQP = (m > 0) ? at(Q, Pp) : 0,
            iPQ = (m > 0) ? at(P, Qp) : 0;
  double re = 0.0, im = 0.0;
  const double* c = z.C64 + (long long)begin * d.csize;
  if (m == 0) {
#pragma unroll 4
    for (int s = 0; s < nsub; ++s, c += d.csize) re += c[iPP];
  } else {
#pragma unroll 4
    for (int s = 0; s < nsub; ++s, c += d.csize) {
      re += c[iPP] + c[iQQ];
      im += c[iQP] - c[iPQ];
    }
  }
  const int l = m + P % nl, b1 = P / nl, lp = m + Pp % nl, b2 = Pp / nl;
  zeta += 2LL * nm * nm * nm * nb * nb * blockIdx.y;
  double* o = zeta + ((((long long)m * nm + l) * nm + lp) * nb + b1) * (2LL * nb) + 2 * b2;
  o[0] += re;
  o[1] += im;
}

}  // namespace

int sum_wm2(const RowLayout& L) {
  int s = 0;
  for (int m = 0; m <= L.lmax; ++m) s += L.wm[m] * L.wm[m];
  return s;
}

RowLayout make_layout(int lmax, int nb) {
  RowLayout L{};
  L.lmax = lmax;
  L.nb = nb;
  int off = 0;
  for (int m = 0; m <= lmax; ++m) {
    L.off[m] = off;
    L.d[m] = (lmax + 1 - m) * nb;
    L.wm[m] = (m == 0) ? L.d[m] : 2 * L.d[m];
    off += L.wm[m];
  }
  L.off[lmax + 1] = off;
  L.W = off;
  return L;
}

// Partials of a pair-block of at most PB primaries.  4096 rows a block keep the
// partials few where there are many rows; a small pair-block is cut into more,
// until the macro tiles times the blocks give every CU, which holds one workgroup
// at a time, about two (a tile's 4096 rows are one serial chain of 128 steps: the
// Gram products of 16 catalogues of 8192, one launch each, took 4.55 ms in blocks of
// 4096 rows and 0.91 ms in 27 blocks; three or six workgroups a CU took the whole call
// 3 to 8% longer, the sum over the blocks growing with them).
static int zeta_blocks(const RowLayout& L, long long PB, int times) {
  const long long tiles = make_mdims(L).mt[L.lmax + 1];
  const long long fill = times * ((2 * 256 + tiles - 1) / tiles);
  const long long least = (PB + kZetaBlock - 1) / kZetaBlock;
  return int(std::max(least, std::min(fill, (PB + kZetaRowsMin - 1) / kZetaRowsMin)));
}

int zeta_parts(const RowLayout& L, long long PB) { return zeta_blocks(L, PB, 1); }

// Four times as many where a batch's small catalogues can fill them.
int zeta_room(const RowLayout& L, long long PB) { return zeta_blocks(L, PB, 4); }

// All blocks of a pair-block (z.K rows at most).
hipError_t launch_zeta_pairblock(const ZetaArgs& z, hipStream_t st) {
  const MDims d = make_mdims(z.lay);
  if (z.K <= 0) return hipSuccess;
  // at most `parts` blocks, each of at least kZetaRowsMin rows but a list part's last
  const long long blocks = std::min<long long>(
      z.parts, (z.K + kZetaRowsMin - 1) / kZetaRowsMin + z.lists - 1);
  const long long chunks = (blocks + kChunkMost - 1) / kChunkMost;
  const int chunk = int((blocks + chunks - 1) / chunks);
  const dim3 grid(unsigned(chunks * chunk * d.mt[d.nm]));
  const dim3 block(kGramThreads);
  if (z.prec == G3PCF_PREC_FP32)
    hipLaunchKernelGGL(k_gram<G3PCF_PREC_FP32>, grid, block, 0, st, z, d, z.C64, chunk);
  else if (z.prec == G3PCF_PREC_BF16X3)
    hipLaunchKernelGGL(k_gram<G3PCF_PREC_BF16X3>, grid, block, 0, st, z, d, z.C64, chunk);
  else
    hipLaunchKernelGGL(k_gram<G3PCF_PREC_FP64>, grid, block, 0, st, z, d, z.C64, chunk);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  unsigned ab = 0;
  for (int m = 0; m <= z.lay.lmax; ++m) {
    const unsigned nt = unsigned((z.lay.d[m] + kAT - 1) / kAT);
    ab += nt * nt;
  }
  hipLaunchKernelGGL(k_zeta_accum_mt, dim3(ab, unsigned(z.lists)), dim3(kAT * kAT), 0, st, z, d, z.zeta);
  return hipGetLastError();
}

// ---------------------------------------------------------------- degenerate triangles
// The triangles j = k (the same secondary on both sides, so b1 = b2) are part
// of the product a_lm conj(a_l'm) (Sec. 3.1).  Without them, zeta^m_{ll'}(b, b)
// loses sum_i w_i sum_{j in b} w_j^2 conj(Y_lm(u_ij)) Y_l'm(u_ij), which is
// sum_n G[m][l][l'][n] D(b, n) with D(b, n) = sum_i w_i sum_{j in b} w_j^2 T_n(u_z).

__device__ double g_deg[kDegTable];

namespace {

constexpr int kDegRows = 512;  // rows of a pair-block summed per workgroup

// partial[blk][c] = sum over the workgroup's rows r, in order, of w_r X[r][c]
// (c < ncols; rows of the pair-block that are not primaries are skipped).
__global__ __launch_bounds__(256) void k_deg_partial(const double* __restrict__ X, int rowW,
                                                     int ncols, const double* __restrict__ wsort,
                                                     const int* __restrict__ plist,
                                                     const long long* __restrict__ nprim,
                                                     const int* __restrict__ range,
                                                     long long p_begin, long long p_count,
                                                     double* __restrict__ partial) {
  long long first;
  const long long valid = valid_rows(nprim, range, p_begin, p_count, first);
  const long long r0 = (long long)blockIdx.x * kDegRows;
  const long long r1 = min(r0 + kDegRows, valid);
  if (r0 >= r1) return;
  X += first * rowW;
  plist += first;
  for (int c = threadIdx.x; c < ncols; c += blockDim.x) {
    double s = 0.0;
    for (long long r = r0; r < r1; ++r) s += wsort[plist[p_begin + r]] * X[r * rowW + c];
    partial[(long long)blockIdx.x * ncols + c] = s;
  }
}

// D[c] += sum over the workgroups, in order, of partial[blk][c]
__global__ void k_deg_accum(const double* __restrict__ partial,
                            const long long* __restrict__ nprim, const int* __restrict__ range,
                            long long p_begin, long long p_count, int ncols,
                            double* __restrict__ D, int* __restrict__ queue) {
  // the pair kernel's next launch starts from cleared counters
  if (blockIdx.x == 0 && threadIdx.x < kQueueAdjoint * kQueues)
    queue[threadIdx.x / kQueueAdjoint * kQueueStride + threadIdx.x % kQueueAdjoint] = 0;
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= ncols) return;
  long long first;
  const int nblk = int((valid_rows(nprim, range, p_begin, p_count, first) + kDegRows - 1) / kDegRows);
  double s = 0.0;
#pragma unroll 4
  for (int b = 0; b < nblk; ++b) s += partial[(long long)b * ncols + c];
  D[c] += s;
}

__device__ __forceinline__ long long zpos(int lmax, int nb, int m, int l, int lp, int b1,
                                          int b2) {
  const int L1 = lmax + 1;
  return ((((long long)m * L1 + l) * L1 + lp) * nb + b1) * nb + b2;
}

// Re zeta^m_{ll'}(b, b) -= sum_n G[m][l][l'][n] D[b][n]  (the removed terms are real)
__global__ void k_deg_apply(const double* __restrict__ D, int lmax, int nb,
                            double* __restrict__ zeta) {
  const int L1 = lmax + 1;
  const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (long long)L1 * L1 * L1 * nb) return;
  const int b = int(idx % nb);
  long long t = idx / nb;
  const int lp = int(t % L1);
  t /= L1;
  const int l = int(t % L1);
  const int m = int(t / L1);
  if (l < m || lp < m) return;
  const int nd = 2 * lmax + 1;
  double s = 0.0;
  for (int n = 0; n <= l + lp; ++n) s += g_deg[deg_index(m, l, lp, n)] * D[b * nd + n];
  zeta[zpos(lmax, nb, m, l, lp, b, b) * 2] -= s;
}

// iso[l][b1][b2] = 4 pi / (2l + 1) (zeta^0_ll + 2 sum_{m >= 1} Re zeta^m_ll)(b1, b2)
__global__ void k_isotropic(const double* __restrict__ zeta, int lmax, int nb,
                            double* __restrict__ iso) {
  const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (long long)(lmax + 1) * nb * nb) return;
  const int b2 = int(idx % nb);
  const int b1 = int((idx / nb) % nb);
  const int l = int(idx / ((long long)nb * nb));
  double s = 0.0;
  for (int m = 1; m <= l; ++m) s += zeta[zpos(lmax, nb, m, l, l, b1, b2) * 2];
  s = zeta[zpos(lmax, nb, 0, l, l, b1, b2) * 2] + 2.0 * s;
  iso[idx] = 4.0 * M_PI / (2.0 * l + 1.0) * s;
}

}  // namespace

hipError_t upload_deg_table() {
  static double host[kDegTable];
  static bool built = false;
  if (!built) {
    build_deg_table(host);
    built = true;
  }
  return hipMemcpyToSymbol(HIP_SYMBOL(g_deg), host, sizeof(host), 0, hipMemcpyHostToDevice);
}

size_t deg_partial_doubles(long long PB, int nb, int lmax) {
  return size_t((PB + kDegRows - 1) / kDegRows) * size_t(nb) * size_t(2 * lmax + 1);
}

hipError_t launch_deg_reduce(const double* X, int rowW, int nb, int lmax, const double* wsort,
                             const int* plist, const long long* nprim, const int* range,
                             long long p_begin, long long p_count, double* partial, double* D,
                             int* queue, hipStream_t st) {
  if (p_count <= 0) return hipSuccess;
  const int ncols = nb * (2 * lmax + 1);
  const unsigned nblk = unsigned((p_count + kDegRows - 1) / kDegRows);
  hipLaunchKernelGGL(k_deg_partial, dim3(nblk), dim3(256), 0, st, X, rowW, ncols, wsort, plist,
                     nprim, range, p_begin, p_count, partial);
  hipLaunchKernelGGL(k_deg_accum, dim3((ncols + 255) / 256), dim3(256), 0, st, partial,
                     nprim, range, p_begin, p_count, ncols, D, queue);
  return hipGetLastError();
}

hipError_t launch_deg_apply(const double* D, int lmax, int nb, double* zeta, hipStream_t st) {
  const long long n = (long long)(lmax + 1) * (lmax + 1) * (lmax + 1) * nb;
  hipLaunchKernelGGL(k_deg_apply, dim3(unsigned((n + 255) / 256)), dim3(256), 0, st, D, lmax,
                     nb, zeta);
  return hipGetLastError();
}

hipError_t launch_isotropic(const double* zeta, int lmax, int nb, double* iso, hipStream_t st) {
  const long long n = (long long)(lmax + 1) * nb * nb;
  hipLaunchKernelGGL(k_isotropic, dim3(unsigned((n + 255) / 256)), dim3(256), 0, st, zeta, lmax,
                     nb, iso);
  return hipGetLastError();
}

}  // namespace g3
