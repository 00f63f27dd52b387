// Catalogue staging: wrap, cell assignment, a stable sort into cell order
// (members of a cell in input order), and the compacted primary list.
//
// The paper keeps its galaxies in a node-local k-d tree for the range search
// (Algorithm 1, "search node-local k-d tree").  On the GPU a uniform cell grid
// sorted by a counting sort serves the same purpose: every (cy, cz) row of
// cells is one contiguous run of galaxies in memory, so the pair kernels read
// candidates with coalesced loads.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "internal.h"

namespace g3 {

namespace {

constexpr int kScanBlock = 256;
constexpr int kScanItems = 4;  // per thread
constexpr int kScanTile = kScanBlock * kScanItems;

__device__ inline double wrap_coord(double x, double lo, double L) {
  double t = x - lo;
  if (t >= 0.0 && t < L) return lo + t;  // fmod is exact: t itself
  t = fmod(t, L);
  if (t < 0.0) t += L;
  if (t >= L) t = 0.0;
  return lo + t;
}

template <typename Real>
struct Vec4;
template <>
struct Vec4<float> {
  using T = float4;
};
template <>
struct Vec4<double> {
  using T = double4;
};

struct GridDev {
  int nc[3];
  double inv_s[3], lo[3], L[3];
  int periodic;
};

// Cell along one axis; coordinates outside the box (open boxes) go to the
// edge cells, and a non-finite coordinate to cell 0 (such a galaxy is never
// accepted as a secondary and has no neighbours as a primary).
__device__ inline int cell_axis(double x, double lo, double inv_s, int nc) {
  const double f = floor((x - lo) * inv_s);
  if (!(f >= 0.0)) return 0;
  return f >= double(nc) ? nc - 1 : int(f);
}

// Wrap (periodic), convert to the compute precision and assign a cell: the
// staged value of galaxy i and its cell.
template <typename Real, typename In>
__device__ __forceinline__ typename Vec4<Real>::T staged(const In* __restrict__ pos,
                                                         const double* __restrict__ w, int64_t i,
                                                         const GridDev& g, int& cell) {
  double x[3];
  for (int a = 0; a < 3; ++a) {
    double v = double(pos[3 * i + a]);
    if (g.periodic) {
      v = wrap_coord(v, g.lo[a], g.L[a]);
      Real r = Real(v);
      // a float that rounds up onto the upper box edge wraps to the lower edge
      if (double(r) >= g.lo[a] + g.L[a]) r = Real(g.lo[a]);
      v = double(r);
    } else {
      v = double(Real(v));
    }
    x[a] = v;
  }
  const int cx = cell_axis(x[0], g.lo[0], g.inv_s[0], g.nc[0]);
  const int cy = cell_axis(x[1], g.lo[1], g.inv_s[1], g.nc[1]);
  const int cz = cell_axis(x[2], g.lo[2], g.inv_s[2], g.nc[2]);
  cell = (cz * g.nc[1] + cy) * g.nc[0] + cx;
  typename Vec4<Real>::T v4;
  v4.x = Real(x[0]);
  v4.y = Real(x[1]);
  v4.z = Real(x[2]);
  v4.w = Real(w[i]);
  return v4;
}

// ---- groups of shells ----
// Quotients of small numbers: x / d with inv about 1 / d, exact below 2^16 (an integer
// division is some thirty instructions).
__device__ __forceinline__ float about_inverse(int d) { return __builtin_amdgcn_rcpf(float(d)); }
__device__ __forceinline__ int quotient(int x, float inv) { return int((float(x) + 0.5f) * inv); }

__device__ __forceinline__ float wave_total(float v) {
  for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

// The table, by one wave: lane b finds how far a group from shell b on may reach, then
// the groups follow one another.  A galaxy shares its block with density x volume +
// excess others on average, and its run of cells too: the density of the footprint,
// and what clusters smaller than a run add.  blocks, runs: these averages times n.
__device__ __forceinline__ void form_groups(const ShellPlan& sp, float blocks, float runs,
                                            GroupTable* out) {
  const int lane = threadIdx.x % kWave;
  const float in_block = blocks / sp.n, in_run = runs / sp.n;
  // (cells wider than R_max: a block is a run, and nothing is known)
  const float crowd = sp.in_block > 1.5f * sp.in_run
                          ? fmaxf(1.0f, (in_block - in_run) / (sp.in_block - sp.in_run))
                          : 1.0f;
  const float density = sp.density * crowd;
  const float excess = fmaxf(0.0f, in_run - crowd * sp.in_run);
  auto fits = [&](int b, int last) {  // the pairs in shells b..last
    const float u = float(last + 1), v = float(b);
    return density * (u * u * u - v * v * v) + (b == 0 ? excess : 0.0f) <= sp.most;
  };
  int e = lane;
  while (e + 1 < sp.nbins && fits(lane, e + 1)) ++e;
  // a shell of its own goes through the list where that leaves nothing to the second
  // launch, or for the cartesian basis, whose later chunks then read it again
  const bool dense = !fits(sp.nbins - 1, sp.nbins - 1) || !fits(0, 0);
  const bool listed = e > lane || ((sp.cart || !dense) && fits(lane, lane));
  int searches = 0;
  for (int b = 0; b < sp.nbins; b = __builtin_amdgcn_readlane(e, b) + 1) ++searches;
  // (whole clusters of galaxies come and go in the shells of one primary and another:
  // lists that hold the mean overflow)
  const bool single = !sp.cart && (sp.nbins - searches < (dense ? kListSavesDense : kListSaves) ||
                                   excess > kListClusters);
  if (single) e = lane;
  int at = 0, nsingle = 0;
  for (int lists = 0; lists < 2; ++lists) {
    for (int b = 0; b < sp.nbins;) {
      const int last = __builtin_amdgcn_readlane(e, b);
      if (__builtin_amdgcn_readlane(int(listed && !single), b) == lists) {
        if (lane == 0) out->range[at] = b | last << 8;
        ++at;
      }
      b = last + 1;
    }
    if (lists == 0) nsingle = at;
  }
  if (lane == 0) {
    out->ngroup = at;
    out->nsingle = nsingle;
    out->density = density;
    out->excess = excess;
  }
}

template <typename Real, typename In>
__global__ void k_assign(const In* __restrict__ pos, const double* __restrict__ w, int64_t n,
                         GridDev g, typename Vec4<Real>::T* __restrict__ out4,
                         int* __restrict__ cid, int* __restrict__ count) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int c;
  out4[i] = staged<Real, In>(pos, w, i, g, c);
  cid[i] = c;
  atomicAdd(&count[c], 1);
}

// Every clear of a pass in one launch.
__global__ __launch_bounds__(256) void k_clear(Clears z) {
  const int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  const int64_t step = int64_t(gridDim.x) * blockDim.x;
  for (int k = 0; k < z.count; ++k)
    for (int64_t i = t; i < z.words[k]; i += step) z.at[k][i] = 0;
}

// ---- stable LSD radix sort of the cell ids (values: original indices) ----
// The galaxies come in input order, so a stable sort by cell id leaves every
// cell's members in increasing input order: the cell list is deterministic
// whatever the data (no atomics decide an order, and a crowded cell costs no
// more than a sparse one).  Digits of kRadixBits bits; each pass counts the
// digits of every tile of kRadixTile keys, scans the counts digit-major across
// tiles, and scatters each tile in order.
constexpr int kRadixBits = 8;
constexpr int kRadixDigits = 1 << kRadixBits;
constexpr int kRadixThreads = 256;
constexpr int kRadixRounds = 8;
constexpr int kRadixTile = kRadixThreads * kRadixRounds;
constexpr int kRadixWaves = kRadixThreads / kWave;

__global__ __launch_bounds__(kRadixThreads) void k_radix_hist(const int* __restrict__ keys,
                                                              int64_t n, int shift, int ntiles,
                                                              int* __restrict__ hist) {
  __shared__ int cnt[kRadixDigits];
  for (int d = threadIdx.x; d < kRadixDigits; d += kRadixThreads) cnt[d] = 0;
  __syncthreads();
  const int64_t base = int64_t(blockIdx.x) * kRadixTile;
  for (int k = 0; k < kRadixRounds; ++k) {
    const int64_t e = base + k * kRadixThreads + threadIdx.x;
    if (e < n) atomicAdd(&cnt[(keys[e] >> shift) & (kRadixDigits - 1)], 1);
  }
  __syncthreads();
  for (int d = threadIdx.x; d < kRadixDigits; d += kRadixThreads)
    hist[int64_t(d) * ntiles + blockIdx.x] = cnt[d];
}

// keys_in / vals_in (vals_in NULL: the value is the key's own index) into
// keys_out (NULL: not written) / vals_out at the scanned offsets.  Within a
// round of kRadixThreads keys, a key's rank among the keys of its wave with
// the same digit comes from eight ballots; the waves' counts per digit give
// the offsets across waves, and `base` carries each digit's running offset
// from round to round.
__global__ __launch_bounds__(kRadixThreads) void k_radix_scatter(
    const int* __restrict__ keys_in, const int* __restrict__ vals_in, int64_t n, int shift,
    int ntiles, const int* __restrict__ offs, int* __restrict__ keys_out,
    int* __restrict__ vals_out) {
  __shared__ int base[kRadixDigits];
  __shared__ int wcnt[kRadixWaves][kRadixDigits];
  for (int d = threadIdx.x; d < kRadixDigits; d += kRadixThreads) {
    base[d] = offs[int64_t(d) * ntiles + blockIdx.x];
    for (int w = 0; w < kRadixWaves; ++w) wcnt[w][d] = 0;
  }
  __syncthreads();
  const int wave = threadIdx.x / kWave;
  const int64_t tile0 = int64_t(blockIdx.x) * kRadixTile;
  for (int k = 0; k < kRadixRounds; ++k) {
    const int64_t e = tile0 + k * kRadixThreads + threadIdx.x;
    const bool valid = e < n;
    const int key = valid ? keys_in[e] : 0;
    const int val = valid ? (vals_in ? vals_in[e] : int(e)) : 0;
    const int d = (key >> shift) & (kRadixDigits - 1);
    unsigned long long peers = __builtin_amdgcn_ballot_w64(valid);
    for (int bit = 0; bit < kRadixBits; ++bit) {
      const bool on = (d >> bit) & 1;
      const unsigned long long b = __builtin_amdgcn_ballot_w64(on);
      peers &= on ? b : ~b;
    }
    const int rank = __builtin_amdgcn_mbcnt_hi(unsigned(peers >> 32),
                                               __builtin_amdgcn_mbcnt_lo(unsigned(peers), 0));
    if (valid && rank == 0) wcnt[wave][d] = __popcll(peers);
    __syncthreads();
    if (valid) {
      int off = base[d] + rank;
      for (int w = 0; w < wave; ++w) off += wcnt[w][d];
      if (keys_out) keys_out[off] = key;
      vals_out[off] = val;
    }
    __syncthreads();
    for (int t = threadIdx.x; t < kRadixDigits; t += kRadixThreads) {
      int add = 0;
      for (int w = 0; w < kRadixWaves; ++w) {
        add += wcnt[w][t];
        wcnt[w][t] = 0;
      }
      base[t] += add;
    }
    __syncthreads();
  }
}

// What the table follows from: the galaxies of the blocks of cells, a wave a block and a
// row of cells a lane, and those of the runs of cells in some rows, a wave a row and a
// run a lane (C and C (C - 1) summed over a row's runs).  (Atomic counts as the cells
// are assigned took 7 us for 16384 galaxies, 26 where they crowd into a fifth of the
// blocks; these take about two.)
__device__ __forceinline__ void count_blocks(const ShellPlan& sp,
                                             const int* __restrict__ cell_start,
                                             int* __restrict__ blocks) {
  const int waves = int(gridDim.x * blockDim.x / kWave), lane = threadIdx.x % kWave;
  const int wave = int((blockIdx.x * blockDim.x + threadIdx.x) / kWave);
  for (int b = wave; b < sp.blocks; b += waves) {
    const int row = b / sp.count[0], bx = b - row * sp.count[0];
    const int bz = row / sp.count[1], by = row - bz * sp.count[1];
    const int x0 = bx * sp.side[0], x1 = min(x0 + sp.side[0], sp.nc[0]);
    const int y0 = by * sp.side[1], ny = min(sp.side[1], sp.nc[1] - y0);
    const int z0 = bz * sp.side[2], nz = min(sp.side[2], sp.nc[2] - z0);
    int c = 0;
    for (int r = lane; r < ny * nz; r += kWave) {
      const int z = r / ny;
      const int* row0 = cell_start + ((z0 + z) * sp.nc[1] + y0 + r - z * ny) * sp.nc[0];
      c += row0[x1] - row0[x0];
    }
    for (int off = kWave / 2; off > 0; off >>= 1) c += __shfl_xor(c, off);
    if (lane == 0) blocks[b] = c;
  }
  int* sums = blocks + kCrowdBlocks;
  const int rows = sp.nc[1] * sp.nc[2];
  for (int i = wave; i < sp.rows; i += waves) {
    const int* row0 = cell_start + int64_t(i) * rows / sp.rows * sp.nc[0];
    float c1 = 0.0f, c2 = 0.0f;
    for (int x = lane * sp.run; x < sp.nc[0]; x += kWave * sp.run) {
      const float c = float(row0[min(x + sp.run, sp.nc[0])] - row0[x]);
      c1 += c;
      c2 += c * (c - 1.0f);
    }
    c1 = wave_total(c1);
    c2 = wave_total(c2);
    if (lane == 0) {
      sums[2 * i] = __float_as_int(c1);
      sums[2 * i + 1] = __float_as_int(c2);
    }
  }
}

// The table from these, in the last workgroup (of 256) of a launch that has one more
// for it; true there.
__device__ __forceinline__ bool groups_workgroup(const ShellPlan& sp,
                                                 const int* __restrict__ blocks,
                                                 GroupTable* __restrict__ groups) {
  if (!sp.lists || blockIdx.x + 1 < gridDim.x) return false;
  __shared__ float part[3][256 / kWave];
  float v[3] = {0.0f, 0.0f, 0.0f};
  for (int i = threadIdx.x; i < sp.blocks; i += 256) {
    const float c = float(blocks[i]);
    v[0] += c * (c - 1.0f);
  }
  const int* sums = blocks + kCrowdBlocks;
  for (int i = threadIdx.x; i < sp.rows; i += 256) {
    v[1] += __int_as_float(sums[2 * i]);
    v[2] += __int_as_float(sums[2 * i + 1]);
  }
  for (int k = 0; k < 3; ++k) {
    v[k] = wave_total(v[k]);
    if (threadIdx.x % kWave == 0) part[k][threadIdx.x / kWave] = v[k];
  }
  __syncthreads();
  if (threadIdx.x < kWave) {
    for (int k = 0; k < 3; ++k) v[k] = part[k][0] + part[k][1] + part[k][2] + part[k][3];
    form_groups(sp, v[0], v[2] / fmaxf(v[1], 1.0f) * sp.n, groups);
  }
  return true;
}

// Cell-order arrays from the sorted original indices, and the kSentinel NaN
// entries after them; the blocks' counts, where shells may be searched together.
template <typename V4>
__global__ __launch_bounds__(256) void k_gather_sorted(
    const V4* __restrict__ in4, const int* __restrict__ perm, int64_t n,
    const double* __restrict__ w, V4* __restrict__ out4, double* __restrict__ wsort, ShellPlan sp,
    const int* __restrict__ cell_start, int* __restrict__ blocks) {
  if (sp.lists) count_blocks(sp, cell_start, blocks);
  const int64_t s = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (s >= n) {
    if (s < n + kSentinel) {
      using T = decltype(out4[0].x);
      const T nan = T(__builtin_nan(""));
      out4[s] = V4{nan, nan, nan, nan};
    }
    return;
  }
  const int i = perm[s];
  out4[s] = in4[i];
  wsort[s] = w[i];
}

// primary flag of the galaxy in cell-order slot s
__global__ __launch_bounds__(256) void k_primary_flags(
    const uint8_t* __restrict__ mask, const int* __restrict__ perm, int64_t n,
    int* __restrict__ flags, ShellPlan sp, const int* __restrict__ blocks,
    GroupTable* __restrict__ groups) {
  if (groups_workgroup(sp, blocks, groups)) return;
  const int64_t s = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (s > n) return;
  flags[s] = s < n && mask[perm[s]] != 0 ? 1 : 0;
}

// region (from region0) of the galaxy in slot s; nregions: none of them
__global__ void k_region_keys(const uint8_t* __restrict__ mask,
                              const int32_t* __restrict__ region, int region0, int nregions,
                              const int* __restrict__ perm, int64_t n, int* __restrict__ keys,
                              int* __restrict__ flags) {
  const int64_t s = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (s > n) return;
  flags[s] = 0;
  if (s == n) return;
  const int i = perm[s];
  const int64_t r = int64_t(region[i]) - region0;
  keys[s] = r >= 0 && r < nregions && (mask == nullptr || mask[i] != 0) ? int(r) : nregions;
}

// starts[r] = slots sorted below region r
__global__ void k_region_starts(const int* __restrict__ keys, int64_t n, int nregions,
                                int* __restrict__ starts, long long* __restrict__ nprim) {
  const int r = int(blockIdx.x) * blockDim.x + threadIdx.x;
  if (r > nregions) return;
  int64_t lo = 0, hi = n;
  while (lo < hi) {
    const int64_t mid = (lo + hi) / 2;
    if (keys[mid] < r) lo = mid + 1;
    else hi = mid;
  }
  starts[r] = int(lo);
  if (r == nregions) *nprim = lo;
}

// every galaxy a primary
__global__ __launch_bounds__(256) void k_primary_all(
    int* __restrict__ flags, int64_t n, int* __restrict__ plist, long long* __restrict__ nprim,
    ShellPlan sp, const int* __restrict__ blocks, GroupTable* __restrict__ groups) {
  if (groups_workgroup(sp, blocks, groups)) return;
  const int64_t s = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (s > n) return;
  flags[s] = 0;
  if (s == n) *nprim = n;
  else plist[s] = int(s);
}

// the table alone
__global__ __launch_bounds__(256) void k_groups(ShellPlan sp, const int* __restrict__ blocks,
                                                GroupTable* __restrict__ groups) {
  groups_workgroup(sp, blocks, groups);
}

// (the flags are left zero)
__global__ void k_primary_list(int* __restrict__ flags, const int* __restrict__ pos,
                               int64_t n, int* __restrict__ plist,
                               long long* __restrict__ nprim) {
  const int64_t s = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (s > n) return;
  if (s == n) {
    *nprim = pos[n];
    return;
  }
  if (flags[s]) plist[pos[s]] = int(s);
  flags[s] = 0;
}

// ---- the whole cell stage of a small catalogue in one workgroup ----
// Up to kSmallN galaxies: the launches of the general path (17 with a mask, each
// 2 to 5 us and as much again between them) cost more than one workgroup's time.
// Bound by the workgroup's instruction issue over two sort passes of two rounds of
// ballots.  The cell ids stay in LDS (below 2^16: the grid has at most 4 n cells) and the
// same stable LSD radix sort by 8-bit digits runs over contiguous chunks, one a
// wave, so the order is that of the general path.  The other workgroups of the
// launch do the pass's clears.
constexpr int kSmallThreads = 1024;
constexpr int kSmallWaves = kSmallThreads / kWave;

struct SmallOut {
  int* perm;
  double* wsort;
  int* cell_start;
  int ncell;
  int* flags;                // [n + 1] zeroed, or NULL: no primary list
  int* plist;
  long long* nprim;
  int* counters;             // zeroed
  int counter_words;
  GroupTable* groups;
};

template <int N>
struct SmallLds {
  unsigned short key[N];
  unsigned short val[2][N];
  union {
    unsigned short hist[kSmallWaves][kRadixDigits];  // then running offsets
    int blocks[kCrowdBlocks];                        // before them
  };
  int wtot[kSmallWaves];
  float wsum[2][kSmallWaves];                      // the table's sums
};

// One workgroup's catalogue of n <= N galaxies; the NaN entries go to nan4.
template <typename Real, typename In, int N>
__device__ __forceinline__ void cells_small(SmallLds<N>& lds, const In* __restrict__ pos,
                                            const double* __restrict__ w, int n, const GridDev& g,
                                            const ShellPlan& sp,
                                            const uint8_t* __restrict__ mask,
                                            typename Vec4<Real>::T* stage4,
                                            typename Vec4<Real>::T* __restrict__ pos4,
                                            typename Vec4<Real>::T* nan4, const SmallOut& o) {
  using V4 = typename Vec4<Real>::T;
  auto& key = lds.key;
  auto& val = lds.val;
  auto& hist = lds.hist;
  auto& wtot = lds.wtot;
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  for (int i = tid; i < o.counter_words; i += kSmallThreads) o.counters[i] = 0;
  const float per_x = about_inverse(sp.nc[0]), per_y = about_inverse(sp.nc[1]);
  if (sp.lists) {
    for (int i = tid; i < sp.blocks; i += kSmallThreads) lds.blocks[i] = 0;
    __syncthreads();
  }
  const float bx = about_inverse(sp.side[0]), by = about_inverse(sp.side[1]),
              bz = about_inverse(sp.side[2]);
  for (int i = tid; i < n; i += kSmallThreads) {
    int c;
    stage4[i] = staged<Real, In>(pos, w, i, g, c);
    key[i] = (unsigned short)c;
    val[0][i] = (unsigned short)i;
    if (sp.lists) {
      const int row = quotient(c, per_x), z = quotient(row, per_y);
      const int b = (quotient(z, bz) * sp.count[1] + quotient(row - z * sp.nc[1], by)) *
                        sp.count[0] + quotient(c - row * sp.nc[0], bx);
      atomicAdd(&lds.blocks[b], 1);
    }
  }
  if (sp.lists) {
    __syncthreads();
    float sum = 0.0f;
    for (int i = tid; i < sp.blocks; i += kSmallThreads) {
      const float c = float(lds.blocks[i]);
      sum += c * (c - 1.0f);
    }
    sum = wave_total(sum);
    if (lane == 0) lds.wsum[0][wave] = sum;
    __syncthreads();
  }
  const int chunk = (n + kSmallThreads - 1) / kSmallThreads * kWave;  // per wave
  const int c0 = wave * chunk, c1 = min(n, c0 + chunk);
  const int passes = o.ncell > kRadixDigits ? 2 : 1;
  for (int pass = 0; pass < passes; ++pass) {
    const unsigned short* in = val[pass];
    unsigned short* out = val[pass ^ 1];
    const int shift = pass * kRadixBits;
    for (int d = lane; d < kRadixDigits; d += kWave) hist[wave][d] = 0;
    __syncthreads();
    // the lane's digit, its rank among the wave's equal digits and their number
    auto match = [&](int e, int& d, int& v, int& rank, int& same) {
      const bool valid = e < c1;
      v = valid ? in[e] : 0;
      d = valid ? (key[v] >> shift) & (kRadixDigits - 1) : 0;
      unsigned long long peers = __builtin_amdgcn_ballot_w64(valid);
      for (int bit = 0; bit < kRadixBits; ++bit) {
        const bool on = (d >> bit) & 1;
        const unsigned long long b = __builtin_amdgcn_ballot_w64(on);
        peers &= on ? b : ~b;
      }
      rank = __builtin_amdgcn_mbcnt_hi(unsigned(peers >> 32),
                                       __builtin_amdgcn_mbcnt_lo(unsigned(peers), 0));
      same = __popcll(peers);
      return valid;
    };
    for (int e = c0 + lane; e - lane < c1; e += kWave) {
      int d, v, rank, same;
      if (match(e, d, v, rank, same) && rank == 0)
        hist[wave][d] = (unsigned short)(hist[wave][d] + same);
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
      __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    // offsets, digit-major across waves: a thread for four waves of a digit
    {
      static_assert(kSmallThreads * 4 == kRadixDigits * kSmallWaves, "four counts a thread");
      const int d = tid / 4, u0 = 4 * (tid % 4);
      int c[4], sum = 0;
      for (int k = 0; k < 4; ++k) {
        c[k] = hist[u0 + k][d];
        sum += c[k];
      }
      int incl = sum;
      for (int off = 1; off < kWave; off <<= 1) {
        const int up = __shfl_up(incl, off);
        if (lane >= off) incl += up;
      }
      if (lane == kWave - 1) wtot[wave] = incl;
      __syncthreads();
      int at = incl - sum;
      for (int u = 0; u < kSmallWaves; ++u) at += u < wave ? wtot[u] : 0;
      for (int k = 0; k < 4; ++k) {
        hist[u0 + k][d] = (unsigned short)at;
        at += c[k];
      }
    }
    __syncthreads();
    for (int e = c0 + lane; e - lane < c1; e += kWave) {
      int d, v, rank, same;
      const bool valid = match(e, d, v, rank, same);
      const int at = valid ? hist[wave][d] : 0;
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
      __builtin_amdgcn_wave_barrier();
      if (valid) out[at + rank] = (unsigned short)v;
      if (valid && rank == 0) hist[wave][d] = (unsigned short)(at + same);
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
      __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
  }
  const unsigned short* order = val[passes & 1];
  for (int s = tid; s < n + kSentinel; s += kSmallThreads) {
    if (s < n) {
      const int i = order[s];
      o.perm[s] = i;
      pos4[s] = stage4[i];
      o.wsort[s] = w[i];
    } else {
      const Real nan = Real(__builtin_nan(""));
      nan4[s - n] = V4{nan, nan, nan, nan};
    }
  }
  auto cell_at = [&](int s) { return int(key[order[s]]); };
  if (sp.lists) {
    // pairs that share a run of cells: from each galaxy on, at most a wave of them
    const int per_row = (sp.nc[0] + sp.run - 1) / sp.run;
    const float per_run = about_inverse(sp.run);
    auto run_at = [&](int s) {
      const int c = cell_at(s), row = quotient(c, per_x);
      return row * per_row + quotient(c - row * sp.nc[0], per_run);
    };
    float sum = 0.0f;
    for (int s = tid; s < n; s += kSmallThreads) {
      const int r = run_at(s), end = min(n, s + kWave);
      for (int t = s + 1; t < end && run_at(t) == r; ++t) sum += 2.0f;
    }
    sum = wave_total(sum);
    if (lane == 0) lds.wsum[1][wave] = sum;
    __syncthreads();
    if (wave == kSmallWaves - 1) {
      float v[2] = {0.0f, 0.0f};
      for (int u = 0; u < kSmallWaves; ++u)
        for (int k = 0; k < 2; ++k) v[k] += lds.wsum[k][u];
      form_groups(sp, v[0], v[1], o.groups);
    }
  }
  // cell_start[c] = galaxies in cells below c; a run of cells per thread, the
  // next start found by doubling steps
  const int per = (o.ncell + 1 + kSmallThreads - 1) / kSmallThreads;
  int s = 0;
  for (int c = tid * per; c < min((tid + 1) * per, o.ncell + 1); ++c) {
    int step = c == tid * per ? n : 1;  // the thread's first cell: a plain bisection
    int hi = s;
    while (hi < n && cell_at(hi) < c) {
      s = hi + 1;
      hi = min(hi + step, n);
      step *= 2;
    }
    while (s < hi) {  // first slot whose cell is not below c
      const int mid = (s + hi) / 2;
      if (cell_at(mid) < c) s = mid + 1;
      else hi = mid;
    }
    o.cell_start[c] = s;
  }
  if (!o.flags) return;
  // primaries in cell order
  for (int i = tid; i <= n; i += kSmallThreads) o.flags[i] = 0;
  if (!mask) {
    for (int i = tid; i < n; i += kSmallThreads) o.plist[i] = i;
    if (tid == 0) *o.nprim = n;
    return;
  }
  int base = 0;
  for (int s0 = 0; s0 < n; s0 += kSmallThreads) {
    const int q = s0 + tid;
    const bool on = q < n && mask[order[q]] != 0;
    const unsigned long long b = __builtin_amdgcn_ballot_w64(on);
    if (lane == 0) wtot[wave] = __popcll(b);
    __syncthreads();
    int before = base;
    for (int u = 0; u < kSmallWaves; ++u) {
      if (u < wave) before += wtot[u];
      base += wtot[u];
    }
    if (on)
      o.plist[before + __builtin_amdgcn_mbcnt_hi(unsigned(b >> 32),
                                                 __builtin_amdgcn_mbcnt_lo(unsigned(b), 0))] = q;
    __syncthreads();
  }
  if (tid == 0) *o.nprim = base;
}

template <typename Real, typename In>
__global__ __launch_bounds__(kSmallThreads) void k_cells_small(
    const In* __restrict__ pos, const double* __restrict__ w, int n, GridDev g, ShellPlan sp,
    const uint8_t* __restrict__ mask, typename Vec4<Real>::T* stage4,
    typename Vec4<Real>::T* __restrict__ pos4, SmallOut o, Clears z) {
  __shared__ SmallLds<kSmallN> lds;
  if (blockIdx.x > 0) {
    const int64_t t = int64_t(blockIdx.x - 1) * kSmallThreads + threadIdx.x;
    const int64_t step = int64_t(gridDim.x - 1) * kSmallThreads;
    for (int k = 0; k < z.count; ++k)
      for (int64_t i = t; i < z.words[k]; i += step) z.at[k][i] = 0;
    return;
  }
  cells_small<Real, In>(lds, pos, w, n, g, sp, mask, stage4, pos4, pos4 + n, o);
}

// A workgroup per catalogue of a batch.
struct BatchGrids {
  GridDev g[kBatchGroup];
  ShellPlan plan[kBatchGroup];
  int first[kBatchGroup], n[kBatchGroup], ncell[kBatchGroup], cells_at[kBatchGroup],
      parts[kBatchGroup];
};
static_assert(sizeof(BatchGrids) + sizeof(SmallOut) <= 3584, "kernel arguments");

template <typename Real, typename In>
__global__ __launch_bounds__(kSmallThreads) void k_cells_batch(
    const In* __restrict__ pos, const double* __restrict__ w, BatchGrids b,
    const uint8_t* __restrict__ mask, typename Vec4<Real>::T* stage4,
    typename Vec4<Real>::T* __restrict__ pos4, typename Vec4<Real>::T* nan4, SmallOut o) {
  __shared__ SmallLds<kBatchN> lds;
  const int c = blockIdx.x;
  const int at = b.first[c];
  SmallOut oc{o.perm + at,  o.wsort + at, o.cell_start + b.cells_at[c], b.ncell[c],
              o.flags + at, o.plist + at, o.nprim + c * kCatStride,
              o.counters + c * kCatStride * 2, kCatStride * 2,
              reinterpret_cast<GroupTable*>(o.nprim + c * kCatStride + kCatGroups)};
  cells_small<Real, In>(lds, pos + 3 * int64_t(at), w + at, b.n[c], b.g[c], b.plan[c],
                        mask ? mask + at : nullptr, stage4 + at, pos4 + at, nan4, oc);
  // (after the barriers that follow the counters' clear)
  if (threadIdx.x == 0) {
    oc.nprim[kCatFirst] = at - b.first[0];
    oc.nprim[kCatParts] = b.parts[c];
  }
}

__global__ void k_fill_int(int* p, int64_t count, int value) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < count) p[i] = value;
}

__global__ void k_fill_double(double* p, int64_t count, double value) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < count) p[i] = value;
}

// ---- exclusive scan of int32 (three phases, recursive over tile sums) ----
__global__ void k_scan_tiles(const int* __restrict__ in, int* __restrict__ out, int64_t count,
                             int* __restrict__ tile_sums) {
  __shared__ int sh[kScanBlock];
  const int64_t base = int64_t(blockIdx.x) * kScanTile + threadIdx.x * kScanItems;
  int v[kScanItems];
  int s = 0;
  for (int k = 0; k < kScanItems; ++k) {
    const int64_t i = base + k;
    v[k] = (i < count) ? in[i] : 0;
    s += v[k];
  }
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int off = 1; off < kScanBlock; off <<= 1) {
    int t = (threadIdx.x >= off) ? sh[threadIdx.x - off] : 0;
    __syncthreads();
    sh[threadIdx.x] += t;
    __syncthreads();
  }
  int run = sh[threadIdx.x] - s;  // exclusive prefix of this thread
  for (int k = 0; k < kScanItems; ++k) {
    const int64_t i = base + k;
    if (i < count) out[i] = run;
    run += v[k];
  }
  if (threadIdx.x == kScanBlock - 1) tile_sums[blockIdx.x] = sh[threadIdx.x];
}

__global__ void k_scan_add(int* __restrict__ out, int64_t count,
                           const int* __restrict__ tile_offsets) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < count) out[i] += tile_offsets[i / kScanTile];
}

inline unsigned blocks_for(int64_t n, int bs) { return unsigned((n + bs - 1) / bs); }

// splitmix64 output function (Steele, Lea and Flood, OOPSLA 2014)
__device__ __forceinline__ unsigned long long mix64(unsigned long long x) {
  x ^= x >> 30;
  x *= 0xbf58476d1ce4e5b9ull;
  x ^= x >> 27;
  x *= 0x94d049bb133111ebull;
  return x ^ (x >> 31);
}

constexpr int kPrintBlocks = 1024;

// Fingerprint of everything the a_lm rows depend on besides the settings:
// per cell-order slot its original index, stored position words and weight,
// and the primary list.  A wrapping sum of per-slot hashes (one atomic per
// workgroup), so the value does not depend on the order of the atomics.
__global__ __launch_bounds__(256) void k_fingerprint(const unsigned* __restrict__ pos_words,
                                                     int words, const double* __restrict__ wsort,
                                                     const int* __restrict__ perm,
                                                     const int* __restrict__ plist,
                                                     const long long* __restrict__ nprim,
                                                     int64_t n, unsigned long long seed,
                                                     unsigned long long* __restrict__ out) {
  __shared__ unsigned long long part[256 / kWave];
  const long long np = *nprim;
  unsigned long long h = 0;
  for (int64_t s = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; s < n;
       s += int64_t(gridDim.x) * blockDim.x) {
    unsigned long long x = mix64(seed + (unsigned long long)s);
    x = mix64(x ^ (unsigned)perm[s]);
    for (int k = 0; k < words; ++k) x = mix64(x ^ pos_words[s * words + k]);
    x = mix64(x ^ (unsigned long long)__double_as_longlong(wsort[s]));
    h += x;
    if (s < np) h += mix64(~seed ^ ((unsigned long long)s << 32) ^ (unsigned)plist[s]);
  }
  for (int off = kWave / 2; off > 0; off >>= 1) h += __shfl_xor(h, off);
  const int wave = threadIdx.x / kWave;
  if (threadIdx.x % kWave == 0) part[wave] = h;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long t = 0;
    for (int k = 0; k < int(blockDim.x) / kWave; ++k) t += part[k];
    atomicAdd(out, t);
  }
}

}  // namespace

hipError_t launch_fingerprint(const void* pos4, int fp64, const double* wsort, const int* perm,
                              const int* plist, const long long* nprim, int64_t n,
                              unsigned long long seed, unsigned long long* out, hipStream_t st) {
  const unsigned nb = std::min<unsigned>(kPrintBlocks, std::max(1u, blocks_for(n, 256)));
  hipLaunchKernelGGL(k_fingerprint, dim3(nb), dim3(256), 0, st,
                     static_cast<const unsigned*>(pos4), fp64 ? 8 : 4, wsort, perm, plist, nprim,
                     n, seed, out);
  return hipGetLastError();
}

size_t scan_tmp_bytes(int64_t count) {
  size_t total = 0;
  int64_t c = count;
  while (c > 1) {
    const int64_t tiles = (c + kScanTile - 1) / kScanTile;
    total += size_t(2 * tiles + 64) * sizeof(int);
    c = tiles;
  }
  return total + 256;
}

hipError_t launch_scan(const int* in, int* out, int64_t count, void* tmp, size_t tmp_bytes,
                       hipStream_t st) {
  if (count <= 0) return hipSuccess;
  const int64_t tiles = (count + kScanTile - 1) / kScanTile;
  int* sums = static_cast<int*>(tmp);
  int* offs = sums + tiles + 32;
  hipLaunchKernelGGL(k_scan_tiles, dim3(unsigned(tiles)), dim3(kScanBlock), 0, st, in, out,
                     count, sums);
  if (tiles > 1) {
    const size_t used = size_t(2 * tiles + 64) * sizeof(int);
    hipError_t e = launch_scan(sums, offs, tiles, static_cast<char*>(tmp) + used,
                               tmp_bytes - used, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_scan_add, dim3(blocks_for(count, 256)), dim3(256), 0, st, out, count,
                       offs);
  }
  return hipGetLastError();
}

hipError_t launch_clears(const Clears& z, hipStream_t st) {
  int64_t most = 0;
  for (int k = 0; k < z.count; ++k) most = std::max(most, z.words[k]);
  if (most == 0) return hipSuccess;
  hipLaunchKernelGGL(k_clear, dim3(std::min(2048u, blocks_for(most, 256))), dim3(256), 0, st, z);
  return hipGetLastError();
}

hipError_t launch_fill_int(int* p, int64_t count, int value, hipStream_t st) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_int, dim3(blocks_for(count, 256)), dim3(256), 0, st, p, count,
                     value);
  return hipGetLastError();
}

hipError_t launch_fill_double(double* p, int64_t count, double value, hipStream_t st) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_double, dim3(blocks_for(count, 256)), dim3(256), 0, st, p, count,
                     value);
  return hipGetLastError();
}

Grid make_grid(const g3pcf_problem& p) {
  Grid g{};
  g.periodic = p.periodic ? 1 : 0;
  // Margin so that every candidate the FP32 acceptance test can accept is
  // visited: positions carry about 1e-7 relative rounding.
  double ext = 0.0;
  for (int a = 0; a < 3; ++a)
    ext = std::max(ext, std::fabs(p.box_lo[a]) + std::fabs(p.box[a]));
  g.rsearch = p.rmax * (1.0 + 1e-5) + 1e-6 * ext + 1e-9;
  // Cells of about R_max / 8 across the rows and R_max / 64 along x: a row
  // (cy, cz) of cells is a contiguous run of galaxies, and the x-interval of
  // an annulus in a row is cut to within one thin cell at each end.
  const double target[3] = {p.rmax / 64.0, p.rmax / 8.0, p.rmax / 8.0};
  int64_t cap = std::max<int64_t>(64, 4 * p.n);
  cap = std::min<int64_t>(cap, int64_t(1) << 24);
  for (int a = 0; a < 3; ++a) {
    g.lo[a] = p.box_lo[a];
    g.L[a] = p.box[a];
    double nc = std::floor(p.box[a] / target[a]);
    nc = std::max(1.0, std::min(nc, 4096.0));
    g.nc[a] = int(nc);
  }
  while (int64_t(g.nc[0]) * g.nc[1] * g.nc[2] > cap) {
    for (int a = 0; a < 3; ++a) g.nc[a] = std::max(1, (g.nc[a] * 4) / 5);
  }
  for (int a = 0; a < 3; ++a) {
    g.s[a] = g.L[a] / g.nc[a];
    g.inv_s[a] = double(g.nc[a]) / g.L[a];
    // periodic axis where [x - R, x + R] can touch more than nc cells
    g.tight[a] = (g.periodic && (2.0 * g.rsearch + 2.0 * g.s[a] >= g.L[a])) ? 1 : 0;
  }
  g.ncell = int64_t(g.nc[0]) * g.nc[1] * g.nc[2];
  return g;
}

// Which shells may be searched together.  Neighbouring shells whose expected pairs fit
// the list make one group: a search costs a wave about 10 us of waiting however little
// it finds (16 catalogues of 8192 with 274 pairs a primary: 5.5 ms a call shell by
// shell, 4.1 in groups; FP64 step of 4096 with 137 pairs: 802 and 607 us).  Not
// where every shell of every primary can have a wave of its own.  The pairs expected
// follow from the density around the galaxies, which is the mean over the declared box
// or (a footprint that fills part of it, clusters) more: the device measures it with
// the cell list and forms the groups (see form_groups).  Taking the mean as it stands,
// lists overflowed for most primaries of such catalogues, and everything was searched
// twice (16384 galaxies in the lowest fifth of their box, 849 pairs, l_max 4: 630 us of
// the call; shell by shell 411).  Where even the mean leaves no groups worth a second
// launch, nothing is measured.  Depends on the catalogue and the settings alone, so
// that every entry point sums a shell's pairs in the same order.
ShellPlan shell_plan(const g3pcf_problem& p, const Grid& g) {
  ShellPlan sp{};
  sp.nbins = p.nbins;
  sp.cart = p.basis == G3PCF_BASIS_CARTESIAN;
  const double most = p.pair_prec == G3PCF_PREC_FP64 ? kListMean64 : kListMean32;
  const double dr = p.rmax / p.nbins;
  const double density =
      double(p.n) / (p.box[0] * p.box[1] * p.box[2]) * 4.0 / 3.0 * M_PI * dr * dr * dr;
  auto cube = [](double x) { return x * x * x; };
  int searches = 0;
  for (int b = 0, e; b < p.nbins; b = e + 1, ++searches)
    for (e = b; e + 1 < p.nbins && density * (cube(e + 2) - cube(b)) <= most;) ++e;
  const int least =
      density * (cube(p.nbins) - cube(p.nbins - 1.0)) > most ? kListSavesDense : kListSaves;
  // nor on a tight axis (few cells, and the kernels would double)
  if (p.n * p.nbins <= kPairWaves || g.tight[0] || g.tight[1] || g.tight[2] ||
      (sp.cart ? density > most : p.nbins - searches < least))
    return sp;
  sp.lists = 1;
  sp.density = float(density);
  // (a uniform catalogue's measured density is a few per cent off its mean)
  sp.most = float(kListSlack * most);
  int64_t count[3];
  for (int a = 0; a < 3; ++a)
    sp.side[a] = std::max(1, std::min(g.nc[a], int(std::lround(p.rmax * g.inv_s[a]))));
  for (;;) {
    for (int a = 0; a < 3; ++a) count[a] = (g.nc[a] + sp.side[a] - 1) / sp.side[a];
    if (count[0] * count[1] * count[2] <= kCrowdBlocks) break;
    for (int a = 0; a < 3; ++a) sp.side[a] += std::max(1, sp.side[a] / 8);
  }
  // chances of two points of the box to share a block, and a run of cells
  auto share = [](int side, int nc) {
    const int whole = nc / side, rest = nc % side;
    return (double(whole) * side * side + double(rest) * rest) / (double(nc) * nc);
  };
  double in_block = 1.0;
  for (int a = 0; a < 3; ++a) {
    in_block *= share(sp.side[a], g.nc[a]);
    sp.nc[a] = g.nc[a];
    sp.count[a] = int(count[a]);
  }
  // (runs of R_max / 8, as long as a cell is wide unless the grid is coarse)
  sp.run = std::max(1, int(std::lround(0.125 * p.rmax * g.inv_s[0])));
  const double in_run = share(sp.run, g.nc[0]) / (double(g.nc[1]) * g.nc[2]);
  sp.blocks = sp.count[0] * sp.count[1] * sp.count[2];
  sp.rows = std::min(kCrowdBlocks, g.nc[1] * g.nc[2]);
  sp.n = float(p.n);
  sp.in_block = float(double(p.n - 1) * in_block);
  sp.in_run = float(double(p.n - 1) * in_run);
  return sp;
}

size_t radix_hist_ints(int64_t n) {
  const int64_t ntiles = std::max<int64_t>(1, (n + kRadixTile - 1) / kRadixTile);
  return size_t(ntiles) * kRadixDigits;
}

// Indices 0..n-1 sorted stably by the keys in b.key_a (below `bound`) into `out`;
// the sorted keys into *keys, if it is not NULL.
static hipError_t radix_sort(const CellBufs& b, int64_t n, int64_t bound, int* out, int** keys,
                             hipStream_t st) {
  int bits = 0;
  while ((int64_t(1) << bits) < bound) ++bits;
  const int passes = std::max(1, (bits + kRadixBits - 1) / kRadixBits);
  const int ntiles = int((n + kRadixTile - 1) / kRadixTile);
  const int64_t nh = int64_t(ntiles) * kRadixDigits;
  int* hist = b.hist;
  int* offs = b.hist + nh;
  const int* kin = b.key_a;
  const int* vin = nullptr;
  hipError_t e;
  for (int pass = 0; pass < passes; ++pass) {
    const int shift = pass * kRadixBits;
    const bool last = pass + 1 == passes;
    int* kout = last && !keys ? nullptr : (kin == b.key_a ? b.key_b : b.key_a);
    // the last pass writes out; the ones before alternate so that it does
    int* vout = ((passes - 1 - pass) % 2 == 0) ? out : b.val_a;
    hipLaunchKernelGGL(k_radix_hist, dim3(ntiles), dim3(kRadixThreads), 0, st, kin, n, shift,
                       ntiles, hist);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = launch_scan(hist, offs, nh, b.scan_tmp, b.scan_bytes, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_radix_scatter, dim3(ntiles), dim3(kRadixThreads), 0, st, kin, vin, n,
                       shift, ntiles, offs, kout, vout);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    kin = kout;
    vin = vout;
  }
  if (keys) *keys = const_cast<int*>(kin);
  return hipSuccess;
}

static GridDev grid_dev(const Grid& g) {
  GridDev gd;
  for (int a = 0; a < 3; ++a) {
    gd.nc[a] = g.nc[a];
    gd.inv_s[a] = g.inv_s[a];
    gd.lo[a] = g.lo[a];
    gd.L[a] = g.L[a];
  }
  gd.periodic = g.periodic;
  return gd;
}

hipError_t launch_cells_batch(const g3pcf_problem& p, const BatchCat* cats, int ncat,
                              const CellBufs& b, int* flags, int* plist, long long* head,
                              int fp64, hipStream_t st) {
  BatchGrids bg{};
  for (int c = 0; c < ncat; ++c) {
    bg.g[c] = grid_dev(cats[c].grid);
    bg.plan[c] = cats[c].plan;
    bg.first[c] = int(cats[c].first);
    bg.n[c] = int(cats[c].n);
    bg.ncell[c] = int(cats[c].grid.ncell);
    bg.cells_at[c] = int(cats[c].cells_at);
    bg.parts[c] = cats[c].parts;
  }
  SmallOut o{b.perm, b.wsort, b.cell_start, 0,      flags,
             plist,  head,    reinterpret_cast<int*>(head), 0, nullptr};
  auto go = [&](auto real, auto in) {
    using Real = decltype(real);
    using In = decltype(in);
    using V = typename Vec4<Real>::T;
    V* pos4 = static_cast<V*>(b.pos4);
    hipLaunchKernelGGL((k_cells_batch<Real, In>), dim3(unsigned(ncat)), dim3(kSmallThreads), 0,
                       st, static_cast<const In*>(p.pos), p.w, bg, p.primary_mask,
                       static_cast<V*>(b.stage4), pos4, pos4 + p.n, o);
  };
  if (fp64) {
    if (p.pos_dtype == G3PCF_F64) go(double(), double());
    else go(double(), float());
  } else {
    if (p.pos_dtype == G3PCF_F64) go(float(), double());
    else go(float(), float());
  }
  return hipGetLastError();
}

// Primary list (cell order): galaxies in the mask (NULL: all).  Leaves flags zero
// (see PairArgs::overflow).  Also forms the table of groups.
static hipError_t launch_primaries(const uint8_t* mask, int64_t n, const ShellPlan& sp,
                                   const CellBufs& b, int* flags, int* plist, long long* nprim,
                                   hipStream_t st) {
  const unsigned nb = blocks_for(n + 1, 256), table = sp.lists ? 1 : 0;
  if (!mask) {
    hipLaunchKernelGGL(k_primary_all, dim3(nb + table), dim3(256), 0, st, flags, n, plist, nprim,
                       sp, b.blocks, b.groups);
    return hipGetLastError();
  }
  // (the blocks' counts are read before the scan writes over them)
  hipLaunchKernelGGL(k_primary_flags, dim3(nb + table), dim3(256), 0, st, mask, b.perm, n, flags,
                     sp, b.blocks, b.groups);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // positions: exclusive scan into flags + (n + 1)
  int* pos = flags + (n + 1);
  if ((e = launch_scan(flags, pos, n + 1, b.scan_tmp, b.scan_bytes, st)) != hipSuccess)
    return e;
  hipLaunchKernelGGL(k_primary_list, dim3(nb), dim3(256), 0, st, flags, pos, n, plist, nprim);
  return hipGetLastError();
}

hipError_t launch_cells(const g3pcf_problem& p, const Grid& g, const ShellPlan& sp,
                        const CellBufs& b, const Primaries& pr, Clears z, int fp64,
                        hipStream_t st) {
  const int64_t n = p.n;
  const GridDev gd = grid_dev(g);
  // n <= kSmallN galaxies: one launch (the grid has at most 4 n cells)
  if (n > 0 && n <= kSmallN && g.ncell <= 4 * kSmallN) {
    SmallOut o{b.perm, b.wsort, b.cell_start, int(g.ncell), pr.flags, pr.plist, pr.nprim,
               pr.counters, pr.counter_words, b.groups};
    int64_t words = 0;
    for (int k = 0; k < z.count; ++k) words += z.words[k];
    const unsigned grid = 1u + unsigned(std::min<int64_t>(255, blocks_for(words, kSmallThreads * 4)));
    auto go = [&](auto real, auto in) {
      using Real = decltype(real);
      using In = decltype(in);
      using V = typename Vec4<Real>::T;
      hipLaunchKernelGGL((k_cells_small<Real, In>), dim3(grid), dim3(kSmallThreads), 0, st,
                         static_cast<const In*>(p.pos), p.w, int(n), gd, sp, pr.mask,
                         static_cast<V*>(b.stage4), static_cast<V*>(b.pos4), o, z);
    };
    if (fp64) {
      if (p.pos_dtype == G3PCF_F64) go(double(), double());
      else go(double(), float());
    } else {
      if (p.pos_dtype == G3PCF_F64) go(float(), double());
      else go(float(), float());
    }
    return hipGetLastError();
  }
  z.add(pr.counters, pr.counter_words);
  z.add(b.cell_count, g.ncell + 1);
  hipError_t e = launch_clears(z, st);
  if (e != hipSuccess) return e;
  const unsigned nb = blocks_for(n, 256);
  // staged values (input order) into stage4, the cell id of every galaxy
  // into key_a, and the cell counts
  if (fp64) {
    if (p.pos_dtype == G3PCF_F64)
      hipLaunchKernelGGL((k_assign<double, double>), dim3(nb), dim3(256), 0, st,
                         static_cast<const double*>(p.pos), p.w, n, gd,
                         static_cast<double4*>(b.stage4), b.key_a, b.cell_count);
    else
      hipLaunchKernelGGL((k_assign<double, float>), dim3(nb), dim3(256), 0, st,
                         static_cast<const float*>(p.pos), p.w, n, gd,
                         static_cast<double4*>(b.stage4), b.key_a, b.cell_count);
  } else {
    if (p.pos_dtype == G3PCF_F64)
      hipLaunchKernelGGL((k_assign<float, double>), dim3(nb), dim3(256), 0, st,
                         static_cast<const double*>(p.pos), p.w, n, gd,
                         static_cast<float4*>(b.stage4), b.key_a, b.cell_count);
    else
      hipLaunchKernelGGL((k_assign<float, float>), dim3(nb), dim3(256), 0, st,
                         static_cast<const float*>(p.pos), p.w, n, gd,
                         static_cast<float4*>(b.stage4), b.key_a, b.cell_count);
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // cell_start = exclusive scan of the counts (ncell + 1 entries, last = n)
  if ((e = launch_scan(b.cell_count, b.cell_start, g.ncell + 1, b.scan_tmp, b.scan_bytes, st)) !=
      hipSuccess)
    return e;
  // perm = input indices sorted stably by cell id
  if ((e = radix_sort(b, n, g.ncell, b.perm, nullptr, st)) != hipSuccess) return e;
  // the gather also writes the kSentinel NaN entries after the catalogue
  const unsigned ng = blocks_for(n + kSentinel, 256);
  if (fp64)
    hipLaunchKernelGGL((k_gather_sorted<double4>), dim3(ng), dim3(256), 0, st,
                       static_cast<const double4*>(b.stage4), b.perm, n, p.w,
                       static_cast<double4*>(b.pos4), b.wsort, sp, b.cell_start, b.blocks);
  else
    hipLaunchKernelGGL((k_gather_sorted<float4>), dim3(ng), dim3(256), 0, st,
                       static_cast<const float4*>(b.stage4), b.perm, n, p.w,
                       static_cast<float4*>(b.pos4), b.wsort, sp, b.cell_start, b.blocks);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (!pr.flags) {
    if (!sp.lists) return hipSuccess;
    hipLaunchKernelGGL(k_groups, dim3(1), dim3(256), 0, st, sp, b.blocks, b.groups);
    return hipGetLastError();
  }
  return launch_primaries(pr.mask, n, sp, b, pr.flags, pr.plist, pr.nprim, st);
}

hipError_t launch_region_primaries(const uint8_t* mask, const int32_t* region, int region0,
                                   int nregions, const CellBufs& b, int64_t n, int* flags,
                                   int* starts, int* plist, long long* nprim, hipStream_t st) {
  hipLaunchKernelGGL(k_region_keys, dim3(blocks_for(n + 1, 256)), dim3(256), 0, st, mask, region,
                     region0, nregions, b.perm, n, b.key_a, flags);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  int* keys = nullptr;
  if ((e = radix_sort(b, n, int64_t(nregions) + 1, plist, &keys, st)) != hipSuccess) return e;
  hipLaunchKernelGGL(k_region_starts, dim3(blocks_for(int64_t(nregions) + 1, 256)), dim3(256), 0,
                     st, keys, n, nregions, starts, nprim);
  return hipGetLastError();
}

}  // namespace g3
