// C ABI of libg3pcf: argument validation, workspace layout and the order of
// the stages on the caller's stream.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <utility>

#include <vector>

#include "internal.h"

struct g3pcf_trace {
  int capacity = 0;
  int count = 0;
  int dropped = 0;
  std::vector<hipEvent_t> ev;  // start, stop per record
  std::vector<int> stage;
};

namespace g3 {
namespace {

// Records a start event now and a stop event when the scope ends.
struct StageScope {
  g3pcf_trace* t;
  hipStream_t st;
  int slot = -1;
  StageScope(g3pcf_trace* tr, int stg, hipStream_t s) : t(tr), st(s) {
    if (!t) return;
    if (t->count < t->capacity) {
      slot = t->count++;
      t->stage[slot] = stg;
      (void)hipEventRecord(t->ev[2 * slot], st);
    } else {
      ++t->dropped;
    }
  }
  ~StageScope() {
    if (slot >= 0) (void)hipEventRecord(t->ev[2 * slot + 1], st);
  }
};

thread_local std::string t_err;

int fail(int code, const std::string& msg) {
  t_err = msg;
  return code;
}

int hip_fail(hipError_t e, const char* where) {
  return fail(G3PCF_EHIP, std::string(where) + ": " + hipGetErrorString(e));
}

constexpr size_t kAlign = 256;
constexpr size_t kCountersBytes = 1024;
size_t up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

struct Ws {
  size_t pos4, tmp4, cid, perm, tmp_perm, rkey, rhist, wsort, cell_start, cell_count, flags,
      plist, scan, counters, spill, A, C, gsort, gsort32, mht, hrows, degD, degP, degX;
  size_t scan_bytes;
  size_t total;
  int64_t blocks_at;  // see CellBufs::blocks
  int64_t PB;   // primaries per pair-block
  int spill_cap;  // spill-list entries per wave (0: none)
  int parts;    // partial Gram products of a pair-block
  int room;     // of several small catalogues' pair-blocks (batches), at least `parts`
  bool deg_fused;  // distinct: the pair kernel also collects the degenerate sums
  Grid grid;
  RowLayout lay;
};

// Workspace layout.  pb_max caps the primaries of a pair-block (the a_lm rows
// held at once); compact = true leaves out the spill lists (a multi-chunk basis
// then repeats its search per chunk) and keeps the Gram partials to four.
Ws plan(const g3pcf_problem& p, int backward, int64_t pb_max = kPairBlockMax,
        bool compact = false) {
  Ws w{};
  const int64_t n = p.n;
  const int fp64 = (p.pair_prec == G3PCF_PREC_FP64);
  const size_t rb = fp64 ? 32 : 16;
  w.grid = make_grid(p);
  w.lay = make_layout(p.lmax, p.nbins);
  const int64_t ncell = w.grid.ncell;
  w.PB = std::max<int64_t>(1, std::min<int64_t>(n, pb_max));
  const int64_t nhist = int64_t(radix_hist_ints(n));
  w.scan_bytes = scan_tmp_bytes(std::max<int64_t>(std::max<int64_t>(ncell + 1, n + 1), nhist));
  size_t at = 0;
  auto take = [&](size_t bytes) {
    const size_t o = at;
    at += up(std::max<size_t>(bytes, 1));
    return o;
  };
  w.pos4 = take(size_t(n + kSentinel) * rb);
  w.tmp4 = take(size_t(n) * rb);
  w.cid = take(size_t(n) * 4);
  w.perm = take(size_t(n) * 4);
  w.tmp_perm = take(size_t(n) * 4);
  w.rkey = take(size_t(n) * 4);
  // (also the heads of a batch's group of catalogues)
  w.rhist = take(std::max(size_t(2 * nhist) * 4, size_t(kBatchGroup) * kCatStride * 8));
  w.wsort = take(size_t(n) * 8);
  w.cell_start = take(size_t(ncell + 1) * 4);
  w.cell_count = take(size_t(ncell + 1) * 4);
  w.flags = take(size_t(2 * (n + 1)) * 4);
  w.blocks_at = n + 1;
  w.plist = take(size_t(n) * 4);
  w.scan = take(w.scan_bytes);
  w.counters = take(kCountersBytes);
  // per-wave spill lists for the basis accumulated in several register chunks
  const bool multi = !compact && p.basis == G3PCF_BASIS_CARTESIAN;
  w.spill = take(multi ? size_t(kPairWaves) * kSpillCap * 4 : 0);
  w.spill_cap = multi ? kSpillCap : 0;
  w.A = take(size_t(w.PB) * w.lay.W * 8);
  // the compact layout's pair-blocks are one block of kZetaBlock rows
  w.parts = compact ? 4 : zeta_parts(w.lay, w.PB);
  w.room = compact ? w.parts : zeta_room(w.lay, w.PB);
  w.C = take(size_t(w.room) * sum_wm2(w.lay) * 8);
  // degenerate triangles: per-shell Chebyshev sums and their per-workgroup partials
  const bool deg = !backward && p.distinct;
  w.degD = take(deg ? size_t(p.nbins) * (2 * p.lmax + 1) * 8 : 0);
  w.degP = take(deg ? deg_partial_doubles(w.PB, p.nbins, p.lmax) * 8 : 0);
  // the spin kernels collect the degenerate sums on the way, into rows of their
  // own; the cartesian kernels have no registers left for them, and the
  // compact layout no room: there a pass of its own writes over the a_lm rows
  w.deg_fused = deg && !compact && p.basis == G3PCF_BASIS_SPIN;
  if (w.deg_fused) w.degX = take(size_t(w.PB) * p.nbins * (2 * p.lmax + 1) * 8);
  if (backward) {
    w.gsort = take(size_t(n) * 8);
    w.gsort32 = take(fp64 ? 0 : size_t(n) * 4);  // FP32 secondary terms (FP32 pair path)
    w.mht = take(adj_matrix_doubles(w.lay) * 8);
    w.hrows = take(size_t(w.PB) * w.lay.W * 8);
  }
  w.total = at;
  return w;
}

bool finite3(const double* v) {
  return std::isfinite(v[0]) && std::isfinite(v[1]) && std::isfinite(v[2]);
}

int validate(const g3pcf_problem* p) {
  if (!p) return fail(G3PCF_EINVAL, "problem is NULL");
  // the pair kernels address the cell-ordered catalogue (16 or 32 bytes per
  // galaxy) with 32-bit byte offsets
  if (p->n < 0 || p->n >= (int64_t(1) << 27))
    return fail(G3PCF_EINVAL, "n must satisfy 0 <= n < 2^27");
  if (p->n > 0 && (!p->pos || !p->w)) return fail(G3PCF_EINVAL, "pos and w must be non-NULL");
  if (p->pos_dtype != G3PCF_F32 && p->pos_dtype != G3PCF_F64)
    return fail(G3PCF_EINVAL, "pos_dtype must be G3PCF_F32 or G3PCF_F64");
  if (!finite3(p->box) || !finite3(p->box_lo) || p->box[0] <= 0 || p->box[1] <= 0 ||
      p->box[2] <= 0)
    return fail(G3PCF_EINVAL, "box must be finite and positive, box_lo finite");
  if (!(p->rmax > 0) || !std::isfinite(p->rmax)) return fail(G3PCF_EINVAL, "rmax must be > 0");
  if (p->periodic) {
    const double mn = std::min(p->box[0], std::min(p->box[1], p->box[2]));
    if (p->rmax > 0.5 * mn)
      return fail(G3PCF_EINVAL, "periodic box needs rmax <= min(box) / 2");
  }
  if (p->nbins < 1 || p->nbins > kMaxBins) return fail(G3PCF_EINVAL, "nbins must be 1..32");
  if (p->lmax < 0 || p->lmax > kDeg) return fail(G3PCF_EINVAL, "lmax must be 0..10");
  if (p->los != G3PCF_LOS_Z && p->los != G3PCF_LOS_OBSERVER)
    return fail(G3PCF_EINVAL, "los must be G3PCF_LOS_Z or G3PCF_LOS_OBSERVER");
  if (p->los == G3PCF_LOS_OBSERVER && !finite3(p->observer))
    return fail(G3PCF_EINVAL, "observer must be finite");
  if (p->pair_prec != G3PCF_PREC_FP64 && p->pair_prec != G3PCF_PREC_FP32)
    return fail(G3PCF_EINVAL, "pair_prec must be G3PCF_PREC_FP64 or G3PCF_PREC_FP32");
  if (p->zeta_prec != G3PCF_PREC_FP64 && p->zeta_prec != G3PCF_PREC_FP32 &&
      p->zeta_prec != G3PCF_PREC_BF16X3)
    return fail(G3PCF_EINVAL, "zeta_prec must be FP64, FP32 or BF16X3");
  if (p->basis != G3PCF_BASIS_CARTESIAN && p->basis != G3PCF_BASIS_SPIN)
    return fail(G3PCF_EINVAL, "basis must be G3PCF_BASIS_CARTESIAN or G3PCF_BASIS_SPIN");
  if (p->distinct != 0 && p->distinct != 1)
    return fail(G3PCF_EINVAL, "distinct must be 0 or 1");
  if (p->accumulate != 0 && p->accumulate != 1)
    return fail(G3PCF_EINVAL, "accumulate must be 0 or 1");
  return G3PCF_OK;
}

std::mutex g_tab_mu;
std::set<std::pair<int, int>> g_tab_done;

// Uploads a table to the current device once: G3PCF_BASIS_CARTESIAN, _SPIN (the
// spin-Chebyshev tables) or kBasisDeg.
int ensure_tables(int basis) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  std::lock_guard<std::mutex> lk(g_tab_mu);
  if (g_tab_done.count({dev, basis})) return G3PCF_OK;
  e = (basis == kBasisDeg)          ? upload_deg_table()
      : (basis == G3PCF_BASIS_SPIN) ? upload_spin_tables()
                                    : upload_cart_tables();
  if (e != hipSuccess) return hip_fail(e, "table upload");
  g_tab_done.insert({dev, basis});
  return G3PCF_OK;
}

template <typename T>
T* at(void* ws, size_t off) {
  return reinterpret_cast<T*>(static_cast<char*>(ws) + off);
}

// Counts of one XCD's waves, on a 64-byte line of their own.
struct XcdCounters {
  int queue[kQueueKinds];        // next item: of the forward, of the adjoint
  unsigned long long pairs;      // accepted pairs
  unsigned long long pairs_adj;
  unsigned long long pad[3];
};
static_assert(sizeof(XcdCounters) == kQueueStride * 4, "one line each");

struct Counters {
  long long nprim;
  unsigned long long inputs_hash;  // backward: fingerprint of its inputs (a_lm store check)
  long long first;                 // first row among its group's (catalogues of a batch)
  long long parts;                 // and its Gram blocks
  GroupTable groups;
  int pad[4];
  XcdCounters xcd[kQueues];
};
static_assert(sizeof(Counters) == kCatStride * 8 && offsetof(Counters, first) == kCatFirst * 8 &&
                  offsetof(Counters, parts) == kCatParts * 8 &&
                  offsetof(Counters, groups) == kCatGroups * 8 &&
                  offsetof(Counters, xcd) % 64 == 0,
              "head of a catalogue of a group");
static_assert(sizeof(Counters) <= kCountersBytes, "counters block");

CellBufs cell_bufs(const Ws& w, void* ws) {
  CellBufs b{};
  b.pos4 = at<void>(ws, w.pos4);
  b.stage4 = at<void>(ws, w.tmp4);
  b.cell_start = at<int>(ws, w.cell_start);
  b.cell_count = at<int>(ws, w.cell_count);
  b.key_a = at<int>(ws, w.cid);
  b.key_b = at<int>(ws, w.rkey);
  b.val_a = at<int>(ws, w.tmp_perm);
  b.perm = at<int>(ws, w.perm);
  b.hist = at<int>(ws, w.rhist);
  b.wsort = at<double>(ws, w.wsort);
  // (the second half of the flags is free until the primary list)
  b.blocks = at<int>(ws, w.flags) + w.blocks_at;
  b.groups = &at<Counters>(ws, w.counters)->groups;
  b.scan_tmp = at<void>(ws, w.scan);
  b.scan_bytes = w.scan_bytes;
  return b;
}

// Stages shared by forward and backward: cell list and primary list, and the
// pass's clears z (n > 0).  primaries = false: the list is left to the caller.
int stage_catalogue(const g3pcf_problem& p, const Ws& w, void* ws, const Clears& z,
                    hipStream_t st, bool primaries = true) {
  const int fp64 = (p.pair_prec == G3PCF_PREC_FP64);
  const CellBufs b = cell_bufs(w, ws);
  Counters* c = at<Counters>(ws, w.counters);
  Primaries pr{p.primary_mask, primaries ? at<int>(ws, w.flags) : nullptr, at<int>(ws, w.plist),
               &c->nprim, reinterpret_cast<int*>(c), int(sizeof(Counters) / 4)};
  const hipError_t e = launch_cells(p, w.grid, shell_plan(p, w.grid), b, pr, z, fp64, st);
  if (e != hipSuccess) return hip_fail(e, "cell list");
  return G3PCF_OK;
}

int pair_args(const g3pcf_problem& p, const Ws& w, void* ws, PairArgs& a) {
  const hipError_t e =
      table_addresses(p.pair_prec == G3PCF_PREC_FP64, &a.cart, &a.spin);
  if (e != hipSuccess) return hip_fail(e, "table address");
  Counters* c = at<Counters>(ws, w.counters);
  a.pos4 = at<void>(ws, w.pos4);
  a.sentinel = int(p.n);
  a.cell_start = at<int>(ws, w.cell_start);
  a.plist = at<int>(ws, w.plist);
  a.nprim = &c->nprim;
  a.overflow = at<unsigned>(ws, w.flags);
  a.spill = at<int>(ws, w.spill);
  a.spill_cap = w.spill_cap;
  a.queue = c->xcd[0].queue;
  for (int k = 0; k < 3; ++k) {
    a.nc[k] = w.grid.nc[k];
    a.s[k] = w.grid.s[k];
    a.inv_s[k] = w.grid.inv_s[k];
    a.lo[k] = w.grid.lo[k];
    a.L[k] = w.grid.L[k];
    a.inv_L[k] = 1.0 / w.grid.L[k];
    a.tight[k] = w.grid.tight[k];
    a.obs[k] = p.observer[k];
  }
  a.periodic = w.grid.periodic;
  a.rmax = p.rmax;
  a.rmax_search = w.grid.rsearch;
  // squared shell edges rounded to float; the lower bound is exclusive, so it
  // is the float just below the edge (0 for the innermost shell, r > 0)
  for (int b = 0; b < p.nbins; ++b) {
    const double e0 = b * p.rmax / p.nbins, e1 = (b + 1) * p.rmax / p.nbins;
    const float t0 = float(e0 * e0);
    a.r2_lo[b] = (b == 0) ? 0.0f : std::nextafter(t0, 0.0f);
    a.r2_hi[b] = (b + 1 == p.nbins) ? float(p.rmax * p.rmax) : float(e1 * e1);
  }
  const ShellPlan sp = shell_plan(p, w.grid);
  a.lists = sp.lists;
  a.groups = &c->groups;
  a.list_mean = sp.most;
  a.nbins = p.nbins;
  a.lmax = p.lmax;
  a.los = p.los;
  a.A = at<double>(ws, w.A);
  a.lay = w.lay;
  a.perm = at<int>(ws, w.perm);
  a.wsort = at<double>(ws, w.wsort);
  a.deg = at<double>(ws, w.degX);
  return G3PCF_OK;
}

int check_workspace(const Ws& w, void* ws, size_t ws_bytes) {
  if (!ws || ws_bytes < w.total)
    return fail(G3PCF_EWORKSPACE, "workspace needs " + std::to_string(w.total) + " bytes");
  if (reinterpret_cast<uintptr_t>(ws) % kAlign)
    return fail(G3PCF_EWORKSPACE, "workspace must be 256-byte aligned");
  return G3PCF_OK;
}

// The a_lm store: a 256-byte header (the fingerprint of the forward pass's
// inputs) and then one row of W doubles per primary in primary-list order.
constexpr size_t kAlmHeader = 256;

size_t alm_total(const g3pcf_problem& p, const RowLayout& lay) {
  return kAlmHeader + size_t(p.n) * size_t(lay.W) * 8;
}

int check_alm(const g3pcf_problem& p, const Ws& w) {
  if (!p.alm) return G3PCF_OK;
  const size_t need = alm_total(p, w.lay);
  if (p.alm_bytes < need)
    return fail(G3PCF_EWORKSPACE, "alm store needs " + std::to_string(need) + " bytes");
  if (reinterpret_cast<uintptr_t>(p.alm) % kAlign)
    return fail(G3PCF_EWORKSPACE, "alm store must be 256-byte aligned");
  return G3PCF_OK;
}

double* alm_rows(const g3pcf_problem& p) {
  return reinterpret_cast<double*>(static_cast<char*>(p.alm) + kAlmHeader);
}

// splitmix64 output function (Steele, Lea and Flood, OOPSLA 2014), host side
uint64_t hmix(uint64_t x) {
  x ^= x >> 30;
  x *= 0xbf58476d1ce4e5b9ull;
  x ^= x >> 27;
  x *= 0x94d049bb133111ebull;
  return x ^ (x >> 31);
}

// Hash of the settings that change the a_lm rows (zeta_prec, accumulate and
// the output pointers do not).
uint64_t settings_seed(const g3pcf_problem& p) {
  uint64_t h = hmix(0x6733706366ull + uint64_t(p.n));
  auto put_d = [&](double v) {
    uint64_t b;
    std::memcpy(&b, &v, 8);
    h = hmix(h ^ b);
  };
  auto put_i = [&](int64_t v) { h = hmix(h ^ uint64_t(v)); };
  for (int k = 0; k < 3; ++k) {
    put_d(p.box[k]);
    put_d(p.box_lo[k]);
    put_d(p.los == G3PCF_LOS_OBSERVER ? p.observer[k] : 0.0);
  }
  put_d(p.rmax);
  put_i(p.periodic);
  put_i(p.nbins);
  put_i(p.lmax);
  put_i(p.los);
  put_i(p.pair_prec);
  put_i(p.basis);
  put_i(p.pos_dtype);
  return h;
}

hipError_t fingerprint(const g3pcf_problem& p, const Ws& w, void* ws, unsigned long long* out,
                       hipStream_t st) {
  hipError_t e = launch_fill_int(reinterpret_cast<int*>(out), 2, 0, st);
  if (e != hipSuccess) return e;
  Counters* c = at<Counters>(ws, w.counters);
  return launch_fingerprint(at<void>(ws, w.pos4), p.pair_prec == G3PCF_PREC_FP64,
                            at<double>(ws, w.wsort), at<int>(ws, w.perm), at<int>(ws, w.plist),
                            &c->nprim, p.n, settings_seed(p), out, st);
}

int forward_tables(const g3pcf_problem& p) {
  int rc = ensure_tables(p.basis);
  if (!rc && p.distinct) rc = ensure_tables(kBasisDeg);
  return rc;
}

// List parts of `n` that one launch of the Gram products takes: so many that each
// has four blocks of partials on average (27 regions of 3700 primaries: 1.84 ms of
// Gram products and their sums in one launch each, 0.74 in five).
int lists_at_once(const Ws& w, int n) {
  const int most = std::max(1, std::min(kZetaLists, w.parts / 4));
  const int launches = (n + most - 1) / most;
  return (n + launches - 1) / launches;
}

// The pair-blocks of the current primary list (at most `cover` primaries):
// pair kernel, Gram products into zeta, and (distinct) the degenerate-triangle
// pass and its correction.  rows: where the a_lm rows go (NULL: the
// workspace's pair-block rows; else rows of every primary, kept).  starts: NULL,
// or the parts of the list (device, nparts + 1 of them, see
// launch_region_primaries), each reduced into a zeta of its own.
int forward_pairs(const g3pcf_problem& p, const Ws& w, void* ws, double* zeta, int64_t cover,
                  double* rows, const int* starts, int nparts, hipStream_t st) {
  hipError_t e;
  PairArgs a{};
  if (int rc = pair_args(p, w, ws, a)) return rc;
  const int fp64 = (p.pair_prec == G3PCF_PREC_FP64);
  Counters* c = at<Counters>(ws, w.counters);
  double* degD = at<double>(ws, w.degD);
  const size_t zlen = g3pcf_zeta_len(p.lmax, p.nbins);
  for (int64_t b0 = 0; b0 < cover; b0 += w.PB) {
    a.p_begin = b0;
    a.p_count = std::min<int64_t>(w.PB, cover - b0);
    a.pairs = p.pairs_out ? &c->xcd[0].pairs : nullptr;
    if (rows) a.A = rows + size_t(b0) * w.lay.W;
    {
      StageScope sc(p.trace, G3PCF_STAGE_PAIRS, st);
      if ((e = launch_pair_forward(a, fp64, p.basis, w.deg_fused, st)) != hipSuccess)
        return hip_fail(e, "pair kernel");
    }
    {
      StageScope scz(p.trace, G3PCF_STAGE_ZETA, st);
      ZetaArgs z{};
      z.A = a.A;
      z.wsort = a.wsort;
      z.plist = a.plist;
      z.nprim = &c->nprim;
      z.row_begin = b0;
      z.K = a.p_count;
      z.lay = w.lay;
      z.C64 = at<double>(ws, w.C);
      z.parts = w.parts;
      z.prec = p.zeta_prec;
      z.queue = a.queue;
      const int lists = lists_at_once(w, nparts);
      for (int r = 0; r < nparts; r += lists) {
        z.range = starts ? starts + r : nullptr;
        z.lists = std::min(lists, nparts - r);
        z.zeta = zeta + zlen * size_t(r);
        if ((e = launch_zeta_pairblock(z, st)) != hipSuccess) return hip_fail(e, "zeta");
      }
    }
    if (p.distinct) {
      // the sums w_j^2 T_n(u_z) of each primary, summed with w_i; without rows
      // of their own the same pairs again, written over the pair-block's A rows
      // (already reduced into zeta)
      StageScope scd(p.trace, G3PCF_STAGE_DISTINCT, st);
      a.pairs = nullptr;  // counted already
      if (!w.deg_fused && (e = launch_pair_distinct(a, fp64, st)) != hipSuccess)
        return hip_fail(e, "degenerate-triangle pass");
      const double* X = w.deg_fused ? a.deg : a.A;
      const int rowW = w.deg_fused ? p.nbins * (2 * p.lmax + 1) : w.lay.W;
      for (int r = 0; r < nparts; ++r) {
        if ((e = launch_fill_double(degD, int64_t(p.nbins) * (2 * p.lmax + 1), 0.0, st)) !=
            hipSuccess)
          return hip_fail(e, "degenerate sums clear");
        if ((e = launch_deg_reduce(X, rowW, p.nbins, p.lmax, a.wsort, a.plist, &c->nprim,
                                   starts ? starts + r : nullptr, b0, a.p_count,
                                   at<double>(ws, w.degP), degD, a.queue, st)) != hipSuccess)
          return hip_fail(e, "degenerate-triangle sums");
        if ((e = launch_deg_apply(degD, p.lmax, p.nbins, zeta + zlen * size_t(r), st)) !=
            hipSuccess)
          return hip_fail(e, "degenerate-triangle correction");
      }
    }
  }
  return G3PCF_OK;
}

// The problem of one catalogue of a batch.
g3pcf_problem catalogue_of(const g3pcf_problem& p, int64_t first, int64_t n) {
  g3pcf_problem q = p;
  q.n = n;
  q.pos = static_cast<const char*>(p.pos) + size_t(first) * (p.pos_dtype == G3PCF_F32 ? 12 : 24);
  q.w = p.w + first;
  q.primary_mask = p.primary_mask ? p.primary_mask + first : nullptr;
  return q;
}

// How many catalogues from c on go through forward_group together (in cats; 0 or
// 1: not in a group): small ones, whose rows and cell starts the workspace of the
// whole call holds beside each other.  Not where the counts are asked for
// (a wait per catalogue) or the degenerate triangles are taken out.
int batch_group(const g3pcf_problem& p, const Ws& w, const int64_t* offsets, int ncat, int c,
                BatchCat* cats) {
  if (p.pairs_out || p.distinct) return 0;
  const int64_t cells = int64_t(w.cell_count - w.cell_start) / 4 + w.grid.ncell + 1;
  const int most = std::min(kBatchGroup, ncat - c);
  int m = 0;
  int64_t at = 0;
  for (; m < most; ++m) {
    BatchCat& k = cats[m];
    k.first = offsets[c + m];
    k.n = offsets[c + m + 1] - k.first;
    k.cells_at = at;
    k.parts = std::max(1, zeta_parts(w.lay, k.n));
    if (k.n > kBatchN || k.first + k.n - cats[0].first > w.PB) break;
    const g3pcf_problem q = catalogue_of(p, k.first, k.n);
    k.grid = make_grid(q);
    k.plan = shell_plan(q, k.grid);
    at += k.grid.ncell + 1;
    if (k.grid.ncell > 4 * kBatchN || at > cells) break;
  }
  return m;
}

// zeta of a group of a batch's catalogues: one launch of the cell stage, their pair
// kernels, and one of the Gram products.  w: the plan of the whole call, whose
// per-galaxy buffers the catalogues share out as the galaxies lie.
int forward_group(const g3pcf_problem& p, const Ws& w, void* ws, const BatchCat* cats, int m,
                  double* zeta, hipStream_t st) {
  const int fp64 = (p.pair_prec == G3PCF_PREC_FP64);
  const int64_t base = cats[0].first, rows = cats[m - 1].first + cats[m - 1].n - base;
  if (rows == 0) return G3PCF_OK;
  hipError_t e;
  Counters* head = at<Counters>(ws, w.rhist);
  int* plist = at<int>(ws, w.plist);
  {
    StageScope sc(p.trace, G3PCF_STAGE_CELLS, st);
    if ((e = launch_cells_batch(p, cats, m, cell_bufs(w, ws), at<int>(ws, w.flags), plist,
                                &head->nprim, fp64, st)) != hipSuccess)
      return hip_fail(e, "cell lists of a batch");
  }
  for (int c = 0; c < m; ++c) {
    const BatchCat& k = cats[c];
    if (k.n == 0) continue;
    Ws v = w;
    v.grid = k.grid;
    v.pos4 += size_t(k.first) * (fp64 ? 32 : 16);
    v.cell_start += size_t(k.cells_at) * 4;
    v.perm += size_t(k.first) * 4;
    v.plist += size_t(k.first) * 4;
    v.flags += size_t(k.first) * 4;
    v.wsort += size_t(k.first) * 8;
    v.A += size_t(k.first - base) * w.lay.W * 8;
    v.counters = w.rhist + size_t(c) * sizeof(Counters);
    StageScope sc(p.trace, G3PCF_STAGE_PAIRS, st);
    PairArgs a{};
    if (int rc = pair_args(catalogue_of(p, k.first, k.n), v, ws, a)) return rc;
    a.sentinel = int(p.n - k.first);
    a.p_begin = 0;
    a.p_count = k.n;
    a.pairs = nullptr;
    if ((e = launch_pair_forward(a, fp64, p.basis, false, st)) != hipSuccess)
      return hip_fail(e, "pair kernel");
  }
  StageScope sc(p.trace, G3PCF_STAGE_ZETA, st);
  ZetaArgs z{};
  z.A = at<double>(ws, w.A);
  z.wsort = at<double>(ws, w.wsort) + base;
  z.plist = plist + base;
  z.row_begin = 0;
  z.lay = w.lay;
  z.C64 = at<double>(ws, w.C);
  z.prec = p.zeta_prec;
  z.queue = head->xcd[0].queue;
  const size_t zlen = g3pcf_zeta_len(p.lmax, p.nbins);
  // every catalogue in the blocks that a call of its own would cut it into, so that
  // its sums are the same bits; as many catalogues a launch as there is room for
  for (int c = 0; c < m; c += z.lists) {
    z.lists = z.parts = 0;
    while (z.lists < std::min(kZetaLists, m - c) &&
           (z.lists == 0 || z.parts + cats[c + z.lists].parts <= w.room))
      z.parts += cats[c + z.lists++].parts;
    z.cats = &head[c].nprim;
    z.zeta = zeta + zlen * size_t(c);
    z.K = cats[c + z.lists - 1].first + cats[c + z.lists - 1].n - cats[c].first;
    if ((e = launch_zeta_pairblock(z, st)) != hipSuccess) return hip_fail(e, "zeta");
  }
  return G3PCF_OK;
}

// pairs_out from the forward count (or, adj = true, the adjoint pass's count)
int finish_pairs(const g3pcf_problem& p, const Ws& w, void* ws, hipStream_t st,
                 bool adj = false) {
  if (!p.pairs_out) return G3PCF_OK;
  XcdCounters host[kQueues];
  Counters* c = at<Counters>(ws, w.counters);
  hipError_t e = hipMemcpyAsync(host, c->xcd, sizeof(host), hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e != hipSuccess) return hip_fail(e, "pair count read-back");
  int64_t sum = 0;
  for (const XcdCounters& x : host) sum += int64_t(adj ? x.pairs_adj : x.pairs);
  *p.pairs_out = sum;
  return G3PCF_OK;
}

// The forward pass in a workspace laid out by `w` (already checked).
int forward_run(const g3pcf_problem& p, const Ws& w, double* zeta, void* ws, hipStream_t st) {
  int rc;
  if (p.alm && p.distinct)
    return fail(G3PCF_EINVAL, "alm store with distinct = 1 (the adjoint does not cover it)");
  if ((rc = check_alm(p, w))) return rc;
  if ((rc = forward_tables(p))) return rc;
  const size_t zlen = g3pcf_zeta_len(p.lmax, p.nbins);
  hipError_t e;
  Clears z;
  if (!p.accumulate) z.add(zeta, int64_t(zlen) * 2);
  if (p.n == 0) {
    if ((e = launch_clears(z, st)) != hipSuccess) return hip_fail(e, "zeta clear");
    if (p.alm && (e = launch_fill_int(static_cast<int*>(p.alm), 2, 0, st)) != hipSuccess)
      return hip_fail(e, "alm store header");
    if (p.pairs_out) *p.pairs_out = 0;
    return G3PCF_OK;
  }
  {
    StageScope sc(p.trace, G3PCF_STAGE_CELLS, st);
    if ((rc = stage_catalogue(p, w, ws, z, st))) return rc;
    if (p.alm && (e = fingerprint(p, w, ws, static_cast<unsigned long long*>(p.alm), st)) !=
                     hipSuccess)
      return hip_fail(e, "alm store fingerprint");
  }
  if ((rc = forward_pairs(p, w, ws, zeta, p.n, p.alm ? alm_rows(p) : nullptr, nullptr, 1, st)))
    return rc;
  return finish_pairs(p, w, ws, st);
}


// Scratch of the allocation-free entry point g3pcf_forward_noalloc: one
// array per device, held until the process ends.  In host code the array's
// name is a stand-in only; its device address comes from
// hipGetSymbolAddress, taken once per device with that device current.
constexpr size_t kScratchBytes = size_t(128) << 20;
// Primaries per pair-block in the scratch (one zeta block of 4096 rows).
constexpr int64_t kScratchPairBlock = kZetaBlock;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

std::mutex g_scratch_mu;
std::map<int, void*> g_scratch_ptr;

int scratch_address(void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  auto it = g_scratch_ptr.find(dev);
  if (it == g_scratch_ptr.end()) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
    if (!ptr || reinterpret_cast<uintptr_t>(ptr) % kAlign)
      return fail(G3PCF_EHIP, "scratch array has no usable device address");
    it = g_scratch_ptr.emplace(dev, ptr).first;
  }
  *out = it->second;
  return G3PCF_OK;
}

}  // namespace
}  // namespace g3

using namespace g3;

extern "C" {

size_t g3pcf_zeta_len(int lmax, int nbins) {
  if (lmax < 0 || nbins < 1) return 0;
  const size_t L1 = size_t(lmax) + 1;
  return L1 * L1 * L1 * size_t(nbins) * size_t(nbins) * 2;
}

int g3pcf_num_terms(int basis) {
  if (basis == G3PCF_BASIS_CARTESIAN) return kTermsCart;
  if (basis == G3PCF_BASIS_SPIN) return kTermsSpin;
  return -1;
}

const char* g3pcf_last_error(void) { return t_err.c_str(); }

g3pcf_trace* g3pcf_trace_create(int capacity) {
  if (capacity < 1) {
    fail(G3PCF_EINVAL, "trace capacity must be >= 1");
    return nullptr;
  }
  g3pcf_trace* t = new g3pcf_trace;
  t->capacity = capacity;
  t->ev.assign(2 * size_t(capacity), nullptr);
  t->stage.assign(size_t(capacity), -1);
  for (auto& e : t->ev) {
    if (hipEventCreate(&e) != hipSuccess) {
      e = nullptr;
      g3pcf_trace_destroy(t);
      fail(G3PCF_EHIP, "hipEventCreate failed");
      return nullptr;
    }
  }
  return t;
}

void g3pcf_trace_reset(g3pcf_trace* t) {
  if (!t) return;
  t->count = 0;
  t->dropped = 0;
}

int g3pcf_trace_read(g3pcf_trace* t, int* stage, float* ms, int max, int* dropped) {
  if (!t || !stage || !ms || max < 0) return fail(G3PCF_EINVAL, "NULL trace or output");
  const int n = std::min(max, t->count);
  for (int k = 0; k < n; ++k) {
    float v = 0.f;
    hipError_t e = hipEventElapsedTime(&v, t->ev[2 * k], t->ev[2 * k + 1]);
    if (e != hipSuccess) return hip_fail(e, "hipEventElapsedTime");
    stage[k] = t->stage[k];
    ms[k] = v;
  }
  if (dropped) *dropped = t->dropped;
  return n;
}

void g3pcf_trace_destroy(g3pcf_trace* t) {
  if (!t) return;
  for (auto& e : t->ev)
    if (e) (void)hipEventDestroy(e);
  delete t;
}

int g3pcf_workspace_bytes(const g3pcf_problem* prob, int backward, size_t* bytes) {
  int rc = validate(prob);
  if (rc) return rc;
  if (!bytes) return fail(G3PCF_EINVAL, "bytes is NULL");
  if (backward != 0 && backward != 1) return fail(G3PCF_EINVAL, "backward must be 0 or 1");
  *bytes = plan(*prob, backward).total;
  return G3PCF_OK;
}

int g3pcf_alm_bytes(const g3pcf_problem* prob, size_t* bytes) {
  int rc = validate(prob);
  if (rc) return rc;
  if (!bytes) return fail(G3PCF_EINVAL, "bytes is NULL");
  *bytes = alm_total(*prob, make_layout(prob->lmax, prob->nbins));
  return G3PCF_OK;
}

int g3pcf_forward(const g3pcf_problem* prob, double* zeta, void* ws, size_t ws_bytes,
                  void* stream) {
  int rc = validate(prob);
  if (rc) return rc;
  if (!zeta) return fail(G3PCF_EINVAL, "zeta is NULL");
  const Ws w = plan(*prob, 0);
  if ((rc = check_workspace(w, ws, ws_bytes))) return rc;
  return forward_run(*prob, w, zeta, ws, static_cast<hipStream_t>(stream));
}

int g3pcf_forward_noalloc(const g3pcf_problem* prob, double* zeta, void* stream) {
  int rc = validate(prob);
  if (rc) return rc;
  if (!zeta) return fail(G3PCF_EINVAL, "zeta is NULL");
  const Ws w = plan(*prob, 0, kScratchPairBlock, true);
  if (w.total > kScratchBytes)
    return fail(G3PCF_EINVAL, "g3pcf_forward_noalloc: this problem needs " +
                                  std::to_string(w.total) + " bytes of scratch, the library "
                                  "holds " + std::to_string(kScratchBytes) +
                                  " (use g3pcf_forward with a workspace)");
  void* ws = nullptr;
  if ((rc = scratch_address(&ws))) return rc;
  return forward_run(*prob, w, zeta, ws, static_cast<hipStream_t>(stream));
}


int g3pcf_forward_regions(const g3pcf_problem* prob, const int32_t* region, int nregions,
                          double* zeta, void* ws, size_t ws_bytes, void* stream) {
  int rc = validate(prob);
  if (rc) return rc;
  if (nregions < 1 || nregions > (1 << 20)) return fail(G3PCF_EINVAL, "nregions must be 1..2^20");
  if (!zeta) return fail(G3PCF_EINVAL, "zeta is NULL");
  if (!region && prob->n > 0) return fail(G3PCF_EINVAL, "region is NULL");
  if (prob->alm) return fail(G3PCF_EINVAL, "alm store is not kept per region (set it to NULL)");
  const g3pcf_problem& p = *prob;
  const Ws w = plan(p, 0);
  if ((rc = check_workspace(w, ws, ws_bytes))) return rc;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if ((rc = forward_tables(p))) return rc;
  const size_t zlen = g3pcf_zeta_len(p.lmax, p.nbins);
  hipError_t e;
  Clears z;
  if (!p.accumulate) z.add(zeta, int64_t(zlen) * nregions * 2);
  if (p.n == 0) {
    if ((e = launch_clears(z, st)) != hipSuccess) return hip_fail(e, "zeta clear");
    if (p.pairs_out) *p.pairs_out = 0;
    return G3PCF_OK;
  }
  {
    StageScope sc(p.trace, G3PCF_STAGE_CELLS, st);
    if ((rc = stage_catalogue(p, w, ws, z, st, false))) return rc;
  }
  // One cell list and, region after region in one primary list, one pass of the
  // pair kernel; then the Gram products of up to kZetaLists regions in a launch.  (As
  // many regions at a time as there are galaxies: their starts share the scan's
  // space.)  27 regions of 3700 primaries as passes of their own took 8.0 ms, of
  // which 4.9 in pair kernels and 1.4 in waits for each region's count; now 4.5, of which
  // 3.9 in the pair kernel and 0.74 in Gram products and their sums (1.84 with a launch
  // per region).
  Counters* c = at<Counters>(ws, w.counters);
  int* flags = at<int>(ws, w.flags);
  int* starts = flags + (p.n + 1);
  for (int r0 = 0; r0 < nregions;) {
    const int m = int(std::min<int64_t>(nregions - r0, p.n));
    {
      StageScope sc(p.trace, G3PCF_STAGE_CELLS, st);
      if ((e = launch_region_primaries(p.primary_mask, region, r0, m, cell_bufs(w, ws), p.n, flags,
                                       starts, at<int>(ws, w.plist), &c->nprim, st)) != hipSuccess)
        return hip_fail(e, "region primary list");
    }
    if ((rc = forward_pairs(p, w, ws, zeta + zlen * size_t(r0), p.n, nullptr, starts, m, st)))
      return rc;
    r0 += m;
  }
  return finish_pairs(p, w, ws, st);
}

int g3pcf_forward_batch(const g3pcf_problem* prob, int ncat, const int64_t* offsets,
                        double* zeta, void* ws, size_t ws_bytes, void* stream) {
  int rc = validate(prob);
  if (rc) return rc;
  if (ncat < 1 || ncat > (1 << 20)) return fail(G3PCF_EINVAL, "ncat must be 1..2^20");
  if (!offsets || !zeta) return fail(G3PCF_EINVAL, "offsets and zeta must be non-NULL");
  if (offsets[0] != 0 || offsets[ncat] != prob->n)
    return fail(G3PCF_EINVAL, "offsets must start at 0 and end at n");
  for (int c = 0; c < ncat; ++c)
    if (offsets[c + 1] < offsets[c]) return fail(G3PCF_EINVAL, "offsets must not decrease");
  if (prob->alm) return fail(G3PCF_EINVAL, "alm store is not kept per catalogue (set it to NULL)");
  const g3pcf_problem& p = *prob;
  const Ws all = plan(p, 0);
  if ((rc = check_workspace(all, ws, ws_bytes))) return rc;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if ((rc = forward_tables(p))) return rc;
  const size_t zlen = g3pcf_zeta_len(p.lmax, p.nbins);
  hipError_t e;
  if (!p.accumulate &&
      (e = launch_fill_double(zeta, int64_t(zlen) * ncat, 0.0, st)) != hipSuccess)
    return hip_fail(e, "zeta clear");
  int64_t total = 0;
  // one group or catalogue after another in the same workspace, in stream order
  // (no host synchronisation unless pairs_out asks for the counts)
  for (int c = 0; c < ncat; ++c) {
    BatchCat cats[kBatchGroup];
    const int m = batch_group(p, all, offsets, ncat, c, cats);
    if (m > 1) {
      if ((rc = forward_group(p, all, ws, cats, m, zeta + zlen * size_t(c), st))) return rc;
      c += m - 1;
      continue;
    }
    g3pcf_problem q = catalogue_of(p, offsets[c], offsets[c + 1] - offsets[c]);
    if (q.n == 0) continue;
    int64_t pairs_c = 0;
    q.pairs_out = p.pairs_out ? &pairs_c : nullptr;
    const Ws w = plan(q, 0);
    if ((rc = check_workspace(w, ws, ws_bytes))) return rc;
    {
      StageScope sc(p.trace, G3PCF_STAGE_CELLS, st);
      if ((rc = stage_catalogue(q, w, ws, Clears(), st))) return rc;
    }
    if ((rc = forward_pairs(q, w, ws, zeta + zlen * size_t(c), q.n, nullptr, nullptr, 1, st)))
      return rc;
    if ((rc = finish_pairs(q, w, ws, st))) return rc;
    total += pairs_c;
  }
  if (p.pairs_out) *p.pairs_out = total;
  return G3PCF_OK;
}

int g3pcf_backward(const g3pcf_problem* prob, const double* grad_zeta, double* grad_w, void* ws,
                   size_t ws_bytes, void* stream) {
  int rc = validate(prob);
  if (rc) return rc;
  if (!grad_zeta || (!grad_w && prob->n > 0))
    return fail(G3PCF_EINVAL, "grad_zeta and grad_w must be non-NULL");
  if (prob->distinct)
    return fail(G3PCF_EUNSUPPORTED, "the adjoint does not cover distinct = 1");
  const g3pcf_problem& p = *prob;
  const Ws w = plan(p, 1);
  if ((rc = check_workspace(w, ws, ws_bytes))) return rc;
  if ((rc = check_alm(p, w))) return rc;
  hipStream_t st = static_cast<hipStream_t>(stream);
  // the adjoint (either basis) evaluates its per-pair polynomial in
  // (x - i y)^m T_n(z), coefficients from the spin-Chebyshev table
  if ((rc = ensure_tables(p.basis)) || (rc = ensure_tables(G3PCF_BASIS_SPIN))) return rc;
  if (p.n == 0) {
    if (p.pairs_out) *p.pairs_out = 0;
    return G3PCF_OK;
  }
  hipError_t e;
  Counters* c = at<Counters>(ws, w.counters);
  double* gsort = at<double>(ws, w.gsort);
  // FP32 pair path: the secondary terms are summed in FP32 on their own array
  float* gsort32 = (p.pair_prec == G3PCF_PREC_FP64) ? nullptr : at<float>(ws, w.gsort32);
  {
    StageScope sc(p.trace, G3PCF_STAGE_CELLS, st);
    Clears z;
    z.add(gsort, 2 * p.n);
    if (gsort32) z.add(gsort32, p.n);
    if ((rc = stage_catalogue(p, w, ws, z, st))) return rc;
    if (p.alm && (e = fingerprint(p, w, ws, &c->inputs_hash, st)) != hipSuccess)
      return hip_fail(e, "input fingerprint");
  }
  {
    StageScope sc(p.trace, G3PCF_STAGE_ADJ_COEF, st);
    if ((e = launch_adj_matrix(grad_zeta, w.lay, at<double>(ws, w.mht), st)) != hipSuccess)
      return hip_fail(e, "adjoint matrices");
  }
  PairArgs a{};
  if ((rc = pair_args(p, w, ws, a))) return rc;
  const int fp64 = (p.pair_prec == G3PCF_PREC_FP64);
  a.H = at<double>(ws, w.hrows);
  a.grad_w = gsort;
  a.grad_w32 = gsort32;
  for (int64_t b0 = 0; b0 < p.n; b0 += w.PB) {
    a.p_begin = b0;
    a.p_count = std::min<int64_t>(w.PB, p.n - b0);
    a.pairs = nullptr;  // the adjoint's are counted
    if (p.alm) {
      // the a_lm rows the forward pass kept
      a.A = alm_rows(p) + size_t(b0) * w.lay.W;
    } else {
      StageScope sc(p.trace, G3PCF_STAGE_PAIRS, st);
      if ((e = launch_pair_forward(a, fp64, p.basis, false, st)) != hipSuccess)
        return hip_fail(e, "pair kernel (recompute)");
    }
    AdjArgs j{};
    j.A = a.A;
    j.nprim = &c->nprim;
    j.p_begin = b0;
    j.p_count = a.p_count;
    j.lay = w.lay;
    j.MHt = at<double>(ws, w.mht);
    j.H = at<double>(ws, w.hrows);
    j.queue = c->xcd[0].queue;
    {
      StageScope sc(p.trace, G3PCF_STAGE_ADJ_COEF, st);
      if ((e = launch_h_gemm(j, st)) != hipSuccess) return hip_fail(e, "adjoint GEMM");
    }
    a.pairs = p.pairs_out ? &c->xcd[0].pairs_adj : nullptr;
    a.queue = c->xcd[0].queue + kQueueAdjoint;
    {
      StageScope sc(p.trace, G3PCF_STAGE_PAIR_ADJOINT, st);
      if ((e = launch_pair_adjoint(a, fp64, st)) != hipSuccess)
        return hip_fail(e, "pair adjoint kernel");
    }
    a.queue = c->xcd[0].queue;
  }
  const unsigned long long* saved = p.alm ? static_cast<const unsigned long long*>(p.alm) : nullptr;
  if ((e = launch_unpermute(gsort, gsort32, a.perm, p.n, p.accumulate, saved, &c->inputs_hash, grad_w,
                            st)) != hipSuccess)
    return hip_fail(e, "gradient permute");
  return finish_pairs(p, w, ws, st, true);
}

int g3pcf_isotropic(int lmax, int nbins, const double* zeta, double* iso, void* stream) {
  if (lmax < 0 || lmax > kDeg) return fail(G3PCF_EINVAL, "lmax must be 0..10");
  if (nbins < 1 || nbins > kMaxBins) return fail(G3PCF_EINVAL, "nbins must be 1..32");
  if (!zeta || !iso) return fail(G3PCF_EINVAL, "zeta and iso must be non-NULL");
  const hipError_t e = launch_isotropic(zeta, lmax, nbins, iso, static_cast<hipStream_t>(stream));
  return e == hipSuccess ? G3PCF_OK : hip_fail(e, "isotropic");
}

int g3pcf_degenerate_term(int lmax, double uz, double* out) {
  if (lmax < 0 || lmax > kDeg || !out) return fail(G3PCF_EINVAL, "lmax 0..10 and out required");
  static std::vector<double> G;
  static std::mutex mu;
  {
    std::lock_guard<std::mutex> lk(mu);
    if (G.empty()) {
      G.resize(kDegTable);
      build_deg_table(G.data());
    }
  }
  double pn[kTermsDeg];
  pn[0] = 1.0;
  pn[1] = uz;
  for (int n = 1; n + 1 < kTermsDeg; ++n) pn[n + 1] = 2.0 * uz * pn[n] - pn[n - 1];
  const int L1 = lmax + 1;
  for (int m = 0; m <= lmax; ++m)
    for (int l = 0; l <= lmax; ++l)
      for (int lp = 0; lp <= lmax; ++lp) {
        double s = 0.0;
        if (l >= m && lp >= m)
          for (int n = 0; n <= l + lp; ++n) s += G[deg_index(m, l, lp, n)] * pn[n];
        out[(m * L1 + l) * L1 + lp] = s;
      }
  return G3PCF_OK;
}

}  // extern "C"
