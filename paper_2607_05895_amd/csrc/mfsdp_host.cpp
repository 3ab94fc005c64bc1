// Host side of the C ABI declared in include/mfsdp.h: argument validation (all before any
// launch), workspace planning, descriptor upload and the launch sequence of the owner step.
//
// Launch sequence of mfsdp_muon_step (all on the caller's stream):
//   1. descriptor upload (pinned staging slot -> workspace)
//   2. prep     : momentum EMA + Nesterov, Sum u^2 partials, u in both layouts   (one launch)
//   3. norm     : per-matrix scale 1 / max(||u||_F, eps)                          (one launch)
//   4. K times  : Gram A = X X^T, square B = bA + cAA, update X' = aX + BX        (3 launches
//                 per step, each grouped over every matrix, heaviest tiles first)
//   5. apply    : p <- p (1 - lr wd) - lr f O                                     (one launch)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/mfsdp.h"
#include "mfsdp_internal.h"

using namespace mfsdp;

static_assert(MFSDP_MAX_GRAD_PARTS == kMaxGradParts, "gradient part limit of the ABI and the descriptor");

namespace {

thread_local std::string g_last_error;

int fail(int status, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  g_last_error = buf;
  return status;
}

}  // namespace

namespace mfsdp {
int set_last_error(int status, const std::string& msg) {
  g_last_error = msg;
  return status;
}
}  // namespace mfsdp

namespace {

constexpr size_t kAlign = 256;
inline size_t align_up(size_t x, size_t a = kAlign) { return (x + a - 1) / a * a; }
inline int64_t round_up(int64_t x, int64_t a) { return (x + a - 1) / a * a; }

bool valid_dtype(int32_t dt) { return dt == MFSDP_F32 || dt == MFSDP_BF16; }
bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// ---------------------------------------------------------------------------------------------
// Workspace plan for one NS problem (shared by the Muon step and standalone NS).
struct NsPlan {
  int64_t m, n, r, s, r_pad, s_pad;
  int64_t r_eff, s_eff;     // the part of the padded domain that the products cover
  bool tall;
  int es;                   // element size of the NS dtype
  size_t off_x[2], off_xt[2], off_g, off_h, off_partials, off_scale;
  int prep_tiles_m, prep_tiles_n;
  size_t bytes;             // total for this problem
};

NsPlan plan_ns(int64_t m, int64_t n, int ns_dtype, size_t base) {
  NsPlan p{};
  p.m = m;
  p.n = n;
  p.tall = m > n;
  p.r = std::min(m, n);
  p.s = std::max(m, n);
  const int tile = ns_dtype == MFSDP_BF16 ? kTileBF16 : kTileF32;
  p.r_pad = round_up(p.r, tile);
  p.s_pad = round_up(p.s, tile);
  p.r_eff = p.r_pad;
  p.s_eff = p.s_pad;
  p.es = ns_dtype == MFSDP_BF16 ? 2 : 4;
  const size_t xb = align_up(size_t(p.r_pad) * size_t(p.s_pad) * p.es);
  const size_t gb = align_up(size_t(p.r_pad) * size_t(p.r_pad) * p.es);
  const int64_t rows = p.tall ? p.s_pad : p.r_pad, cols = p.tall ? p.r_pad : p.s_pad;
  p.prep_tiles_m = int(rows / kPrepRows);
  p.prep_tiles_n = int(cols / (ns_dtype == MFSDP_BF16 ? kPrepColsBF16 : kPrepColsF32));
  size_t o = base;
  p.off_x[0] = o; o += xb;
  p.off_x[1] = o; o += xb;
  p.off_xt[0] = o; o += xb;
  p.off_xt[1] = o; o += xb;
  p.off_g = o; o += gb;
  p.off_h = o; o += gb;
  p.off_partials = o; o += align_up(size_t(p.prep_tiles_m) * p.prep_tiles_n * sizeof(float));
  p.off_scale = o; o += kAlign;
  p.bytes = o - base;
  return p;
}

// Descriptor region at the start of the workspace.
struct DescLayout {
  size_t off_prep, off_norm, off_gemm[3], off_apply, off_sched[3], off_jobs, bytes;
  int ngroups[3];
  int njobs;  // tiles of the split Gram problems (second pass)
};


DescLayout plan_descs(int64_t count, const size_t sched_bytes[3], int njobs) {
  DescLayout d{};
  size_t o = 0;
  d.off_prep = o; o += align_up(sizeof(PrepDesc) * count);
  d.off_norm = o; o += align_up(sizeof(NormDesc) * count);
  for (int k = 0; k < 3; ++k) { d.off_gemm[k] = o; o += align_up(sizeof(GemmDesc) * count); }
  d.off_apply = o; o += align_up(sizeof(ApplyDesc) * count);
  for (int k = 0; k < 3; ++k) { d.off_sched[k] = o; o += align_up(sched_bytes[k]); }
  d.off_jobs = o; o += align_up(sizeof(TileRef) * size_t(njobs));
  d.njobs = njobs;
  d.bytes = o;
  return d;
}

// ---------------------------------------------------------------------------------------------
// Pinned staging ring for descriptor uploads. A slot is reused only after the copy that read it
// has completed (event per slot).
class StagingRing {
 public:
  static constexpr int kSlots = 16;
  int acquire(size_t bytes, void** host, hipStream_t st) {
    (void)st;
    std::lock_guard<std::mutex> lk(mu_);
    const int s = next_;
    next_ = (next_ + 1) % kSlots;
    Slot& sl = slots_[s];
    if (sl.event) {
      hipError_t e = hipEventSynchronize(sl.event);
      if (e != hipSuccess) return fail(MFSDP_E_HIP, "staging event: %s", hipGetErrorString(e));
    }
    if (sl.cap < bytes) {
      if (sl.ptr) (void)hipHostFree(sl.ptr);
      sl.ptr = nullptr;
      sl.cap = 0;
      size_t cap = std::max<size_t>(bytes, 64 * 1024);
      hipError_t e = hipHostMalloc(&sl.ptr, cap, hipHostMallocDefault);
      if (e != hipSuccess) return fail(MFSDP_E_HIP, "hipHostMalloc: %s", hipGetErrorString(e));
      sl.cap = cap;
    }
    if (!sl.event) {
      hipError_t e = hipEventCreateWithFlags(&sl.event, hipEventDisableTiming);
      if (e != hipSuccess) return fail(MFSDP_E_HIP, "hipEventCreate: %s", hipGetErrorString(e));
    }
    *host = sl.ptr;
    return s;
  }
  int upload(int slot, void* dst, size_t bytes, hipStream_t st) {
    Slot& sl = slots_[slot];
    hipError_t e = hipMemcpyAsync(dst, sl.ptr, bytes, hipMemcpyHostToDevice, st);
    if (e != hipSuccess) return fail(MFSDP_E_HIP, "descriptor upload: %s", hipGetErrorString(e));
    e = hipEventRecord(sl.event, st);
    if (e != hipSuccess) return fail(MFSDP_E_HIP, "hipEventRecord: %s", hipGetErrorString(e));
    return MFSDP_OK;
  }

 private:
  struct Slot {
    void* ptr = nullptr;
    size_t cap = 0;
    hipEvent_t event = nullptr;
  };
  std::mutex mu_;
  int next_ = 0;
  Slot slots_[kSlots];
};

StagingRing& ring() {
  static StagingRing* r = new StagingRing();  // lives until process exit
  return *r;
}

int check_hp(const mfsdp_muon_hparams* hp) {
  if (!hp) return fail(MFSDP_E_INVALID, "hparams is NULL");
  if (!(hp->lr >= 0.0) || !std::isfinite(hp->lr)) return fail(MFSDP_E_INVALID, "lr must be >= 0");
  if (!(hp->weight_decay >= 0.0) || !std::isfinite(hp->weight_decay))
    return fail(MFSDP_E_INVALID, "weight_decay must be >= 0");
  if (!(hp->momentum >= 0.0 && hp->momentum < 1.0))
    return fail(MFSDP_E_INVALID, "momentum must be in [0, 1)");
  if (hp->nesterov != 0 && hp->nesterov != 1) return fail(MFSDP_E_INVALID, "nesterov must be 0 or 1");
  if (hp->ns_steps < 0 || hp->ns_steps >= 100) return fail(MFSDP_E_INVALID, "ns_steps must be in [0, 100)");
  if (hp->ns_schedule) {
    for (int i = 0; i < 3 * hp->ns_steps; ++i)
      if (!std::isfinite(hp->ns_schedule[i]))
        return fail(MFSDP_E_INVALID, "ns_schedule entry %d is not finite", i);
  } else if (!std::isfinite(hp->a) || !std::isfinite(hp->b) || !std::isfinite(hp->c)) {
    return fail(MFSDP_E_INVALID, "NS coefficients must be finite");
  }
  if (!(hp->eps > 0.0) || !std::isfinite(hp->eps)) return fail(MFSDP_E_INVALID, "eps must be > 0");
  if (hp->lr_adjust < MFSDP_LR_NONE || hp->lr_adjust > MFSDP_LR_MATCH_RMS_ADAMW)
    return fail(MFSDP_E_INVALID, "unknown lr_adjust %d", hp->lr_adjust);
  if (!valid_dtype(hp->ns_dtype)) return fail(MFSDP_E_INVALID, "unknown ns_dtype %d", hp->ns_dtype);
  return MFSDP_OK;
}

constexpr int64_t kMaxDim = int64_t(1) << 20;   // per-side limit (index math stays in int32 tiles)

int check_shape(int64_t m, int64_t n, const char* what, int64_t i) {
  if (m <= 0 || n <= 0) return fail(MFSDP_E_INVALID, "%s %lld: shape %lldx%lld must be positive", what,
                                    (long long)i, (long long)m, (long long)n);
  if (m > kMaxDim || n > kMaxDim)
    return fail(MFSDP_E_INVALID, "%s %lld: side larger than %lld", what, (long long)i, (long long)kMaxDim);
  return MFSDP_OK;
}

// need_grad: the entries' grad pointers are read (0 for the workspace query and the fused
// reduction, which read no entry grad)
int check_entries(const mfsdp_muon_entry* entries, int64_t count, bool need_grad = true) {
  if (count < 0) return fail(MFSDP_E_INVALID, "count must be >= 0");
  if (count > 0 && !entries) return fail(MFSDP_E_INVALID, "entries is NULL");
  if (count > (1 << 20)) return fail(MFSDP_E_INVALID, "too many entries");
  int64_t units = 0;  // bound on the 64 x 64 tiles of any one grouped launch (grid and int32 counters)
  for (int64_t i = 0; i < count; ++i) {
    const mfsdp_muon_entry& e = entries[i];
    if (!e.param || (need_grad && !e.grad) || !e.momentum)
      return fail(MFSDP_E_INVALID, "entry %lld: NULL pointer", (long long)i);
    int st = check_shape(e.m, e.n, "entry", i);
    if (st) return st;
    units += (round_up(e.m, kTileBF16) / 64) * (round_up(e.n, kTileBF16) / 64);
    if (units > (int64_t(1) << 30))
      return fail(MFSDP_E_INVALID, "the entries of one call exceed 2^30 tiles per launch");
    if (!valid_dtype(e.param_dtype) || !valid_dtype(e.grad_dtype))
      return fail(MFSDP_E_INVALID, "entry %lld: unsupported dtype", (long long)i);
    if (!aligned16(e.param) || (need_grad && !aligned16(e.grad)) || !aligned16(e.momentum) ||
        (e.update_out && !aligned16(e.update_out)))
      return fail(MFSDP_E_INVALID, "entry %lld: pointers must be 16-byte aligned", (long long)i);
  }
  return MFSDP_OK;
}

double lr_factor(int64_t m, int64_t n, int mode) {
  if (mode == MFSDP_LR_ORIGINAL) return std::sqrt(std::max(1.0, double(m) / double(n)));
  if (mode == MFSDP_LR_MATCH_RMS_ADAMW) return 0.2 * std::sqrt(double(std::max(m, n)));
  return 1.0;
}

int hip_fail(hipError_t e, const char* what) {
  return fail(MFSDP_E_HIP, "%s: %s", what, hipGetErrorString(e));
}

// Builds and enqueues the NS pipeline for a set of problems that already have their prep
// descriptors filled. Shared by the Muon step and standalone NS.
// Problem order of one NS product: heaviest K first (all tiles have the same size, so the work
// of a tile is proportional to K).
std::vector<int> phase_order(const std::vector<NsPlan>& plans, int phase) {
  std::vector<int> ord(plans.size());
  for (size_t i = 0; i < ord.size(); ++i) ord[i] = int(i);
  std::stable_sort(ord.begin(), ord.end(), [&](int x, int y) {
    const int64_t kx = phase == 0 ? plans[x].s_pad : plans[x].r_pad;
    const int64_t ky = phase == 0 ? plans[y].s_pad : plans[y].r_pad;
    return kx > ky;
  });
  return ord;
}

// Everything about a call that follows from the shapes and the NS dtype: per-matrix buffers,
// the problem order and tile schedule of each NS product, and the descriptor region layout.
struct Plan {
  std::vector<NsPlan> ns;
  std::vector<int> order[3];
  std::vector<TileRef> sched[3];
  int tiles[3] = {0, 0, 0};
  int tile[3] = {0, 0, 0};     // output tile of each product's launch
  std::vector<int> split;      // per Gram problem (launch order): K ranges per tile
  std::vector<size_t> part;    // per Gram problem: offset of its partial tiles (split ones)
  std::vector<TileRef> jobs;   // the split problems' upper tiles (second pass)
  DescLayout dl{};
  size_t bytes = 0;
  bool fine = false;           // every product on 128 x 128 tiles, matrices padded to 128
};

// Output tile of a product of the fp32 path: 64 x 64 where 128 x 128 tiles would leave more than half of the
// CUs without one.
int h2_tile(const std::vector<NsPlan>& shapes, int phase) {
  int64_t n = 0;
  for (const NsPlan& p : shapes) {
    const int64_t tr = (p.r_pad + 127) / 128, ts = (p.s_pad + 127) / 128;
    n += phase == 2 ? tr * ts : tr * (tr + 1) / 2;
  }
  return n <= 128 ? 64 : 128;
}

// K ranges of the fp32 path's Gram tiles (in launch order): while the launch has fewer tiles than the chip
// holds workgroups, the most ranges (at most 8, of whole pairs of K steps) that keep a range at least
// 256 long and at least the launch's work per workgroup, and whose partial tiles fit the iterate's free
// buffer (r_pad x s_pad fp32).
std::vector<int> h2_splits(const std::vector<NsPlan>& shapes, const std::vector<int>& order, int tile) {
  std::vector<int> f(order.size(), 1);
  const int64_t slots = 512;
  int64_t T = 0, W = 0;
  auto tiles = [&](const NsPlan& p) {
    const int64_t t = (p.r_pad + tile - 1) / tile;
    return t * (t + 1) / 2;
  };
  for (const NsPlan& p : shapes) {
    T += tiles(p);
    W += tiles(p) * p.s_pad;
  }
  if (T >= slots) return f;
  const int64_t target = std::max<int64_t>(256, W / slots);
  for (size_t k = 0; k < order.size(); ++k) {
    const NsPlan& p = shapes[size_t(order[k])];
    for (int c = 2; c <= 8; ++c)
      if ((p.s_pad / 32) % c == 0 && p.s_pad / c >= target && tiles(p) * c * tile * tile <= p.r_pad * p.s_pad)
        f[k] = c;
  }
  return f;
}

// On the bf16 path a Gram launch with fewer tiles than the persistent grid has workgroups may split
// long contractions (gram_splits); the split problems' partial tiles follow the per-matrix buffers
// and take at most a quarter of their bytes. When the r x r products' 128 x 128 tiles fit one round
// of the two-workgroups-per-CU grid, the Gram and square launches run on those (small shares: four
// times the tiles of launches that would leave most CUs idle, each with a quarter of the epilogue).
// When the updates' 128 x 128 tiles fit one round too, every product runs on them and covers the matrices
// padded to 128 only (`fine`): one 1000 x 2777 matrix has 44 256 x 256 update tiles for 256 CUs, 35.6 us per
// update, against 176 tiles and 17.0 us (the whole orthogonalisation, with its last epilogue, 410 -> 295 us).
template <typename ShapeAt>
Plan make_plan_tiles(int64_t count, int ns_dtype, ShapeAt shape_at, bool fine) {
  Plan P;
  std::vector<NsPlan> shapes;
  for (int64_t i = 0; i < count; ++i) {
    int64_t m, n;
    shape_at(i, m, n);
    shapes.push_back(plan_ns(m, n, ns_dtype, 0));
  }
  const bool bf = ns_dtype == MFSDP_BF16;
  const int64_t small_slots = int64_t(kGemmXcds) * 2 * kGemmSlots;
  int64_t small_tiles = 0, fine_tiles = 0;  // 128 x 128 tiles: upper ones of the r x r products, the updates'
  for (const NsPlan& p : shapes) {
    const int64_t t = p.r_pad / kTileBF16Small;
    small_tiles += t * (t + 1) / 2;
    fine_tiles += ((p.r + kTileBF16Small - 1) / kTileBF16Small) * ((p.s + kTileBF16Small - 1) / kTileBF16Small);
  }
  fine = fine && bf && fine_tiles <= small_slots;
  P.fine = fine;
  const bool small_gram = bf && small_tiles <= small_slots;  // of the plan that is not fine
  if (fine)
    for (NsPlan& p : shapes) {
      p.r_eff = round_up(p.r, kTileBF16Small);
      p.s_eff = round_up(p.s, kTileBF16Small);
    }
  size_t sched_bytes[3] = {0, 0, 0};
  for (int ph = 0; ph < 3; ++ph) {
    const bool small = bf && (fine || (ph < 2 && small_gram));
    const int tile = !bf ? h2_tile(shapes, ph) : small ? kTileBF16Small : kTileBF16;
    P.tile[ph] = tile;
    P.order[ph] = phase_order(shapes, ph);
    std::vector<TileGrid> grids;
    std::vector<int> pos;
    std::vector<int64_t> cost;
    for (int k = 0; k < int(count); ++k) {
      const NsPlan& p = shapes[P.order[ph][k]];
      const int tr = int((p.r_eff + tile - 1) / tile), ts = int((p.s_eff + tile - 1) / tile);
      const TileGrid g = ph == 2 ? TileGrid{tr, ts, false} : TileGrid{tr, tr, true};
      grids.push_back(g);
      pos.push_back(k);
      cost.push_back(ph == 0 ? p.s_eff : p.r_eff);
      P.tiles[ph] += g.sym ? g.tm * (g.tm + 1) / 2 : g.tm * g.tn;
    }
    if (ph == 0) {
      P.split.assign(size_t(count), 1);
      if (bf) {
        // The K ranges follow from the matrices padded to 256 and the tile of the plan that is not fine, whichever
        // plan this is: a range's sum is rounded on its own, so both plans give the same bits.
        const int64_t ct = small_gram ? kTileBF16Small : kTileBF16;
        std::vector<int64_t> tl, kl;
        size_t base = 0;
        for (const NsPlan& q : shapes) base += q.bytes;
        for (int k : P.order[0]) {
          const NsPlan& q = shapes[size_t(k)];
          const int64_t t = q.r_pad / ct;
          tl.push_back(t * (t + 1) / 2);
          kl.push_back(q.s_pad);
        }
        P.split = gram_splits(tl, kl, int64_t(base / 4 / size_t(ct * ct * int64_t(sizeof(float)))),
                              small_gram ? small_slots : int64_t(kGemmXcds) * kGemmSlots);
      }
      if (!bf) {
        P.split = h2_splits(shapes, P.order[0], tile);
        P.tiles[0] = 0;
        for (size_t k = 0; k < grids.size(); ++k)
          P.tiles[0] += grids[k].tm * (grids[k].tm + 1) / 2 * P.split[k];
      }
      for (int k = 0; bf && k < int(count); ++k)
        if (P.split[size_t(k)] > 1)
          for (int bi = 0; bi < grids[size_t(k)].tm; ++bi)
            for (int bj = bi; bj < grids[size_t(k)].tm; ++bj)
              P.jobs.push_back(TileRef{k, int16_t(bi), int16_t(bj), 0, 0});
    }
    if (bf && small) {
      // at most one tile per CU when they fit: groups of kGemmSlots tiles on the 2 x kGemmSlots slots
      int64_t n = 0;
      for (size_t k = 0; k < grids.size(); ++k)
        n += ph == 2 ? int64_t(grids[k].tm) * grids[k].tn
                     : int64_t(grids[k].tm) * (grids[k].tm + 1) / 2 * (ph == 0 ? P.split[k] : 1);
      const int fill = n <= int64_t(kGemmXcds) * kGemmSlots ? kGemmSlots : 2 * kGemmSlots;
      P.sched[ph] = build_schedule(pos, grids, cost, ph == 0 ? &P.split : nullptr, 2 * kGemmSlots,
                                   2 * kGroupRows, fill);
    } else if (bf)
      P.sched[ph] = build_schedule(pos, grids, cost, ph == 0 ? &P.split : nullptr);
    sched_bytes[ph] = P.sched[ph].size() * sizeof(TileRef);
  }
  P.dl = plan_descs(count, sched_bytes, int(P.jobs.size()));
  for (int ph = 0; ph < 3; ++ph)
    P.dl.ngroups[ph] = int(P.sched[ph].size() / (P.tile[ph] == kTileBF16Small ? 2 * kGemmSlots : kGemmSlots));
  size_t o = P.dl.bytes;
  for (int64_t i = 0; i < count; ++i) {
    P.ns.push_back(plan_ns(shapes[i].m, shapes[i].n, ns_dtype, o));
    P.ns.back().r_eff = shapes[i].r_eff;
    P.ns.back().s_eff = shapes[i].s_eff;
    o += P.ns.back().bytes;
  }
  P.part.assign(size_t(count), 0);
  for (int k = 0; k < int(count); ++k) {
    const int f = P.split[size_t(k)];
    if (f <= 1 || !bf) continue;
    const int64_t tr = shapes[size_t(P.order[0][size_t(k)])].r_eff / P.tile[0];
    P.part[size_t(k)] = o;
    o += align_up(size_t(tr * (tr + 1) / 2) * size_t(f) * P.tile[0] * P.tile[0] * sizeof(float));
  }
  P.bytes = o;
  return P;
}

// in_scratch: for the allocation-free step, whose scratch array has a fixed size. (The fine plan's update schedule
// is a few KiB larger: entries that fit the array without it keep the plan that fits.)
template <typename ShapeAt>
Plan make_plan(int64_t count, int ns_dtype, ShapeAt shape_at, bool in_scratch = false) {
  Plan P = make_plan_tiles(count, ns_dtype, shape_at, true);
  if (in_scratch && P.fine && P.bytes > size_t(MFSDP_NOALLOC_SCRATCH_BYTES)) {
    Plan coarse = make_plan_tiles(count, ns_dtype, shape_at, false);
    if (coarse.bytes <= size_t(MFSDP_NOALLOC_SCRATCH_BYTES)) return coarse;
  }
  return P;
}

// Coefficients of every NS step: the schedule if given, else the fixed triple.
std::vector<double> step_coeffs(double a, double b, double c, int steps, const double* schedule) {
  std::vector<double> v(3 * size_t(steps));
  for (int k = 0; k < steps; ++k) {
    v[3 * k] = schedule ? schedule[3 * k] : a;
    v[3 * k + 1] = schedule ? schedule[3 * k + 1] : b;
    v[3 * k + 2] = schedule ? schedule[3 * k + 2] : c;
  }
  return v;
}

// With at least one NS step the last update product applies the parameter update in its epilogue (from
// the fp32 accumulators); otherwise a separate apply pass reads the iterate.
bool apply_fused(int steps) { return steps >= 1; }

// The fp32 path's scales, step by step, where bounds from the coefficients alone serve; else none (the kernels
// then form them from the data). Every buffer's elements are bounded by a bound on its singular values: sigma of X
// (1 at first: the Frobenius norm), sigma^2 of A, max |a + b y + c y^2| over [0, sigma^2] of B', max |x (a + b x^2 +
// c x^4)| over [0, sigma] of the next X (with 1 % for rounding). A buffer's exponent takes its bound to at
// most 2^14, a factor of four inside fp16's range (2^15 and two for X_0).
// slack bounds by how much the true singular values can have shrunk against sigma since the start: a step moves
// every singular value by at least min |a + b y + c y^2| and the bound by its ratio. The fixed triple reaches 2^3.4
// in five steps; a schedule whose bounds run away, or that may cancel singular values, passes 2^10 at once.
constexpr double kH2MaxSlack = 1024.0;
std::vector<NsH2Exponents> h2_exponents(const double* coeffs, int steps) {
  auto exponent = [](double bound) { return int(std::min(100.0, std::max(-100.0, std::floor(14.0 - std::log2(bound))))); };
  std::vector<NsH2Exponents> s;
  double sigma = 1.0, slack = 1.0, growth = 1.0;  // growth: of a small X, whatever the bounds
  int ex = kNsH2First, gx = 0;
  for (int k = 0; k < steps; ++k) {
    const double a = coeffs[3 * k], b = coeffs[3 * k + 1], c = coeffs[3 * k + 2];
    auto q = [&](double y) { return std::fabs(a + b * y + c * y * y); };
    auto p = [&](double y) { return std::sqrt(y) * q(y); };
    const double y1 = sigma * sigma;
    double bb = std::max(q(0.0), q(y1)), bx = p(y1), low = std::min(q(0.0), q(y1));
    if ((a > 0.0) != (a + b * y1 + c * y1 * y1 > 0.0)) low = 0.0;  // a zero between
    auto at = [&](double y) {
      if (!(y > 0.0 && y < y1)) return;
      bb = std::max(bb, q(y));
      bx = std::max(bx, p(y));
      low = (a > 0.0) != (a + b * y + c * y * y > 0.0) ? 0.0 : std::min(low, q(y));
    };
    if (c != 0.0) {
      at(-b / (2.0 * c));
      const double disc = 9.0 * b * b - 20.0 * a * c;  // a + 3 b y + 5 c y^2 = 0
      if (disc >= 0.0) {
        at((-3.0 * b + std::sqrt(disc)) / (10.0 * c));
        at((-3.0 * b - std::sqrt(disc)) / (10.0 * c));
      }
    } else if (b != 0.0) {
      at(-a / (3.0 * b));
    }
    const double next = 1.01 * bx;
    slack *= next / (sigma * low);
    if (!(slack <= kH2MaxSlack) || !(bb > 1e-18 && bb < 1e18) || !(next > 1e-18 && next < 1e18)) return {};
    sigma = next;
    growth *= 1.01 * bb;
    NsH2Exponents h{ex, exponent(y1), exponent(bb), exponent(sigma), gx, 0};
    h.gxn = int(std::max(-1000.0, std::floor(std::log2(sigma / growth))));
    ex = h.exn;
    gx = h.gxn;
    s.push_back(h);
  }
  return s;
}

// Descriptors of the three products, stored in the phase's problem order; the schedules refer
// to problems by that position.
void fill_gemm_descs(const Plan& P, uint8_t* ws, const mfsdp_muon_hparams& hp, uint8_t* h) {
  const int n = int(P.ns.size());
  for (int phase = 0; phase < 3; ++phase) {
    const int tile = P.tile[phase];
    GemmDesc* out = reinterpret_cast<GemmDesc*>(h + P.dl.off_gemm[phase]);
    const std::vector<int>& ord = P.order[phase];
    int begin = 0, sum_begin = 0;
    for (int k = 0; k < n; ++k) {
      const NsPlan& p = P.ns[ord[k]];
      GemmDesc d{};
      const int tr = int((p.r_eff + tile - 1) / tile), ts = int((p.s_eff + tile - 1) / tile);
      const bool h2 = hp.ns_dtype == MFSDP_F32;
      for (int par = 0; par < 2; ++par) {
        uint8_t* xin = ws + p.off_x[par];
        uint8_t* xtin = ws + p.off_xt[par];
        uint8_t* xout = ws + p.off_x[par ^ 1];
        uint8_t* xtout = ws + p.off_xt[par ^ 1];
        if (phase == 0) {         // A = X X^T
          d.P[par] = xin; d.Q[par] = xin; d.E[par] = nullptr;
          d.C[par] = ws + p.off_g; d.CT[par] = h2 ? ws + p.off_x[par ^ 1] : nullptr;
        } else if (phase == 1) {  // B' = c A A + b A + a I
          d.P[par] = ws + p.off_g; d.Q[par] = ws + p.off_g; d.E[par] = ws + p.off_g;
          d.C[par] = ws + p.off_h; d.CT[par] = nullptr;
        } else {                  // X' = B' X (= a X + B X), stored as X' and X'^T
          d.P[par] = ws + p.off_h; d.Q[par] = xtin; d.E[par] = nullptr;
          d.C[par] = xout; d.CT[par] = xtout;
        }
      }
      d.scale = reinterpret_cast<const float*>(ws + p.off_scale);
      if (phase == 0) {
        d.ldp = d.ldq = p.s_pad; d.lde = 0; d.ldc = p.r_pad; d.ldct = 0;
        d.M = d.N = int(p.r_eff); d.K = int(p.s_eff);
        d.alpha = 1.0f; d.beta = 0.0f; d.alpha_scale_pow = 2; d.beta_scale_pow = 0;
        d.sym = 1; d.tiles_m = d.tiles_n = tr;
        d.tile_count = tr * (tr + 1) / 2;
        d.last_c = 1; d.last_ct = 0;
        d.nks = P.split[size_t(k)];
        // (the last range ends at K, which the padded length that the ranges divide exceeds by less than a range)
        d.kper = int(p.s_pad / kBlkCols / d.nks);
        d.part = d.nks > 1 && !h2 ? reinterpret_cast<float*>(ws + P.part[size_t(k)]) : nullptr;
        if (h2) {
          d.ldct = sum_begin;
          sum_begin += d.tile_count * (tile / 16);
          d.tile_count *= d.nks;
        }
      } else if (phase == 1) {
        d.ldp = d.ldq = d.lde = d.ldc = p.r_pad; d.ldct = 0;
        d.M = d.N = d.K = int(p.r_eff);
        d.alpha = 0.0f; d.beta = 0.0f;  // the step's (a, b, c) come with each launch
        d.alpha_scale_pow = 0; d.beta_scale_pow = 0;
        d.sym = 1; d.tiles_m = d.tiles_n = tr;
        d.tile_count = tr * (tr + 1) / 2;
        d.last_c = 1; d.last_ct = 0;
      } else {
        d.ldp = p.r_pad; d.ldq = p.r_pad; d.lde = 0; d.ldc = p.s_pad; d.ldct = p.r_pad;
        d.M = int(p.r_eff); d.N = int(p.s_eff); d.K = int(p.r_eff);
        d.alpha = 1.0f; d.beta = 0.0f; d.alpha_scale_pow = 1; d.beta_scale_pow = 0;
        d.sym = 0; d.tiles_m = tr; d.tiles_n = ts;
        d.tile_count = tr * ts;
        // the final iterate is read in the parameter's orientation only
        d.last_c = p.tall ? 0 : 1;
        d.last_ct = p.tall ? 1 : 0;
        if (apply_fused(hp.ns_steps))
          d.fused = reinterpret_cast<const ApplyDesc*>(ws + P.dl.off_apply) + ord[k];
      }
      d.tile_begin = begin;
      begin += d.tile_count;
      out[k] = d;
    }
    if (!P.sched[phase].empty())
      std::memcpy(h + P.dl.off_sched[phase], P.sched[phase].data(),
                  P.sched[phase].size() * sizeof(TileRef));
  }
  if (!P.jobs.empty()) std::memcpy(h + P.dl.off_jobs, P.jobs.data(), P.jobs.size() * sizeof(TileRef));
}

PrepDesc make_prep(const NsPlan& p, uint8_t* ws, const void* grad, int grad_dtype, float* momentum,
                   int tile_begin) {
  PrepDesc d{};
  d.grad = grad;
  d.momentum = momentum;
  // u in its stored orientation is X (wide) or X^T (tall); its transpose goes to the other one. On the fp32
  // path u goes to the second buffer of the pair, from where the split pass forms X_0 in both layouts.
  const int u = p.es == 4 ? 1 : 0;
  if (p.tall) {
    d.d_out = ws + p.off_xt[u]; d.ld_d = p.r_pad;
    d.t_out = ws + p.off_x[0];  d.ld_t = p.s_pad;
  } else {
    d.d_out = ws + p.off_x[u];  d.ld_d = p.s_pad;
    d.t_out = ws + p.off_xt[0]; d.ld_t = p.r_pad;
  }
  d.partials = reinterpret_cast<float*>(ws + p.off_partials);
  d.m = p.m;
  d.n = p.n;
  d.tiles_m = p.prep_tiles_m;
  d.tiles_n = p.prep_tiles_n;
  d.grad_dtype = grad_dtype;
  d.tile_begin = tile_begin;
  return d;
}

ApplyDesc make_apply(const NsPlan& p, uint8_t* ws, int steps, void* param, int param_dtype,
                     float* update_out, int mode, float decay, float step, int tile_begin) {
  ApplyDesc d{};
  // the buffer holding the final iterate (read by the apply pass when there is no NS step)
  const int par = p.es == 4 && steps == 0 ? 1 : steps & 1;
  if (p.tall) { d.o = ws + p.off_xt[par]; d.ld_o = p.r_pad; }
  else        { d.o = ws + p.off_x[par];  d.ld_o = p.s_pad; }
  d.param = param;
  d.update_out = update_out;
  d.scale = reinterpret_cast<const float*>(ws + p.off_scale);
  d.use_scale = steps == 0 ? 1 : 0;
  d.m = p.m;
  d.n = p.n;
  d.param_dtype = param_dtype;
  d.mode = mode;
  d.decay = decay;
  d.step = step;
  d.tiles_m = int((p.m + kApplyRows - 1) / kApplyRows);
  d.tiles_n = int((p.n + kApplyCols - 1) / kApplyCols);
  d.tile_begin = tile_begin;
  return d;
}

// Enqueue everything after the descriptors are in host staging memory `h`.
int record(void* const* events, int k, hipStream_t st) {
  if (!events || !events[k]) return MFSDP_OK;
  hipError_t e = hipEventRecord(static_cast<hipEvent_t>(events[k]), st);
  return e == hipSuccess ? MFSDP_OK : hip_fail(e, "hipEventRecord");
}

int upload_as_kernel_args(const uint8_t* host, size_t bytes, uint8_t* dst, hipStream_t st);

// coeffs: 3 * steps doubles, (a_k, b_k, c_k) of NS step k.
// Descriptors: slot >= 0 uploads them from that pinned staging slot; slot < 0 passes them from the
// host buffer `host_descs` as kernel arguments (the allocation-free step).
int enqueue_pipeline(const Plan& P, uint8_t* ws, int slot, int steps, const double* coeffs,
                     int ns_dtype, double beta, int nesterov, double eps, int prep_tiles,
                     int apply_tiles, hipStream_t st, void* const* events, bool reduce = false,
                     const uint8_t* host_descs = nullptr) {
  const int count = int(P.ns.size());
  const DescLayout& dl = P.dl;
  int rc = slot >= 0 ? ring().upload(slot, ws, dl.bytes, st) : upload_as_kernel_args(host_descs, dl.bytes, ws, st);
  if (rc) return rc;
  if ((rc = record(events, 0, st))) return rc;
  hipError_t e;
  e = launch_prep(reinterpret_cast<const PrepDesc*>(ws + dl.off_prep), count, prep_tiles, ns_dtype,
                  reduce ? 1 : 0, float(beta), float(1.0 - beta), nesterov, st);
  if (e != hipSuccess) return hip_fail(e, "prep launch");
  e = launch_norm(reinterpret_cast<const NormDesc*>(ws + dl.off_norm), count, float(eps), st);
  if (e != hipSuccess) return hip_fail(e, "norm launch");
  if ((rc = record(events, 1, st))) return rc;
  auto descs = [&](int ph) { return reinterpret_cast<const GemmDesc*>(ws + dl.off_gemm[ph]); };
  if (ns_dtype == MFSDP_F32 && steps > 0) {
    e = launch_ns_h2_split(reinterpret_cast<const PrepDesc*>(ws + dl.off_prep), count, prep_tiles, st);
    if (e != hipSuccess) return hip_fail(e, "split launch");
    const bool split = std::any_of(P.split.begin(), P.split.end(), [](int f) { return f > 1; });
    int sum_blocks = 0;
    for (const NsPlan& p : P.ns) {
      const int tr = int((p.r_pad + P.tile[0] - 1) / P.tile[0]);
      sum_blocks += tr * (tr + 1) / 2 * (P.tile[0] / 16);
    }
    const std::vector<NsH2Exponents> hs = h2_exponents(coeffs, steps);
    for (int k = 0; k < steps; ++k) {
      const NsH2Exponents* he = hs.empty() ? nullptr : &hs[size_t(k)];
      const float ca = float(coeffs[3 * k]), cb = float(coeffs[3 * k + 1]), cc = float(coeffs[3 * k + 2]);
      const int par = k & 1;
      for (int ph = 0; ph < 3 && e == hipSuccess; ++ph) {
        const int product = ph == 2 && k == steps - 1 ? 3 : ph;
        e = launch_ns_h2(descs(ph), count, P.tiles[ph], product, par, ca, cb, cc, he, P.tile[ph], st);
        if (e == hipSuccess && ph == 0 && split) e = launch_ns_h2_sum(descs(0), count, sum_blocks, par, he, P.tile[0], st);
      }
      if (e != hipSuccess) return hip_fail(e, "NS GEMM launch");
    }
  }
  for (int k = 0; ns_dtype == MFSDP_BF16 && k < steps; ++k) {
    for (int ph = 0; ph < 3; ++ph) {
      // the last update applies the parameter update in its epilogue (kind 3)
      const int kind = ph == 2 && k == steps - 1 ? 3 : ph;
      e = launch_gemm(descs(ph), P.tiles[ph], reinterpret_cast<const TileRef*>(ws + dl.off_sched[ph]), dl.ngroups[ph],
                      kind, k & 1, k == 0 ? 1 : 0, k == steps - 1 ? 1 : 0, float(coeffs[3 * k]),
                      float(coeffs[3 * k + 1]), float(coeffs[3 * k + 2]), P.tile[ph], st);
      if (e != hipSuccess) return hip_fail(e, "NS GEMM launch");
      if (ph == 0 && dl.njobs > 0) {
        e = launch_gram_sum(descs(0), reinterpret_cast<const TileRef*>(ws + dl.off_jobs), dl.njobs, k & 1,
                            k == 0 ? 1 : 0, P.tile[0], st);
        if (e != hipSuccess) return hip_fail(e, "split Gram sum launch");
      }
    }
  }
  if ((rc = record(events, 2, st))) return rc;
  if (!apply_fused(steps)) {
    e = launch_apply(reinterpret_cast<const ApplyDesc*>(ws + dl.off_apply), count, apply_tiles,
                     ns_dtype, st);
    if (e != hipSuccess) return hip_fail(e, "apply launch");
  }
  return record(events, 3, st);
}

int ns_impl(const void* x, int32_t x_dtype, void* out, int32_t out_dtype, int64_t m, int64_t n,
            const double* coeffs, int32_t steps, double eps, int32_t ns_dtype, void* workspace,
            size_t workspace_bytes, void* stream);

// The fused owner-side gradient reduction of mfsdp_muon_step_reduce (validated).
struct ReduceArgs {
  const void* const* parts;  // count * nparts device pointers
  int nparts;
  double scale;
  void* const* out;          // NULL or count pointers (each may be NULL)
};
int muon_impl(const mfsdp_muon_entry* entries, int64_t count, const mfsdp_muon_hparams* hp,
              void* workspace, size_t workspace_bytes, void* stream, void* const* events,
              const ReduceArgs* ra, bool in_scratch = false);

}  // namespace

extern "C" {

int mfsdp_abi_version(void) { return MFSDP_ABI_VERSION; }

#ifndef MFSDP_BUILD_ID
#define MFSDP_BUILD_ID "unknown"
#endif
const char* mfsdp_build_id(void) { return MFSDP_BUILD_ID; }

const char* mfsdp_last_error(void) { return g_last_error.c_str(); }

const char* mfsdp_status_string(int status) {
  switch (status) {
    case MFSDP_OK: return "MFSDP_OK";
    case MFSDP_E_INVALID: return "MFSDP_E_INVALID";
    case MFSDP_E_WORKSPACE: return "MFSDP_E_WORKSPACE";
    case MFSDP_E_HIP: return "MFSDP_E_HIP";
    default: return "MFSDP_E_UNKNOWN";
  }
}

size_t mfsdp_muon_workspace_size(const mfsdp_muon_entry* entries, int64_t count,
                                 const mfsdp_muon_hparams* hp) {
  g_last_error.clear();
  if (check_hp(hp) || check_entries(entries, count, false)) return 0;
  if (count == 0) return 0;
  return make_plan(count, hp->ns_dtype, [&](int64_t i, int64_t& m, int64_t& n) {
           m = entries[i].m;
           n = entries[i].n;
         }).bytes;
}

int mfsdp_muon_step(const mfsdp_muon_entry* entries, int64_t count, const mfsdp_muon_hparams* hp,
                    void* workspace, size_t workspace_bytes, void* stream) {
  return mfsdp_muon_step_timed(entries, count, hp, workspace, workspace_bytes, stream, nullptr);
}

int mfsdp_muon_step_timed(const mfsdp_muon_entry* entries, int64_t count,
                          const mfsdp_muon_hparams* hp, void* workspace, size_t workspace_bytes,
                          void* stream, void* const* events) {
  g_last_error.clear();
  return muon_impl(entries, count, hp, workspace, workspace_bytes, stream, events, nullptr);
}

int mfsdp_muon_step_reduce(const mfsdp_muon_entry* entries, int64_t count,
                           const void* const* grad_parts, int32_t nparts, double grad_scale,
                           void* const* reduced_out, const mfsdp_muon_hparams* hp, void* workspace,
                           size_t workspace_bytes, void* stream) {
  g_last_error.clear();
  if (nparts < 1 || nparts > MFSDP_MAX_GRAD_PARTS)
    return fail(MFSDP_E_INVALID, "nparts must be in [1, %d]", MFSDP_MAX_GRAD_PARTS);
  if (!std::isfinite(grad_scale)) return fail(MFSDP_E_INVALID, "grad_scale must be finite");
  if (count > 0 && !grad_parts) return fail(MFSDP_E_INVALID, "grad_parts is NULL");
  for (int64_t i = 0; i < count; ++i) {
    for (int w = 0; w < nparts; ++w) {
      const void* pw = grad_parts[i * nparts + w];
      if (!pw || !aligned16(pw))
        return fail(MFSDP_E_INVALID, "entry %lld part %d: NULL or not 16-byte aligned", (long long)i, w);
    }
    if (reduced_out && reduced_out[i] && !aligned16(reduced_out[i]))
      return fail(MFSDP_E_INVALID, "entry %lld: reduced_out not 16-byte aligned", (long long)i);
  }
  const ReduceArgs ra{grad_parts, nparts, grad_scale, reduced_out};
  return muon_impl(entries, count, hp, workspace, workspace_bytes, stream, nullptr, &ra);
}

}  // extern "C"

namespace {

int scratch_address(void** out);

// in_scratch: the allocation-free step. The workspace is this device's static scratch array
// (`workspace` and `workspace_bytes` are ignored) and the descriptors travel as kernel arguments
// from ordinary host memory instead of through the pinned staging ring.
int muon_impl(const mfsdp_muon_entry* entries, int64_t count, const mfsdp_muon_hparams* hp,
              void* workspace, size_t workspace_bytes, void* stream, void* const* events,
              const ReduceArgs* ra, bool in_scratch) {
  int rc = check_hp(hp);
  if (rc) return rc;
  rc = check_entries(entries, count, ra == nullptr);
  if (rc) return rc;
  if (count == 0) return MFSDP_OK;
  const Plan P = make_plan(count, hp->ns_dtype, [&](int64_t i, int64_t& m, int64_t& n) {
    m = entries[i].m;
    n = entries[i].n;
  }, in_scratch);
  const std::vector<NsPlan>& plans = P.ns;
  const size_t need = P.bytes;
  if (in_scratch) {
    if (need > size_t(MFSDP_NOALLOC_SCRATCH_BYTES))
      return fail(MFSDP_E_INVALID,
                  "these entries need %zu bytes of workspace; the allocation-free step holds at most "
                  "%zu (MFSDP_NOALLOC_SCRATCH_BYTES): use mfsdp_muon_step with a caller workspace",
                  need, size_t(MFSDP_NOALLOC_SCRATCH_BYTES));
    if ((rc = scratch_address(&workspace))) return rc;
    workspace_bytes = MFSDP_NOALLOC_SCRATCH_BYTES;
  }
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) % kAlign) != 0)
    return fail(MFSDP_E_WORKSPACE, "workspace must be non-NULL and 256-byte aligned");
  if (workspace_bytes < need)
    return fail(MFSDP_E_WORKSPACE, "workspace too small: %zu < %zu bytes", workspace_bytes, need);

  hipStream_t st = static_cast<hipStream_t>(stream);
  uint8_t* ws = static_cast<uint8_t*>(workspace);
  const DescLayout& dl = P.dl;
  int slot = -1;
  std::vector<uint8_t> host_descs;
  uint8_t* h = nullptr;
  if (in_scratch) {
    host_descs.assign(dl.bytes, 0);
    h = host_descs.data();
  } else {
    void* hptr = nullptr;
    slot = ring().acquire(dl.bytes, &hptr, st);
    if (slot < 0) return slot;
    h = static_cast<uint8_t*>(hptr);
    std::memset(h, 0, dl.bytes);
  }

  auto* prep = reinterpret_cast<PrepDesc*>(h + dl.off_prep);
  auto* norm = reinterpret_cast<NormDesc*>(h + dl.off_norm);
  auto* apply = reinterpret_cast<ApplyDesc*>(h + dl.off_apply);
  int prep_tiles = 0, apply_tiles = 0;
  for (int64_t i = 0; i < count; ++i) {
    const mfsdp_muon_entry& en = entries[i];
    const NsPlan& p = plans[i];
    prep[i] = make_prep(p, ws, en.grad, en.grad_dtype, en.momentum, prep_tiles);
    if (ra) {
      prep[i].nparts = ra->nparts;
      prep[i].gscale = float(ra->scale);
      prep[i].gout = ra->out ? ra->out[i] : nullptr;
      for (int w = 0; w < ra->nparts; ++w) prep[i].parts[w] = ra->parts[i * ra->nparts + w];
    }
    prep_tiles += p.prep_tiles_m * p.prep_tiles_n;
    norm[i].partials = reinterpret_cast<const float*>(ws + p.off_partials);
    norm[i].count = p.prep_tiles_m * p.prep_tiles_n;
    norm[i].scale = reinterpret_cast<float*>(ws + p.off_scale);
    const double f = lr_factor(en.m, en.n, hp->lr_adjust);
    apply[i] = make_apply(p, ws, hp->ns_steps, en.param, en.param_dtype, en.update_out, 0,
                          float(1.0 - hp->lr * hp->weight_decay), float(hp->lr * f), apply_tiles);
    apply_tiles += apply[i].tiles_m * apply[i].tiles_n;
  }
  fill_gemm_descs(P, ws, *hp, h);
  const std::vector<double> coeffs = step_coeffs(hp->a, hp->b, hp->c, hp->ns_steps, hp->ns_schedule);
  return enqueue_pipeline(P, ws, slot, hp->ns_steps, coeffs.data(), hp->ns_dtype, hp->momentum,
                          hp->nesterov, hp->eps, prep_tiles, apply_tiles, st, events, ra != nullptr,
                          h);
}

}  // namespace

extern "C" {

size_t mfsdp_ns_workspace_size(int64_t m, int64_t n, int32_t ns_dtype) {
  g_last_error.clear();
  if (!valid_dtype(ns_dtype)) { fail(MFSDP_E_INVALID, "unknown ns_dtype %d", ns_dtype); return 0; }
  if (check_shape(m, n, "matrix", 0)) return 0;
  return make_plan(1, ns_dtype, [&](int64_t, int64_t& mm, int64_t& nn) { mm = m; nn = n; }).bytes;
}

int mfsdp_newton_schulz(const void* x, int32_t x_dtype, void* out, int32_t out_dtype, int64_t m,
                        int64_t n, double a, double b, double c, int32_t steps, double eps,
                        int32_t ns_dtype, void* workspace, size_t workspace_bytes, void* stream) {
  g_last_error.clear();
  if (!std::isfinite(a) || !std::isfinite(b) || !std::isfinite(c))
    return fail(MFSDP_E_INVALID, "NS coefficients must be finite");
  if (steps < 0 || steps >= 100) return fail(MFSDP_E_INVALID, "steps must be in [0, 100)");
  const std::vector<double> coeffs = step_coeffs(a, b, c, steps, nullptr);
  return ns_impl(x, x_dtype, out, out_dtype, m, n, coeffs.data(), steps, eps, ns_dtype, workspace,
                 workspace_bytes, stream);
}

int mfsdp_newton_schulz_schedule(const void* x, int32_t x_dtype, void* out, int32_t out_dtype,
                                 int64_t m, int64_t n, const double* coeffs, int32_t steps,
                                 double eps, int32_t ns_dtype, void* workspace,
                                 size_t workspace_bytes, void* stream) {
  g_last_error.clear();
  if (steps < 0 || steps >= 100) return fail(MFSDP_E_INVALID, "steps must be in [0, 100)");
  if (steps > 0 && !coeffs) return fail(MFSDP_E_INVALID, "coeffs is NULL");
  for (int i = 0; i < 3 * steps; ++i)
    if (!std::isfinite(coeffs[i])) return fail(MFSDP_E_INVALID, "coeffs entry %d is not finite", i);
  return ns_impl(x, x_dtype, out, out_dtype, m, n, coeffs, steps, eps, ns_dtype, workspace,
                 workspace_bytes, stream);
}

}  // extern "C"

namespace {

// Standalone NS: prep in copy mode (no momentum), the NS products, the output written by the last
// update (bf16) or by the apply pass. coeffs: 3 * steps validated doubles.
int ns_impl(const void* x, int32_t x_dtype, void* out, int32_t out_dtype, int64_t m, int64_t n,
            const double* coeffs, int32_t steps, double eps, int32_t ns_dtype, void* workspace,
            size_t workspace_bytes, void* stream) {
  if (!x || !out) return fail(MFSDP_E_INVALID, "x and out must be non-NULL");
  if (x == out) return fail(MFSDP_E_INVALID, "out must not alias x");
  if (!valid_dtype(x_dtype) || !valid_dtype(out_dtype) || !valid_dtype(ns_dtype))
    return fail(MFSDP_E_INVALID, "unsupported dtype");
  int rc = check_shape(m, n, "matrix", 0);
  if (rc) return rc;
  if (!aligned16(x) || !aligned16(out)) return fail(MFSDP_E_INVALID, "pointers must be 16-byte aligned");
  if (!(eps > 0.0) || !std::isfinite(eps)) return fail(MFSDP_E_INVALID, "eps must be > 0");
  const Plan P = make_plan(1, ns_dtype, [&](int64_t, int64_t& mm, int64_t& nn) { mm = m; nn = n; });
  const DescLayout& dl = P.dl;
  const std::vector<NsPlan>& plans = P.ns;
  const size_t need = P.bytes;
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) % kAlign) != 0)
    return fail(MFSDP_E_WORKSPACE, "workspace must be non-NULL and 256-byte aligned");
  if (workspace_bytes < need)
    return fail(MFSDP_E_WORKSPACE, "workspace too small: %zu < %zu bytes", workspace_bytes, need);

  hipStream_t st = static_cast<hipStream_t>(stream);
  uint8_t* ws = static_cast<uint8_t*>(workspace);
  void* hptr = nullptr;
  const int slot = ring().acquire(dl.bytes, &hptr, st);
  if (slot < 0) return slot;
  uint8_t* h = static_cast<uint8_t*>(hptr);
  std::memset(h, 0, dl.bytes);
  const NsPlan& p = plans[0];
  auto* prep = reinterpret_cast<PrepDesc*>(h + dl.off_prep);
  auto* norm = reinterpret_cast<NormDesc*>(h + dl.off_norm);
  auto* apply = reinterpret_cast<ApplyDesc*>(h + dl.off_apply);
  prep[0] = make_prep(p, ws, x, x_dtype, nullptr, 0);
  norm[0].partials = reinterpret_cast<const float*>(ws + p.off_partials);
  norm[0].count = p.prep_tiles_m * p.prep_tiles_n;
  norm[0].scale = reinterpret_cast<float*>(ws + p.off_scale);
  apply[0] = make_apply(p, ws, steps, out, out_dtype, nullptr, 1, 1.0f, 0.0f, 0);
  mfsdp_muon_hparams hp{};
  hp.ns_steps = steps;
  hp.ns_dtype = ns_dtype;
  fill_gemm_descs(P, ws, hp, h);
  return enqueue_pipeline(P, ws, slot, steps, coeffs, ns_dtype, 0.0, 0, eps,
                          p.prep_tiles_m * p.prep_tiles_n, apply[0].tiles_m * apply[0].tiles_n, st,
                          nullptr);
}

}  // namespace

extern "C" {

int mfsdp_adamw_step(const mfsdp_adamw_entry* entries, int64_t count, double lr, double beta1,
                     double beta2, double eps, double weight_decay, int64_t step, void* stream) {
  g_last_error.clear();
  if (count < 0) return fail(MFSDP_E_INVALID, "count must be >= 0");
  if (count > 0 && !entries) return fail(MFSDP_E_INVALID, "entries is NULL");
  if (!(lr >= 0.0) || !std::isfinite(lr)) return fail(MFSDP_E_INVALID, "lr must be >= 0");
  if (!(weight_decay >= 0.0) || !std::isfinite(weight_decay))
    return fail(MFSDP_E_INVALID, "weight_decay must be >= 0");
  if (!(beta1 >= 0.0 && beta1 < 1.0) || !(beta2 >= 0.0 && beta2 < 1.0))
    return fail(MFSDP_E_INVALID, "betas must be in [0, 1)");
  if (!(eps > 0.0) || !std::isfinite(eps)) return fail(MFSDP_E_INVALID, "eps must be > 0");
  if (step < 1) return fail(MFSDP_E_INVALID, "step must be >= 1");
  for (int64_t i = 0; i < count; ++i) {
    const mfsdp_adamw_entry& e = entries[i];
    if (!e.param || !e.grad || !e.exp_avg || !e.exp_avg_sq)
      return fail(MFSDP_E_INVALID, "entry %lld: NULL pointer", (long long)i);
    if (e.numel <= 0) return fail(MFSDP_E_INVALID, "entry %lld: numel must be positive", (long long)i);
    if (e.numel > (int64_t(1) << 40)) return fail(MFSDP_E_INVALID, "entry %lld: numel too large", (long long)i);
    if (!valid_dtype(e.param_dtype) || !valid_dtype(e.grad_dtype))
      return fail(MFSDP_E_INVALID, "entry %lld: unsupported dtype", (long long)i);
    if (!aligned16(e.param) || !aligned16(e.grad) || !aligned16(e.exp_avg) || !aligned16(e.exp_avg_sq))
      return fail(MFSDP_E_INVALID, "entry %lld: pointers must be 16-byte aligned", (long long)i);
  }
  if (count == 0) return MFSDP_OK;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const double bc1 = 1.0 - std::pow(beta1, double(step));
  const double bc2 = 1.0 - std::pow(beta2, double(step));
  AdamWBatch batch{};
  batch.decay = float(1.0 - lr * weight_decay);
  batch.beta1 = float(beta1);
  batch.beta2 = float(beta2);
  batch.omb1 = float(1.0 - beta1);
  batch.omb2 = float(1.0 - beta2);
  batch.step_size = float(lr / bc1);
  batch.inv_sqrt_bc2 = float(1.0 / std::sqrt(bc2));
  batch.eps = float(eps);
  int64_t i = 0;
  while (i < count) {
    batch.count = 0;
    int64_t blocks = 0;
    // one launch per group of up to kAdamWMaxPerLaunch tensors; grid kept below 2^31 blocks
    while (i < count && batch.count < kAdamWMaxPerLaunch) {
      const int64_t nb = (entries[i].numel + kAdamWBlockElems - 1) / kAdamWBlockElems;
      if (batch.count > 0 && blocks + nb > (int64_t(1) << 30)) break;
      AdamWDesc& d = batch.d[batch.count++];
      d.param = entries[i].param;
      d.grad = entries[i].grad;
      d.exp_avg = entries[i].exp_avg;
      d.exp_avg_sq = entries[i].exp_avg_sq;
      d.numel = entries[i].numel;
      d.param_dtype = entries[i].param_dtype;
      d.grad_dtype = entries[i].grad_dtype;
      d.block_begin = int32_t(blocks);
      blocks += nb;
      ++i;
    }
    hipError_t e = launch_adamw(batch, int(blocks), st);
    if (e != hipSuccess) return hip_fail(e, "AdamW launch");
  }
  return MFSDP_OK;
}

}  // extern "C"

// ---------------------------------------------------------------------------------------------
// Allocation-free Muon step (mfsdp_muon_step_noalloc): its workspace is this static device array,
// one copy per GPU the library runs on, held until the process ends. In host code `scratch` is
// only a host-side stand-in for the symbol; the device address of each GPU's copy comes from
// hipGetSymbolAddress, looked up once per device with that device current and cached here, and
// only that address is handed to kernels. Every call on one GPU shares that GPU's copy.
static __device__ __align__(256) uint8_t scratch[MFSDP_NOALLOC_SCRATCH_BYTES];

namespace {

constexpr int kMaxScratchDevices = 256;
std::mutex g_scratch_mu;
void* g_scratch_dev[kMaxScratchDevices] = {};

// Device address of the current device's scratch array (looked up on the first call per device).
int scratch_address(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  if (dev < 0 || dev >= kMaxScratchDevices)
    return fail(MFSDP_E_HIP, "device ordinal %d outside [0, %d)", dev, kMaxScratchDevices);
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_dev[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
    if (!p || (reinterpret_cast<uintptr_t>(p) % kAlign) != 0)
      return fail(MFSDP_E_HIP, "scratch array of device %d is not 256-byte aligned", dev);
    g_scratch_dev[dev] = p;
  }
  *out = g_scratch_dev[dev];
  return MFSDP_OK;
}

// Descriptor bytes handed over as kernel arguments, one launch per chunk (vector stores only).
constexpr int kArgChunkWords = 448;  // 1792 bytes of payload per launch
struct ArgChunk {
  uint32_t w[kArgChunkWords];
  uint32_t words;
};

__global__ __launch_bounds__(256) void arg_copy_kernel(ArgChunk c, uint32_t* __restrict__ dst) {
  for (uint32_t i = threadIdx.x; i < c.words; i += blockDim.x) dst[i] = c.w[i];
}

int upload_as_kernel_args(const uint8_t* host, size_t bytes, uint8_t* dst, hipStream_t st) {
  if (bytes % 4) return fail(MFSDP_E_INVALID, "descriptor region of %zu bytes is not whole words", bytes);
  const size_t words = bytes / 4;
  for (size_t w0 = 0; w0 < words; w0 += kArgChunkWords) {
    ArgChunk c;
    c.words = uint32_t(std::min<size_t>(kArgChunkWords, words - w0));
    std::memcpy(c.w, host + 4 * w0, 4 * size_t(c.words));
    hipLaunchKernelGGL(arg_copy_kernel, dim3(1), dim3(256), 0, st, c,
                       reinterpret_cast<uint32_t*>(dst + 4 * w0));
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "descriptor launch");
  }
  return MFSDP_OK;
}

}  // namespace

extern "C" int mfsdp_muon_step_noalloc(const mfsdp_muon_entry* entries, int64_t count,
                                       const mfsdp_muon_hparams* hp, void* stream) {
  g_last_error.clear();
  return muon_impl(entries, count, hp, nullptr, 0, stream, nullptr, nullptr, true);
}

namespace mfsdp {
// Descriptor staging shared with the other host modules of the library.
int staging_acquire(size_t bytes, void** host) { return ring().acquire(bytes, host, nullptr); }
int staging_upload(int slot, void* dst, size_t bytes, hipStream_t st) {
  return ring().upload(slot, dst, bytes, st);
}

// One auxiliary stream per device (default priority, non-blocking) and a ring of events for the
// fork / join dependencies between it and the caller's stream, created on first use and kept until
// the process ends. An event may be recorded again while an earlier wait on it is still pending: a
// wait takes the record that precedes it on the host. Record and wait are one step under the lock, so that
// no other thread records the event between them.
namespace {
struct AuxState {
  hipStream_t stream = nullptr;
  hipEvent_t events[8] = {};
  unsigned next = 0;
};
std::mutex g_aux_mu;
std::vector<AuxState> g_aux;
}  // namespace

int aux_order(bool fork, hipStream_t main_st, hipStream_t* aux) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  std::lock_guard<std::mutex> lk(g_aux_mu);
  if (dev >= int(g_aux.size())) g_aux.resize(size_t(dev) + 1);
  AuxState& a = g_aux[size_t(dev)];
  if (!a.stream) {
    e = hipStreamCreateWithFlags(&a.stream, hipStreamNonBlocking);
    if (e != hipSuccess) {
      a.stream = nullptr;
      return hip_fail(e, "hipStreamCreateWithFlags");
    }
  }
  hipEvent_t& ev = a.events[a.next++ % 8];
  if (!ev) {
    e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
    if (e != hipSuccess) {
      ev = nullptr;
      return hip_fail(e, "hipEventCreateWithFlags");
    }
  }
  *aux = a.stream;
  e = hipEventRecord(ev, fork ? main_st : a.stream);
  if (e == hipSuccess) e = hipStreamWaitEvent(fork ? a.stream : main_st, ev, 0);
  return e == hipSuccess ? MFSDP_OK : hip_fail(e, "stream fork / join");
}
}  // namespace mfsdp
