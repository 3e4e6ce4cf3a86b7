// Batched persistent form: PageRank on many graphs of uneven size (each with
// its own TOCAB pull partition) and personalised PageRank for up to 64
// one-hot seed vectors on one graph, all iterations in ONE kernel launch.
//
// The grid holds at most as many work-groups as the GPU keeps resident, and
// no more than a phase has items; every phase hands out work items (pull
// tiles, merge ranges, PPR row runs, dangling reductions) by striding over
// one flat item space built from per-graph prefix tables. An iteration has
// two phases (pull, then merge), each ended by a grid barrier; dangling
// totals are added inside the phase before the one that reads them. A
// barrier that waits longer than a spin limit sets an error flag that makes
// every work-group leave, so the launch always ends. Nothing is allocated
// and no host synchronisation happens inside batch_run, so it can be
// captured into a HIP graph (batch_capture / batch_launch).

#include <algorithm>
#include <vector>

#include "gc_internal.h"
#include "gc_pr_device.h"

namespace {

constexpr int kBatchK = 1024;   // merge range of batched partitions
constexpr int kPprLanes = 64;   // one lane per seed vector
constexpr int kPprRows = 32;    // rows per PPR start item (8 per wave)
// Weight (in-arcs, and kPprRowCost per row finished) a PPR unit is cut at: a
// wave each, kWaves units per item. Between the two bounds it is chosen so
// that every wave the grid may hold has about two units: with 2048 arcs per
// unit a graph of 1.6 M arcs kept 780 of 3000 waves busy, each 130 dependent
// gathers deep.
constexpr int32_t kPprUnitMin = 128, kPprUnitMax = 2048;
constexpr int32_t kPprRowCost = 4;
constexpr int kWaves = kThreads / kWave;
constexpr int kPprBatch = 16;   // 256-byte row gathers a wave keeps in flight
constexpr unsigned long long kSpinLimit = 1ull << 21;

struct BGraph {
  int32_t n, n_tiles, R, B;
  const int32_t* rowptr;     // out-arc CSR offsets (out-degrees)
  const int32_t* row_ptr;    // partition
  const int32_t* col;
  const int32_t* tile_row;
  const int32_t* range_ptr;
  const uint16_t* id16;
  float* partial;
  float* contrib;
  double* dpart;             // >= max(ceil(n/256), R) slots
  double* dtotal;            // [2]
  int64_t rank_off;
};

// Personalised PageRank of up to 64 seeds, lane q of a wave = seed q. An
// iteration gathers, per in-arc u -> v, the 256-byte row c[u][0..64) of the
// current contributions. The rows are cut into units of about equal weight,
// one wave each (rather than handed out one by one), so every wave keeps
// kPprBatch gathers in flight: a run of whole rows, or a piece of one long
// row, which leaves its FP64 sum for the next phase to add up.
struct PprUnit {
  int32_t a0, a1;  // in-arcs
  int32_t r0, r1;  // rows [r0, r1), or (r0 < 0) piece ~r0 of a long row
};
struct PprLong {
  int32_t row, p0, p1;  // pieces [p0, p1)
};
struct BPpr {
  int32_t n, S;
  int32_t init_items;         // start items: kPprRows rows each
  int32_t n_units, items;     // pull items: kWaves units each
  int32_t n_long, fix_items;  // long rows; finishing items: kWaves rows each
  const int32_t* t_rowptr;
  const int32_t* t_col;
  const int32_t* rowptr;
  const int32_t* seeds;      // [S]
  const PprUnit* units;
  const PprLong* longs;
  float* c[2];               // [n][64]
  double* piece;             // [pieces][64]
  double* dpart;             // [max(init_items, items)][64]: dangling mass of the start / pull items
  double* dfix[2];           // [fix_items][64]: of the finishing items, iterations in turn
  double* dsum;              // [2][64]: dpart's total
};

struct BatchArgs {
  const BGraph* graphs;
  int32_t G;
  const int32_t* tile_pre;   // [G+1] prefix of tiles
  const int32_t* range_pre;  // [G+1] prefix of merge ranges
  const int32_t* vert_pre;   // [G+1] prefix of 256-vertex init items
  BPpr ppr;
  int32_t has_ppr;
  double damping;
  int32_t iters;
  const float* rank_in;
  float* rank_out;
  float* ppr_out;            // [n][S]
  struct GridBar* bar;
  int32_t* err;
};

// State of the grid barrier, zeroed before every launch; one word per
// 128-byte line.
constexpr int kBarXcds = 16, kBarLine = 32;
struct GridBar {
  unsigned members[kBarXcds * kBarLine];  // work-groups on each XCD
  unsigned arrived[kBarXcds * kBarLine];  // of them, arrivals so far
  unsigned passed[kBarXcds * kBarLine];   // barriers the XCD has left
  unsigned xcds[kBarLine], ready[kBarLine];
  unsigned root[kBarLine], gen[kBarLine];  // XCD arrivals so far, barriers done
};

// What a work-group knows of the barrier: its XCD, the work-groups there, the
// XCDs in use, and the barriers passed.
struct BarSelf {
  unsigned xcd, members, xcds, n;
};

// Item -> (graph, local index) by binary search in a prefix table.
__device__ __forceinline__ int32_t which(const int32_t* pre, int32_t G, int32_t item) {
  int32_t lo = 0, hi = G - 1;
  while (lo < hi) {
    const int32_t mid = (lo + hi + 1) >> 1;
    if (pre[mid] <= item) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

__device__ __forceinline__ unsigned bar_load(const unsigned* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned bar_add(unsigned* p) {
  return __hip_atomic_fetch_add(p, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Waits (one thread) until *p reaches `target`; false after the spin limit
// or when another work-group gave up.
__device__ bool bar_wait(const BatchArgs& a, const unsigned* p, unsigned target) {
  unsigned long long spins = 0;
  while (bar_load(p) < target) {
    if (++spins > kSpinLimit || __hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
      atomicExch(a.err, 1);
      return false;
    }
    __builtin_amdgcn_s_sleep(1);
  }
  return true;
}

// Joins the barrier: counts the work-groups of each XCD (the hardware
// register names the one this work-group runs on, for all of its life).
__device__ bool grid_join(const BatchArgs& a, BarSelf* self) {
  __shared__ BarSelf sh;
  __shared__ int ok;
  if (threadIdx.x == 0) {
    constexpr int kXccId = 20 | ((4 - 1) << 11);  // hardware register XCC_ID, 4 bits from bit 0
    sh.xcd = __builtin_amdgcn_s_getreg(kXccId) & (kBarXcds - 1);
    if (bar_add(&a.bar->members[sh.xcd * kBarLine]) == 0) bar_add(a.bar->xcds);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // counted before this work-group is ready
    bar_add(a.bar->ready);
    ok = bar_wait(a, a.bar->ready, gridDim.x);
    sh.members = bar_load(&a.bar->members[sh.xcd * kBarLine]);
    sh.xcds = bar_load(a.bar->xcds);
    sh.n = 0;
  }
  __syncthreads();
  *self = sh;
  return ok;
}

// Grid barrier. The writes of a work-group are in its XCD's L2 once its
// waves have seen them complete; the last work-group of an XCD to arrive
// writes that L2 back (one release per XCD), then the XCDs meet, and every
// work-group drops its stale lines on the way out. With a release and an
// acquire by each work-group, one after the other in its L2, a barrier of
// 1024 work-groups took 25 us (43 us with two full fences and one counter);
// with one release per XCD it takes 4.6 us at 256 work-groups, 6.9 at 512
// and 9.5 at 768.
__device__ bool grid_sync(const BatchArgs& a, BarSelf* self) {
  __shared__ int ok;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // every wave: its stores have reached the L2
  __syncthreads();
  const unsigned n = ++self->n;
  if (threadIdx.x == 0) {
    const unsigned x = self->xcd * kBarLine;
    bool good;
    if (bar_add(&a.bar->arrived[x]) == n * self->members - 1) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      if (bar_add(a.bar->root) == n * self->xcds - 1)
        __hip_atomic_store(a.bar->gen, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      good = bar_wait(a, a.bar->gen, n);
      __hip_atomic_store(&a.bar->passed[x], n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
      good = bar_wait(a, &a.bar->passed[x], n);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    ok = good;
  }
  __syncthreads();
  return ok;
}

__device__ __forceinline__ Update make_update(const BGraph& g, double d, const double* dtotal, float* rank_out) {
  Update u;
  u.base = (1.0 - d) / g.n;
  u.d = d;
  u.inv_n = 1.0 / g.n;
  u.din = dtotal;
  u.dcount = 1;
  u.dpart = g.dpart;
  u.rowptr = g.rowptr;
  u.contrib = g.contrib;
  u.rank_out = rank_out;
  u.n = g.n;
  return u;
}

// Sum over a work-group of double partials of `count` slots, index order.
__device__ __forceinline__ double sum_slots(const double* p, int32_t count, int32_t stride) {
  double acc = 0.0;
  for (int32_t i = threadIdx.x; i < count; i += kThreads) acc += p[static_cast<int64_t>(i) * stride];
  return wg_sum(acc);
}

// Finishes row v of an iteration from its in-arc sum s (lane = seed):
// writes its next contribution and, on the last iteration, its rank; returns
// its dangling mass (its rank when it has no out-arc).
__device__ __forceinline__ double ppr_finish(const BPpr& p, int32_t v, int32_t deg, double s, int32_t it, double d,
                                             double D, int32_t seed, float* out) {
  const int lane = threadIdx.x & (kWave - 1);
  const double pv = (v == seed) ? 1.0 : 0.0;
  const double r = (1.0 - d) * pv + d * (s + D * pv);
  const float r32 = static_cast<float>(r);
  p.c[(it + 1) & 1][static_cast<int64_t>(v) * kPprLanes + lane] =
      deg ? static_cast<float>(static_cast<double>(r32) / deg) : 0.0f;
  if (out && lane < p.S) out[static_cast<int64_t>(v) * p.S + lane] = r32;
  return deg ? 0.0 : static_cast<double>(r32);
}

// The contributions c[u][lane] of kPprBatch in-arcs from a on (clamped to
// the last before a1).
__device__ __forceinline__ void ppr_gather(const BPpr& p, const float* cur, int32_t a, int32_t a1,
                                           float (&x)[kPprBatch]) {
  const int lane = threadIdx.x & (kWave - 1);
  const int32_t u = p.t_col[min(a + min(lane, kPprBatch - 1), a1 - 1)];
#pragma unroll
  for (int k = 0; k < kPprBatch; ++k)
    x[k] = cur[static_cast<int64_t>(__builtin_amdgcn_readlane(u, k)) * kPprLanes + lane];
}

// One wave takes a unit: it finishes the rows of a run, or leaves the sum of
// a long row's piece. Returns the wave's dangling mass.
__device__ double ppr_unit(const BPpr& p, const PprUnit& q, int32_t it, double d, double D, int32_t seed, float* out) {
  const int lane = threadIdx.x & (kWave - 1);
  const float* cur = p.c[it & 1];
  const bool run = q.r0 >= 0;
  int32_t v = run ? q.r0 : 0;  // current row
  const int32_t last = run ? q.r1 : 0;
  // ends and out-degrees of rows base .. base + 63, one per lane (a load of
  // each row's own where it is finished is a round trip per row: one graph of
  // 200,003 vertices and 8 seeds, 20 iterations, 3154 -> 2998 us)
  int32_t base = v, ends, degs;
  auto load_rows = [&] {
    ends = p.t_rowptr[min(base + 1 + lane, p.n)];
    degs = p.rowptr[min(base + 1 + lane, p.n)] - p.rowptr[min(base + lane, p.n)];
  };
  load_rows();
  auto row_end = [&](int32_t r) {
    if (r - base >= kWave) {
      base = r;
      load_rows();
    }
    return __builtin_amdgcn_readlane(ends, r - base);
  };
  double s = 0.0, dang = 0.0;
  int32_t vend = v < last ? row_end(v) : INT32_MAX;
  // rows that end at or before arc a (empty ones included) are finished
  auto flush_to = [&](int32_t a) {
    while (v < last && vend <= a) {
      dang += ppr_finish(p, v, __builtin_amdgcn_readlane(degs, v - base), s, it, d, D, seed, out);
      s = 0.0;
      ++v;
      vend = v < last ? row_end(v) : INT32_MAX;
    }
  };
  // the next batch's gathers are in flight while one is added
  float x[kPprBatch], y[kPprBatch];
  if (q.a0 < q.a1) ppr_gather(p, cur, q.a0, q.a1, x);  // uniform
  for (int32_t a = q.a0; a < q.a1; a += kPprBatch) {
    ppr_gather(p, cur, min(a + kPprBatch, q.a1 - 1), q.a1, y);
#pragma unroll
    for (int k = 0; k < kPprBatch; ++k) {
      if (a + k < q.a1) {
        flush_to(a + k);
        s += static_cast<double>(x[k]);
      }
    }
#pragma unroll
    for (int k = 0; k < kPprBatch; ++k) x[k] = y[k];
  }
  flush_to(q.a1);
  if (!run) p.piece[static_cast<int64_t>(~q.r0) * kPprLanes + lane] = s;
  return dang;
}

// Writes the work-group's dangling partial (one per seed).
__device__ __forceinline__ void ppr_dangling(double* slot, double mine) {
  __shared__ double dp[kWaves][kPprLanes];
  const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
  dp[wid][lane] = mine;
  __syncthreads();
  if (wid == 0) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) t += dp[w][lane];
    slot[lane] = t;
  }
  __syncthreads();
}

// Dangling mass of the ranks iteration `it` starts from, for this lane's
// seed: the pull (or start) items' total and the finishing items' partials
// of the iteration before.
__device__ double ppr_mass(const BPpr& p, int32_t it) {
  const int lane = threadIdx.x & (kWave - 1);
  double D = p.dsum[(it & 1) * kPprLanes + lane];
  if (it > 0) {
    const double* f = p.dfix[(it - 1) & 1] + lane;
    double t = 0.0;
#pragma unroll 8
    for (int32_t i = 0; i < p.fix_items; ++i) t += f[static_cast<int64_t>(i) * kPprLanes];
    D += t;
  }
  return D;
}

// Pull item: units kWaves * item + wave.
__device__ void ppr_units(const BPpr& p, int32_t item, int32_t it, double d, double D, float* out) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wid = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
  const int32_t seed = lane < p.S ? p.seeds[lane] : -1;
  const int32_t i = item * kWaves + wid;
  double mine = 0.0;
  if (i < p.n_units) mine = ppr_unit(p, p.units[i], it, d, D, seed, out);
  ppr_dangling(p.dpart + static_cast<int64_t>(item) * kPprLanes, mine);
}

// Finishing item (the phase after the pull): long rows, kWaves * item + wave,
// from their pieces.
__device__ void ppr_long_rows(const BPpr& p, int32_t item, int32_t it, double d, double D, float* out) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wid = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
  const int32_t seed = lane < p.S ? p.seeds[lane] : -1;
  const int32_t i = item * kWaves + wid;
  double mine = 0.0;
  if (i < p.n_long) {
    const PprLong l = p.longs[i];
    double s = 0.0;
#pragma unroll 8
    for (int32_t c = l.p0; c < l.p1; ++c) s += p.piece[static_cast<int64_t>(c) * kPprLanes + lane];
    mine = ppr_finish(p, l.row, p.rowptr[l.row + 1] - p.rowptr[l.row], s, it, d, D, seed, out);
  }
  ppr_dangling(p.dfix[it & 1] + static_cast<int64_t>(item) * kPprLanes, mine);
}

// PPR start: r0 = p (one-hot per seed), c0 = r0 / outdeg, dangling partials.
__device__ void ppr_init_rows(const BPpr& p, int32_t item) {
  __shared__ double dp[kThreads / kWave][kPprLanes];
  const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
  const int32_t seed = lane < p.S ? p.seeds[lane] : -1;
  double mine = 0.0;
  const int32_t r0 = item * kPprRows;
  for (int32_t v = r0 + wid; v < min(p.n, r0 + kPprRows); v += kThreads / kWave) {
    const int32_t deg = p.rowptr[v + 1] - p.rowptr[v];
    const float r = (v == seed) ? 1.0f : 0.0f;
    p.c[0][static_cast<int64_t>(v) * kPprLanes + lane] = deg ? r / static_cast<float>(deg) : 0.0f;
    if (!deg) mine += r;
  }
  dp[wid][lane] = mine;
  __syncthreads();
  if (wid == 0) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kThreads / kWave; ++w) t += dp[w][lane];
    p.dpart[static_cast<int64_t>(item) * kPprLanes + lane] = t;
  }
  __syncthreads();
}

__global__ __launch_bounds__(kThreads) void k_batch_reset(GridBar* bar, int32_t* err) {
  unsigned* w = reinterpret_cast<unsigned*>(bar);
  for (int i = threadIdx.x; i < static_cast<int>(sizeof(GridBar) / sizeof(unsigned)); i += kThreads) w[i] = 0u;
  if (threadIdx.x == 0) *err = 0;
}

// Total of a graph's dangling partials.
__device__ __forceinline__ void graph_mass(const BatchArgs& a, int32_t gi, int32_t it) {
  const BGraph& g = a.graphs[gi];
  const double t = sum_slots(g.dpart, it == 0 ? a.vert_pre[gi + 1] - a.vert_pre[gi] : g.R, 1);
  if (threadIdx.x == 0) g.dtotal[it & 1] = t;
}

__global__ __launch_bounds__(kThreads) void k_batch(BatchArgs a) {
  __shared__ float vals[kStageCap];
  __shared__ double acc[kBatchK];
  const int32_t G = a.G;
  const int32_t tiles = G ? a.tile_pre[G] : 0, ranges = G ? a.range_pre[G] : 0, verts = G ? a.vert_pre[G] : 0;
  const int32_t init_items = a.has_ppr ? a.ppr.init_items : 0;
  const int32_t pitems = a.has_ppr ? a.ppr.items : 0;
  const int32_t fitems = a.has_ppr ? a.ppr.fix_items : 0;
  const int32_t lanes = a.has_ppr ? kPprLanes : 0;
  BarSelf bar;
  if (!grid_join(a, &bar)) return;

  // ---- start: contributions of the start vectors and their dangling mass
  for (int32_t item = blockIdx.x; item < verts + init_items; item += gridDim.x) {
    if (item < verts) {
      const int32_t gi = which(a.vert_pre, G, item);
      const BGraph& g = a.graphs[gi];
      const int32_t v = (item - a.vert_pre[gi]) * kThreads + threadIdx.x;
      double mine = 0.0;
      if (v < g.n) {
        const float r = a.rank_in[g.rank_off + v];
        const int32_t deg = g.rowptr[v + 1] - g.rowptr[v];
        g.contrib[v] = deg ? static_cast<float>(static_cast<double>(r) / deg) : 0.0f;
        mine = deg ? 0.0 : static_cast<double>(r);
      }
      const double t = wg_sum(mine);
      if (threadIdx.x == 0) g.dpart[item - a.vert_pre[gi]] = t;
    } else {
      ppr_init_rows(a.ppr, item - verts);
    }
  }
  if (!grid_sync(a, &bar)) return;
  if (a.has_ppr) {  // uniform over the grid
    for (int32_t q = blockIdx.x; q < lanes; q += gridDim.x) {
      const double t = sum_slots(a.ppr.dpart + q, init_items, kPprLanes);
      if (threadIdx.x == 0) a.ppr.dsum[q] = t;
    }
    if (!grid_sync(a, &bar)) return;
  }

  for (int32_t it = 0; it < a.iters; ++it) {
    const bool last = it == a.iters - 1;
    double D = 0.0;  // PPR: the lane's dangling mass
    if (a.has_ppr) D = ppr_mass(a.ppr, it);
    // ---- PPR units, pull tiles of every graph (Algorithm 4), and the
    // dangling totals that the merge phase reads
    for (int32_t item = blockIdx.x; item < pitems + tiles + G; item += gridDim.x) {
      if (item < pitems) {
        ppr_units(a.ppr, item, it, a.damping, D, last ? a.ppr_out : nullptr);
      } else if (item < pitems + tiles) {
        const int32_t x = item - pitems;
        const int32_t gi = which(a.tile_pre, G, x);
        const BGraph& g = a.graphs[gi];
        const int32_t t = x - a.tile_pre[gi];
        const int32_t r0 = g.tile_row[t], r1 = g.tile_row[t + 1];
        if (r0 < r1)
          pull_tile(g.row_ptr, g.col, g.contrib, r0, r1, vals,
                    [&](int32_t r, double s) { g.partial[r] = static_cast<float>(s); });
        __syncthreads();  // vals is reused by the next item
      } else {
        graph_mass(a, item - pitems - tiles, it);
      }
    }
    if (!grid_sync(a, &bar)) return;
    // ---- merge ranges fused with the update (Figure 5), the long PPR rows,
    // and the PPR mass of the pull items for the next iteration
    for (int32_t item = blockIdx.x; item < ranges + fitems + (last ? 0 : lanes); item += gridDim.x) {
      if (item >= ranges + fitems) {
        const int32_t q = item - ranges - fitems;
        const double t = sum_slots(a.ppr.dpart + q, pitems, kPprLanes);
        if (threadIdx.x == 0) a.ppr.dsum[((it + 1) & 1) * kPprLanes + q] = t;
        continue;
      }
      if (item >= ranges) {
        ppr_long_rows(a.ppr, item - ranges, it, a.damping, D, last ? a.ppr_out : nullptr);
        continue;
      }
      const int32_t gi = which(a.range_pre, G, item);
      const BGraph& g = a.graphs[gi];
      const int32_t j = item - a.range_pre[gi];
      merge_accumulate<kBatchK, true>(g.range_ptr, g.B, g.id16, g.partial, j, acc);
      const Update u = make_update(g, a.damping, g.dtotal + (it & 1), last ? a.rank_out + g.rank_off : nullptr);
      const double Dg = g.dtotal[it & 1];
      double mine = 0.0;
      for (int i = threadIdx.x; i < kBatchK; i += kThreads) {
        const int32_t v = j * kBatchK + i;
        if (v < g.n) mine += update_vertex(u, v, acc[i], Dg);
      }
      const double t = wg_sum(mine);
      if (threadIdx.x == 0) g.dpart[j] = t;
      __syncthreads();  // acc is reused by the next item
    }
    if (!last && !grid_sync(a, &bar)) return;
  }
}

}  // namespace

struct gc_batch_s {
  std::vector<gc_graph> graphs;
  std::vector<gc_tocab> parts;
  std::vector<int64_t> rank_off;
  std::vector<int32_t> widths;
  gc_graph ppr_graph = nullptr;
  int32_t n_seeds = 0;
  BatchArgs args{};
  int32_t grid = 0;
  int64_t bytes = 0;
  std::vector<void*> owned;
  int32_t* err_host = nullptr;
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
};

namespace {

int bfail(int code, const char* fmt, const char* what = "") {
  gcx::set_error(fmt, what);
  return code;
}

void* own(gc_batch b, size_t bytes) {
  void* p = gcx::dev_alloc(bytes, nullptr);
  if (p) {
    b->owned.push_back(p);
    b->bytes += static_cast<int64_t>(bytes);
  }
  return p;
}

void destroy(gc_batch b) {
  if (!b) return;
  if (b->exec) (void)hipGraphExecDestroy(b->exec);
  if (b->graph) (void)hipGraphDestroy(b->graph);
  for (gc_tocab t : b->parts) tocab_free(t);
  for (void* p : b->owned) gcx::dev_free(p, nullptr);
  if (b->err_host) (void)hipHostFree(b->err_host);
  delete b;
}

}  // namespace

extern "C" {

int batch_create(const gc_graph* graphs, int32_t n_graphs, const int32_t* block_widths, gc_graph ppr_graph,
                 const int32_t* seeds, int32_t n_seeds, hipStream_t stream, gc_batch* out) {
  if (!out) return bfail(GC_EINVAL, "batch_create: out is NULL");
  *out = nullptr;
  if (n_graphs < 0 || (n_graphs > 0 && !graphs)) return bfail(GC_EINVAL, "batch_create: bad graph list");
  if (n_seeds < 0 || n_seeds > kPprLanes || (n_seeds > 0 && (!ppr_graph || !seeds)))
    return bfail(GC_EINVAL, "batch_create: 0..64 seeds on a graph");
  if (n_graphs == 0 && n_seeds == 0) return bfail(GC_EINVAL, "batch_create: nothing to run");
  for (int32_t i = 0; i < n_graphs; ++i)
    if (!graphs[i]) return bfail(GC_EINVAL, "batch_create: NULL graph");
  for (int32_t q = 0; q < n_seeds; ++q)
    if (seeds[q] < 0 || seeds[q] >= ppr_graph->n) return bfail(GC_EINVAL, "batch_create: seed out of range");
  int32_t resident = 0;  // work-groups the GPU keeps resident
  {
    int per_cu = 0, dev = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess)
      e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(&k_batch), kThreads, 0);
    if (e != hipSuccess || per_cu < 1 || cus < 1) return bfail(GC_EHIP, "batch_create: device query failed");
    resident = per_cu * cus;
  }
  gc_batch b = new (std::nothrow) gc_batch_s;
  if (!b) return bfail(GC_ENOMEM, "batch_create: host allocation failed");
  std::vector<BGraph> hg(n_graphs);
  std::vector<int32_t> tile_pre(n_graphs + 1, 0), range_pre(n_graphs + 1, 0), vert_pre(n_graphs + 1, 0);
  int64_t off = 0;
  for (int32_t i = 0; i < n_graphs; ++i) {
    gc_graph g = graphs[i];
    int32_t W = block_widths ? block_widths[i] : 0;
    if (W == 0) {  // autotuned among widths whose slices stay in the last-level cache
      int32_t k = 0;
      float ms = 0.0f;
      if (gcx::autotune(g, GC_PULL, 1 << 16, &W, &k, &ms, stream) != hipSuccess) {
        destroy(b);
        return bfail(GC_EHIP, "batch_create: autotune failed");
      }
    }
    gc_tocab t = nullptr;
    const int rc = tocab_partition(g, GC_PULL, W, kBatchK, stream, &t);
    if (rc != GC_OK) {
      destroy(b);
      return rc;
    }
    if (t->B > kFlatB || t->col16) {
      tocab_free(t);
      destroy(b);
      return bfail(GC_EUNSUPPORTED, "batch_create: widths below 2^16 or above 1024 blocks are not batched");
    }
    b->parts.push_back(t);
    b->graphs.push_back(g);
    b->widths.push_back(W);
    BGraph& d = hg[i];
    d.n = g->n;
    d.n_tiles = t->n_tiles;
    d.R = t->mR;
    d.B = t->B;
    d.rowptr = g->rowptr;
    d.row_ptr = t->row_ptr;
    d.col = t->col;
    d.tile_row = t->tile_row;
    d.range_ptr = t->mrange;
    d.id16 = t->id16;
    d.partial = t->partial;
    const int32_t vgrid = (g->n + kThreads - 1) / kThreads;
    d.contrib = static_cast<float*>(own(b, sizeof(float) * g->n));
    d.dpart = static_cast<double*>(own(b, sizeof(double) * std::max(vgrid, t->mR)));
    d.dtotal = static_cast<double*>(own(b, sizeof(double) * 2));
    d.rank_off = off;
    if (!d.contrib || !d.dpart || !d.dtotal) {
      destroy(b);
      return bfail(GC_ENOMEM, "batch_create: allocation failed");
    }
    b->rank_off.push_back(off);
    off += g->n;
    tile_pre[i + 1] = tile_pre[i] + t->n_tiles;
    range_pre[i + 1] = range_pre[i] + t->mR;
    vert_pre[i + 1] = vert_pre[i] + vgrid;
  }
  b->rank_off.push_back(off);
  BatchArgs& a = b->args;
  a.G = n_graphs;
  a.has_ppr = n_seeds > 0;
  if (n_seeds > 0) {
    gc_graph pg = ppr_graph;
    b->ppr_graph = pg;
    b->n_seeds = n_seeds;
    BPpr& p = a.ppr;
    p.n = pg->n;
    p.S = n_seeds;
    p.init_items = (pg->n + kPprRows - 1) / kPprRows;
    p.t_rowptr = pg->t_rowptr;
    p.t_col = pg->t_colidx;
    p.rowptr = pg->rowptr;
    // units of whole rows, long rows in pieces
    std::vector<int32_t> trp(static_cast<size_t>(pg->n) + 1);
    if (hipMemcpy(trp.data(), pg->t_rowptr, sizeof(int32_t) * trp.size(), hipMemcpyDeviceToHost) != hipSuccess) {
      destroy(b);
      return bfail(GC_EHIP, "batch_create: copy failed");
    }
    const int64_t weight = pg->m + kPprRowCost * static_cast<int64_t>(pg->n);
    const int32_t unit = static_cast<int32_t>(
        std::min<int64_t>(kPprUnitMax, std::max<int64_t>(kPprUnitMin, weight / (2 * kWaves * std::max(resident, 1)))));
    std::vector<PprUnit> units;
    std::vector<PprLong> longs;
    int32_t pieces = 0;
    for (int32_t v = 0; v < pg->n;) {
      const int32_t a0 = trp[v], len = trp[v + 1] - a0;
      if (len > 2 * unit) {
        const int32_t k = (len + unit - 1) / unit, p0 = pieces;
        for (int32_t i = 0; i < k; ++i)
          units.push_back({a0 + static_cast<int32_t>(static_cast<int64_t>(len) * i / k),
                           a0 + static_cast<int32_t>(static_cast<int64_t>(len) * (i + 1) / k), ~pieces++, 0});
        longs.push_back({v, p0, pieces});
        ++v;
        continue;
      }
      int32_t r = v;
      int64_t w = 0;
      while (r < pg->n && w < unit && trp[r + 1] - trp[r] <= 2 * unit) {
        w += trp[r + 1] - trp[r] + kPprRowCost;
        ++r;
      }
      units.push_back({a0, trp[r], v, r});
      v = r;
    }
    p.n_units = static_cast<int32_t>(units.size());
    p.items = (p.n_units + kWaves - 1) / kWaves;
    p.n_long = static_cast<int32_t>(longs.size());
    p.fix_items = (p.n_long + kWaves - 1) / kWaves;
    const size_t lanes = kPprLanes;
    int32_t* ds = static_cast<int32_t*>(own(b, sizeof(int32_t) * n_seeds));
    PprUnit* du = static_cast<PprUnit*>(own(b, sizeof(PprUnit) * units.size()));
    PprLong* dl = static_cast<PprLong*>(own(b, sizeof(PprLong) * std::max<size_t>(longs.size(), 1)));
    p.c[0] = static_cast<float*>(own(b, sizeof(float) * lanes * static_cast<size_t>(pg->n)));
    p.c[1] = static_cast<float*>(own(b, sizeof(float) * lanes * static_cast<size_t>(pg->n)));
    p.piece = static_cast<double*>(own(b, sizeof(double) * lanes * static_cast<size_t>(std::max(pieces, 1))));
    const size_t slots = static_cast<size_t>(std::max(p.init_items, p.items));
    p.dpart = static_cast<double*>(own(b, sizeof(double) * lanes * slots));
    p.dfix[0] = static_cast<double*>(own(b, sizeof(double) * lanes * static_cast<size_t>(std::max(p.fix_items, 1))));
    p.dfix[1] = static_cast<double*>(own(b, sizeof(double) * lanes * static_cast<size_t>(std::max(p.fix_items, 1))));
    p.dsum = static_cast<double*>(own(b, sizeof(double) * 2 * lanes));
    if (!ds || !du || !dl || !p.c[0] || !p.c[1] || !p.piece || !p.dpart || !p.dfix[0] || !p.dfix[1] || !p.dsum) {
      destroy(b);
      return bfail(GC_ENOMEM, "batch_create: allocation failed");
    }
    if (hipMemcpy(ds, seeds, sizeof(int32_t) * n_seeds, hipMemcpyDefault) != hipSuccess ||
        hipMemcpy(du, units.data(), sizeof(PprUnit) * units.size(), hipMemcpyHostToDevice) != hipSuccess ||
        (!longs.empty() &&
         hipMemcpy(dl, longs.data(), sizeof(PprLong) * longs.size(), hipMemcpyHostToDevice) != hipSuccess)) {
      destroy(b);
      return bfail(GC_EHIP, "batch_create: copy failed");
    }
    p.units = du;
    p.longs = dl;
    p.seeds = ds;
  }
  BGraph* dg = static_cast<BGraph*>(own(b, sizeof(BGraph) * std::max(1, n_graphs)));
  int32_t* pre = static_cast<int32_t*>(own(b, sizeof(int32_t) * 3 * (n_graphs + 1)));
  a.bar = static_cast<GridBar*>(own(b, sizeof(GridBar)));
  a.err = static_cast<int32_t*>(own(b, sizeof(int32_t)));
  if (!dg || !pre || !a.bar || !a.err ||
      hipHostMalloc(reinterpret_cast<void**>(&b->err_host), sizeof(int32_t), hipHostMallocDefault) != hipSuccess) {
    destroy(b);
    return bfail(GC_ENOMEM, "batch_create: allocation failed");
  }
  hipError_t e = hipSuccess;
  if (n_graphs > 0) e = hipMemcpy(dg, hg.data(), sizeof(BGraph) * n_graphs, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(pre, tile_pre.data(), sizeof(int32_t) * (n_graphs + 1), hipMemcpyHostToDevice);
  if (e == hipSuccess)
    e = hipMemcpy(pre + n_graphs + 1, range_pre.data(), sizeof(int32_t) * (n_graphs + 1), hipMemcpyHostToDevice);
  if (e == hipSuccess)
    e = hipMemcpy(pre + 2 * (n_graphs + 1), vert_pre.data(), sizeof(int32_t) * (n_graphs + 1), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    destroy(b);
    return bfail(GC_EHIP, "batch_create: copy failed");
  }
  // every work-group must be live for the grid barrier; no more of them than
  // the largest phase has items (a barrier's cost grows with them)
  const int64_t tiles = tile_pre[n_graphs], ranges = range_pre[n_graphs], verts = vert_pre[n_graphs];
  int64_t most = std::max<int64_t>(tiles + n_graphs, std::max(ranges, verts));
  if (n_seeds > 0)
    most = std::max({static_cast<int64_t>(a.ppr.items) + tiles + n_graphs,
                     ranges + a.ppr.fix_items + kPprLanes, verts + a.ppr.init_items});
  b->grid = static_cast<int32_t>(std::min<int64_t>(resident, most));
  a.graphs = dg;
  a.tile_pre = pre;
  a.range_pre = pre + n_graphs + 1;
  a.vert_pre = pre + 2 * (n_graphs + 1);
  *out = b;
  return GC_OK;
}

int batch_info(gc_batch b, int64_t* rank_offsets, int32_t* block_widths, int32_t* grid, int64_t* bytes) {
  if (!b) return bfail(GC_EINVAL, "batch_info: NULL batch");
  for (size_t i = 0; i < b->rank_off.size() && rank_offsets; ++i) rank_offsets[i] = b->rank_off[i];
  for (size_t i = 0; i < b->widths.size() && block_widths; ++i) block_widths[i] = b->widths[i];
  if (grid) *grid = b->grid;
  if (bytes) *bytes = b->bytes;
  return GC_OK;
}

int batch_run(gc_batch b, float damping, int32_t iters, const float* ranks_in, float* ranks_out, float* ppr_out,
              hipStream_t stream) {
  if (!b) return bfail(GC_EINVAL, "batch_run: NULL batch");
  if (!(damping >= 0.0f && damping <= 1.0f) || iters < 1) return bfail(GC_EINVAL, "batch_run: bad damping or iters");
  if (!b->graphs.empty() && (!ranks_in || !ranks_out)) return bfail(GC_EINVAL, "batch_run: NULL rank buffers");
  if (b->n_seeds > 0 && !ppr_out) return bfail(GC_EINVAL, "batch_run: NULL ppr output");
  BatchArgs a = b->args;
  a.damping = damping;
  a.iters = iters;
  a.rank_in = ranks_in;
  a.rank_out = ranks_out;
  a.ppr_out = ppr_out;
  gcx::ProfScope prof("batch", stream);
  k_batch_reset<<<1, kThreads, 0, stream>>>(a.bar, a.err);
  k_batch<<<b->grid, kThreads, 0, stream>>>(a);
  return hipGetLastError() == hipSuccess ? GC_OK : bfail(GC_EHIP, "batch_run: launch failed");
}

int batch_capture(gc_batch b, float damping, int32_t iters, const float* ranks_in, float* ranks_out, float* ppr_out) {
  if (!b) return bfail(GC_EINVAL, "batch_capture: NULL batch");
  if (b->exec) (void)hipGraphExecDestroy(b->exec);
  if (b->graph) (void)hipGraphDestroy(b->graph);
  b->exec = nullptr;
  b->graph = nullptr;
  hipStream_t cs;
  if (hipStreamCreate(&cs) != hipSuccess) return bfail(GC_EHIP, "batch_capture: stream");
  hipError_t e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
  int rc = GC_OK;
  if (e == hipSuccess) rc = batch_run(b, damping, iters, ranks_in, ranks_out, ppr_out, cs);
  const hipError_t e2 = hipStreamEndCapture(cs, &b->graph);
  if (e == hipSuccess) e = e2;
  if (e == hipSuccess && rc == GC_OK) e = hipGraphInstantiate(&b->exec, b->graph, nullptr, nullptr, 0);
  (void)hipStreamDestroy(cs);
  if (rc != GC_OK) return rc;
  return e == hipSuccess ? GC_OK : bfail(GC_EHIP, "batch_capture: capture failed");
}

int batch_launch(gc_batch b, hipStream_t stream) {
  if (!b || !b->exec) return bfail(GC_EINVAL, "batch_launch: nothing captured");
  gcx::ProfScope prof("batch_graph", stream);
  return hipGraphLaunch(b->exec, stream) == hipSuccess ? GC_OK : bfail(GC_EHIP, "batch_launch: launch failed");
}

int batch_status(gc_batch b, hipStream_t stream, int32_t* barrier_timeout) {
  if (!b || !barrier_timeout) return bfail(GC_EINVAL, "batch_status: bad argument");
  hipError_t e = hipMemcpyAsync(b->err_host, b->args.err, sizeof(int32_t), hipMemcpyDeviceToHost, stream);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  if (e != hipSuccess) return bfail(GC_EHIP, "batch_status: %s", hipGetErrorString(e));
  *barrier_timeout = *b->err_host;
  return GC_OK;
}

int batch_free(gc_batch b) {
  if (!b) return bfail(GC_EINVAL, "batch_free: NULL batch");
  (void)hipDeviceSynchronize();
  destroy(b);
  return GC_OK;
}

}  // extern "C"
