// Traversal on gfx950: BFS and SSSP level by level (Section 3.3).
//
// Frontier state kept by the library, per graph handle:
//   front      status of the current frontier, one bit per vertex (the
//              paper's status array, at n/8 bytes: 2 MB at 2^24 vertices,
//              so the random tests of a pull level stay in one XCD's L2)
//   next       the same for the next level; all zero when a level starts
//              (k_level_end clears the old frontier's)
//   queue      list of the current frontier (size n_f), and the list being
//              filled for the next level
//   visited    bitmap of vertices with a final depth (BFS)
// A level runs in one of three ways:
//   pull  topology-driven over the transposed graph: every unvisited vertex
//         scans its in-arcs for an active source (BFS stops at the first);
//   tocab the same over a GC_PULL partition: each block writes a flag (BFS)
//         or a minimum (SSSP) per local row, and a merge over vertex ranges
//         reduces them, updates depth / dist and builds the next frontier;
//   push  data-driven from the queue: every frontier vertex relaxes its
//         out-arcs with atomics (CAS on depth, atomicMin on dist).
// A push level appends the next frontier to a queue together with the arc
// prefix of its out-degrees, so the next push finds its arcs without a scan of
// its own; a pull level sets status bits. Where a level of one kind follows
// the other, it builds what it needs (a pass over n bits or depths). Both
// count the next frontier's vertices and out-arcs, which the host reads once
// per level from pinned memory that the level's last kernel writes. Counters
// take as few atomics as a launch allows: on one address they cost 25 ns
// each on this GPU, whoever issues them (one per 256 vertices of a pull over
// 2^23 vertices: 0.8 ms).

#include <algorithm>
#include <chrono>
#include <climits>
#include <cmath>
#include <cstring>
#include <vector>

#include "gc_device.h"
#include "gc_internal.h"
#include "gc_mlp.h"
#include "gc_merge.h"
#include "gc_stream.h"

namespace {

using gcd::kWave;
using gcx::Buf;
using gcx::ProfScope;

constexpr int kThreads = 256;
constexpr int32_t kInf = INT32_MAX;

// stats slots (device int32[gcx::kStatSlots], written to the pinned mirror once per level)
constexpr int kOverflow = gcx::kStatOverflow;

// Where a push puts the next frontier: its vertices, each one's first
// position in the concatenation of their out-arcs, and (t_rowptr given) the
// count of their in-arcs. `counter` is the slot of the packed count.
struct Sink {
  int32_t* queue;
  int32_t* pre;
  const int32_t* rowptr;
  const int32_t* t_rowptr;
  int32_t* stats;
  int counter = gcx::kStatArcs;
};

__device__ __forceinline__ uint64_t one_vertex(int32_t deg) { return (1ull << 32) | static_cast<uint32_t>(deg); }

// Adds every thread's vertices, mine = vertices << 32 | their out-arcs, to
// the packed counter (and their in-arcs to theirs), one atomic per
// work-group and counter. With kReserve returns the thread's first position
// and arc, packed alike: both counts live in one 64-bit word, so positions
// and arc prefixes ascend together. Synchronises the work-group: every
// thread must reach each call.
template <int NT, bool kReserve>
__device__ __forceinline__ uint64_t wg_count(uint64_t mine, uint64_t in_arcs, bool with_in, int32_t* stats,
                                             int counter) {
  __shared__ uint64_t tot[NT / kWave], base[NT / kWave], in_tot[NT / kWave];
  const int lane = gcd::lane_id();
  const int wid = threadIdx.x / kWave;
  uint64_t incl = mine;  // inclusive sum over the wave's lanes
  if (__any(mine != 0)) {
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const uint64_t y = __shfl_up(incl, o, kWave);
      if (lane >= o) incl += y;
    }
    if (with_in)  // uniform
      for (int o = 32; o > 0; o >>= 1) in_arcs += __shfl_xor(in_arcs, o, kWave);
  }
  if (lane == kWave - 1) {
    tot[wid] = incl;
    in_tot[wid] = in_arcs;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t t = 0, ti = 0;
    for (int w = 0; w < NT / kWave; ++w) {
      base[w] = t;
      t += tot[w];
      ti += in_tot[w];
    }
    if (t) {
      const uint64_t at = atomicAdd(reinterpret_cast<unsigned long long*>(stats + counter), t);
      if (kReserve)
        for (int w = 0; w < NT / kWave; ++w) base[w] += at;
      if (with_in && ti) atomicAdd(reinterpret_cast<unsigned long long*>(stats + gcx::kStatInDegLo), ti);
    }
  }
  if (!kReserve) return 0;
  __syncthreads();
  return base[wid] + incl - mine;
}

__device__ __forceinline__ void sink_put(const Sink& s, uint64_t at, int32_t v) {
  s.queue[at >> 32] = v;
  s.pre[at >> 32] = static_cast<int32_t>(static_cast<uint32_t>(at));
}

// What a pull counts of the next frontier.
struct Tally {
  const int32_t* rowptr;
  const int32_t* t_rowptr;  // null: in-arcs are not counted
  int32_t* stats;
};

struct Counted {
  uint64_t mine = 0, in = 0;
  __device__ __forceinline__ void add(const Tally& t, int32_t v) {
    mine += one_vertex(t.rowptr[v + 1] - t.rowptr[v]);
    if (t.t_rowptr) in += static_cast<uint64_t>(t.t_rowptr[v + 1] - t.t_rowptr[v]);
  }
};

template <int NT>
__device__ __forceinline__ void publish_count(const Tally& t, const Counted& c) {
  wg_count<NT, false>(c.mine, c.in, t.t_rowptr != nullptr, t.stats, gcx::kStatArcs);
}

__device__ __forceinline__ bool bit_test(const uint32_t* bits, int32_t v) {
  return (bits[v >> 5] >> (v & 31)) & 1u;
}

// Sets bit v in `bits` for the lanes where `take` holds, one atomic per
// 32-bit word: every lane of the wave calls it, and lane l holds vertex
// v0 + l for a v0 that is a multiple of 32 (a wave of consecutive
// vertices). Per-vertex atomics on the few words a wave shares serialise in
// L2 on levels that discover millions of vertices.
__device__ __forceinline__ void wave_bits_set(uint32_t* bits, int32_t v, bool take) {
  const uint64_t m = __ballot(take);
  const int lane = gcd::lane_id();
  const uint32_t word = static_cast<uint32_t>(m >> (lane & 32));
  if ((lane & 31) == 0 && word != 0u) atomicOr(&bits[v >> 5], word);
}

__global__ void k_fill_i32(int32_t* __restrict__ a, int64_t n, int32_t x) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) a[i] = x;
}

// Clears what the next level accumulates.
__device__ __forceinline__ void reset_stats(int32_t* stats) {
  if (gcd::lane_id() < gcx::kStatSeq) stats[gcd::lane_id()] = 0;
  if (gcd::lane_id() < 2) stats[gcx::kStatInDegLo + gcd::lane_id()] = 0;
  if (gcd::lane_id() < 2) stats[gcx::kStatBuild + gcd::lane_id()] = 0;
}

// Writes the level's counters (the first 16 slots and `outs` scheduler
// outputs) and the clock t1 at its end to the pinned mirror, clears them for
// the next level, then writes `seq`, which the host waits for: once it is
// there, the counters are the next user's. One wave.
__device__ __forceinline__ void publish_stats(int32_t* stats, int32_t* host, int32_t seq, int outs, uint64_t t1) {
  for (int i = gcd::lane_id(); i < gcx::kStatOut + outs; i += kWave) {
    int32_t v = __hip_atomic_load(stats + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (i == gcx::kStatT1) v = static_cast<int32_t>(t1);
    if (i == gcx::kStatT1 + 1) v = static_cast<int32_t>(t1 >> 32);
    if (i != gcx::kStatSeq) __hip_atomic_store(host + i, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
  reset_stats(stats);
  // one fence for both (it waits for the stores of all lanes of the wave; a
  // second one between them, or a release here, costs 1.7 us a level)
  __threadfence_system();
  if (gcd::lane_id() == 0)
    __hip_atomic_store(host + gcx::kStatSeq, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Start of a traversal: values (and round stamps, path counts and
// coefficients where given), the frontier {src} and its out-degree for the
// host. Counters and source are handled by the first work-group.
__global__ __launch_bounds__(kThreads) void k_start(int32_t n, int32_t src, const int32_t* __restrict__ rowptr,
                                                    int32_t* __restrict__ value, int32_t* __restrict__ mark,
                                                    double* __restrict__ sigma, double* __restrict__ coef,
                                                    int32_t* __restrict__ queue, int32_t* __restrict__ pre,
                                                    int32_t* __restrict__ stats, int32_t* __restrict__ host,
                                                    int32_t seq) {
  if (blockIdx.x == 0 && threadIdx.x < kWave) {
    if (threadIdx.x == 0) {
      queue[0] = src;
      pre[0] = 0;
      __hip_atomic_store(host + gcx::kStatArcs, rowptr[src + 1] - rowptr[src], __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_SYSTEM);
      __hip_atomic_store(host + gcx::kStatSeq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    reset_stats(stats);
  }
  const int64_t stride = static_cast<int64_t>(gridDim.x) * kThreads;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x; i < n; i += stride) {
    value[i] = i == src ? 0 : kInf;
    if (mark) mark[i] = -1;
    if (sigma) {
      sigma[i] = i == src ? 1.0 : 0.0;
      coef[i] = 0.0;
      coef[n + i] = 0.0;
    }
  }
}

// Status bits of a pull level that follows a push: the frontier (depth ==
// level) and the visited vertices, from the depths.
__global__ __launch_bounds__(kThreads) void k_bits_from_depth(const int32_t* __restrict__ depth, int32_t n,
                                                              int32_t level, uint32_t* __restrict__ front,
                                                              uint32_t* __restrict__ visited) {
  const int64_t v = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
  const int32_t d = v < n ? depth[v] : kInf;
  const uint64_t f = __ballot(d == level), x = __ballot(d != kInf);
  const int lane = gcd::lane_id();
  if ((lane & 31) == 0 && v < n) {
    front[v >> 5] = static_cast<uint32_t>(f >> (lane & 32));
    visited[v >> 5] = static_cast<uint32_t>(x >> (lane & 32));
  }
}

// The same for SSSP, whose frontier is known by its queue alone (front is
// all zero on entry).
__global__ __launch_bounds__(kThreads) void k_bits_from_queue(const int32_t* __restrict__ queue, int32_t qn,
                                                              uint32_t* __restrict__ front) {
  const int32_t i = blockIdx.x * kThreads + threadIdx.x;
  if (i < qn) atomicOr(&front[queue[i] >> 5], 1u << (queue[i] & 31));
}

// The queue of a push level that follows a pull, from the status bits: a
// thread takes kWords words, the queue comes out in vertex order within a
// work-group.
template <int kWords>
__global__ __launch_bounds__(kThreads) void k_queue_from_bits(const uint32_t* __restrict__ front, int64_t words,
                                                              Sink sink) {
  const int64_t w0 = (static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x) * kWords;
  uint32_t bits[kWords];
#pragma unroll
  for (int k = 0; k < kWords; ++k) bits[k] = w0 + k < words ? front[w0 + k] : 0u;
  uint64_t mine = 0;
#pragma unroll
  for (int k = 0; k < kWords; ++k)
    for (uint32_t x = bits[k]; x; x &= x - 1u) {
      const int32_t v = static_cast<int32_t>((w0 + k) << 5) + __ffs(x) - 1;
      mine += one_vertex(sink.rowptr[v + 1] - sink.rowptr[v]);
    }
  uint64_t at = wg_count<kThreads, true>(mine, 0, false, sink.stats, sink.counter);
#pragma unroll
  for (int k = 0; k < kWords; ++k)
    for (uint32_t x = bits[k]; x; x &= x - 1u) {
      const int32_t v = static_cast<int32_t>((w0 + k) << 5) + __ffs(x) - 1;
      sink_put(sink, at, v);
      at += one_vertex(sink.rowptr[v + 1] - sink.rowptr[v]);
    }
}

// Device wall clock at a level's start, by the first thread of each of its
// kernels (the last one that runs first is the level's relaxation kernel).
__device__ __forceinline__ void stamp_start(int32_t* stats) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *reinterpret_cast<uint64_t*>(stats + gcx::kStatT0) = wall_clock64();
}

// What the learned scheduler needs to decide the next level on the device:
// its parameters and the graph's and level's counts.
struct LevelDecide {
  const float* params = nullptr;
  const float* frange = nullptr;
  int32_t K = 0;
  int64_t n = 0, m = 0;
  int32_t level = 0;
  int64_t prior_arcs = 0;
  int32_t clock_khz = 1;
  // the working-set rule's direction test for the next level (the network
  // only picks the form of pull levels, so push levels skip it): its state,
  // and the unexplored arcs before the next frontier's are taken off (BFS)
  // or the whole arc count (SSSP)
  bool pulling = false;
  bool sub_next = false;
  int64_t unexplored = 0;
  double alpha = 0.0, beta = 0.0;
};

// LDS the learned decision needs: the parameters, and W2 again at a pitch
// of one word more than its rows.
size_t level_decide_lds(int32_t K) {
  return sizeof(float) * (static_cast<size_t>(gcmlp::Layout(K).total) + gcmlp::kHid * (gcmlp::kHid + 1));
}

// The learned scheduler's decision for the next level, from the counters of
// the level just ended: the next frontier's size and out-arcs and the
// level's time from its clock stamps. The network only picks the form of
// pull levels, so the work-group first applies the working-set rule's
// direction test and stops on a push level. Else it stages the parameters in
// LDS (coalesced, all loads in flight together; W2 at a pitch of kHid + 1,
// since each lane reads its own row) and its first wave runs the network.
// LDS: level_decide_lds(K) bytes at sp.
__device__ void level_decide(int32_t* __restrict__ stats, const LevelDecide& dec, uint64_t t1, float* sp) {
  const int64_t n_f = stats[gcx::kStatQLen];
  const int64_t m_f = static_cast<uint32_t>(stats[gcx::kStatArcs]);
  const double mu = static_cast<double>(dec.sub_next ? dec.unexplored - m_f : dec.unexplored);
  const bool pull_next = dec.pulling ? !(static_cast<double>(n_f) < static_cast<double>(dec.n) / dec.beta)
                                     : static_cast<double>(m_f) > mu / dec.alpha;
  if (!pull_next) {  // uniform
    if (threadIdx.x == 0) stats[gcx::kStatChoice] = -1;  // push: the rule alone
    return;
  }
  const gcmlp::Layout L(dec.K);
  float* w2 = sp + L.total;  // row r at r * (kHid + 1)
  constexpr int kIn = 16;  // loads in flight per thread
  for (int32_t i0 = threadIdx.x; i0 < L.total; i0 += kIn * kThreads) {
    float x[kIn];
#pragma unroll
    for (int u = 0; u < kIn; ++u) x[u] = dec.params[min(i0 + u * kThreads, L.total - 1)];
#pragma unroll
    for (int u = 0; u < kIn; ++u) {
      const int32_t i = i0 + u * kThreads, r = i - L.W2;
      if (i >= L.total) break;
      if (r >= 0 && r < gcmlp::kHid * gcmlp::kHid) w2[r + r / gcmlp::kHid] = x[u];
      else sp[i] = x[u];
    }
  }
  __syncthreads();
  if (threadIdx.x >= kWave) return;
  const uint64_t t0 = *reinterpret_cast<const uint64_t*>(stats + gcx::kStatT0);
  const double prior_ms = t1 > t0 ? static_cast<double>(t1 - t0) / dec.clock_khz : 0.0;
  float in[GC_SCHED_INPUTS];
  gcx::level_features(dec.n, dec.m, n_f, m_f, dec.level, prior_ms, dec.prior_arcs, in);
  gcmlp::mlp_decide<gcmlp::kHid + 1>(sp, w2, dec.K, in, dec.frange, stats + gcx::kStatChoice,
                                     reinterpret_cast<float*>(stats + gcx::kStatOut));
}

// End of a level: stamps the clock (the kernel runs right after the level's
// relaxation kernels), takes the scheduler's decision when dec has a
// network, hands the counters to the host and clears them (all by the first
// work-group), and zeroes the status words of the frontier just expanded
// when they are set: by all work-groups, which the host does not wait for, or
// (one work-group) by the waves beside the first, before it tells the host.
// The second costs a level less than waiting for the first costs the last
// level (4 us) while a thread has few words: BFS of uniform graphs of 20,000
// and 120,000 vertices 139 -> 132 and 152 -> 149 us.
constexpr int64_t kClearFirst = 4096;  // words that one work-group zeroes

__global__ __launch_bounds__(kThreads) void k_level_end(int32_t* __restrict__ stats, int32_t* __restrict__ host,
                                                        int32_t seq, LevelDecide dec, uint32_t* __restrict__ clear,
                                                        int64_t words) {
  extern __shared__ float sp[];
  const bool first = clear && gridDim.x == 1;  // uniform
  if (blockIdx.x == 0) {
    const uint64_t t1 = wall_clock64();
    if (dec.params) level_decide(stats, dec, t1, sp);  // uniform
    if (first) {
      if (threadIdx.x >= kWave)
        for (int64_t i = threadIdx.x - kWave; i < words; i += kThreads - kWave) clear[i] = 0u;
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the zeros have reached the L2
      __syncthreads();
    }
    if (threadIdx.x < kWave) {
      if (dec.params) __threadfence();  // the wave reads back the decision that its lanes have written
      publish_stats(stats, host, seq, dec.params ? dec.K : 0, t1);
    }
  }
  if (!clear || first) return;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * kThreads;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x; i < words; i += stride) clear[i] = 0u;
}

// ---------------------------------------------------------------------------
// BFS

// One wave's rows in LDS.
struct WaveRows {
  int32_t pre[kWave], off[kWave];
};

// Walks the rows of a wave (each lane's starts at b and has len arcs) end to
// end, 64 x kU arcs a step, so that the step's chain (column, frontier bit,
// value) is paid once for all rows and a lane has kU arcs in flight: a row per
// lane, and the whole wave for each row of more than 32 arcs in turn, paid it
// once per row. (The kernels' bound of 8 waves per SIMD keeps their registers
// at 64, so that both work-groups of 1024 threads are resident.) step(at, e, in) gets each arc's row (lane) and index, and a
// mask of those that exist.
template <int kU, class Step>
__device__ __forceinline__ void walk_rows(WaveRows& rows, int32_t b, int32_t len, Step&& step) {
  const int lane = gcd::lane_id();
  const int32_t incl = gcd::wave_incl_scan(len);
  const int32_t total = __builtin_amdgcn_readlane(incl, kWave - 1);
  if (total == 0) return;  // uniform
  rows.pre[lane] = incl - len;
  rows.off[lane] = b - (incl - len);
  gcd::wave_lds_fence();
  for (int64_t a0 = 0; a0 < total; a0 += kWave * kU) {  // uniform
    int at[kU];
    int32_t e[kU];
    uint32_t in = 0;
#pragma unroll
    for (int k = 0; k < kU; ++k) {
      const int64_t a = a0 + lane + k * kWave;
      int lo = 0;  // the last row with pre <= a
#pragma unroll
      for (int d = kWave / 2; d > 0; d >>= 1)
        if (rows.pre[lo + d] <= a) lo += d;
      at[k] = lo;
      e[k] = static_cast<int32_t>(a) + rows.off[lo];
      in |= static_cast<uint32_t>(a < total) << k;
    }
    step(at, e, in);
  }
  gcd::wave_lds_fence();
}

// Whether in-arcs [b, e) of each lane's row (none unless active) have an active
// source. Most rows of a level that is pulled end within their first
// kFirst arcs, which every lane looks at alone, four at a time; the wave then
// walks what is left of the others (no further for a row that was hit in an
// earlier step). BFS of an R-MAT graph of 8 M vertices and 64 M arcs 377 us
// with whole rows per lane (up to 32 arcs), 333 so; 335 with kFirst 4, 343
// with 16; a uniform graph of 4 M vertices and 64 M arcs 466, 473, 502, 479.
struct FrontRows : WaveRows {
  int32_t hit[kWave];
};
__device__ __forceinline__ bool scan_front(const int32_t* __restrict__ col, const uint32_t* __restrict__ front,
                                           bool active, int32_t b, int32_t e, FrontRows& rows) {
  constexpr int kFirst = 8;
  const int lane = gcd::lane_id();
  bool found = false;
  if (!active) e = b;
  const int32_t own = min(e, b + kFirst);
  for (int32_t i = b; i < own && !found; i += 4) {
    int32_t u[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) u[k] = col[min(i + k, e - 1)];
    uint32_t any = 0;  // all tests, no short circuit
#pragma unroll
    for (int k = 0; k < 4; ++k) any |= (front[u[k] >> 5] >> (u[k] & 31)) & 1u;
    found = any;
  }
  rows.hit[lane] = 0;
  walk_rows<4>(rows, own, found ? 0 : e - own, [&](const int(&at)[4], const int32_t(&i)[4], uint32_t in) {
#pragma unroll
    for (int k = 0; k < 4; ++k) in &= ~(static_cast<uint32_t>(rows.hit[at[k]] != 0) << k);
    int32_t u[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) u[k] = (in >> k) & 1u ? col[i[k]] : 0;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (((in >> k) & 1u) && bit_test(front, u[k])) rows.hit[at[k]] = 1;
    gcd::wave_lds_fence();
  });
  return found || rows.hit[lane];
}

// Topology-driven pull over the whole transposed graph. The work-groups
// stride over the vertices (their waves by themselves, without barriers), so
// the counters take one atomic per resident work-group.
template <int NT>
__global__ __launch_bounds__(NT, 8) void k_bfs_pull(const int32_t* __restrict__ t_rowptr,
                                                 const int32_t* __restrict__ t_col, int32_t n,
                                                 const uint32_t* __restrict__ front, int32_t* __restrict__ depth,
                                                 int32_t level, uint32_t* __restrict__ next,
                                                 uint32_t* __restrict__ visited, Tally tally) {
  __shared__ FrontRows rows[NT / kWave];
  stamp_start(tally.stats);
  Counted cnt;
  for (int64_t base = static_cast<int64_t>(blockIdx.x) * NT; base < n; base += static_cast<int64_t>(gridDim.x) * NT) {
    const int32_t v = static_cast<int32_t>(min<int64_t>(base + threadIdx.x, INT32_MAX));
    // the visited word and the row bounds are loaded together (one memory
    // round trip before the scan, not two)
    uint32_t vw = ~0u;
    int32_t b = 0, e = 0;
    if (v < n) {
      vw = visited[v >> 5];
      b = t_rowptr[v];
      e = t_rowptr[v + 1];
    }
    const bool active = !((vw >> (v & 31)) & 1u);
    const bool found = scan_front(t_col, front, active, b, e, rows[threadIdx.x / kWave]);
    if (found) {
      depth[v] = level + 1;
      cnt.add(tally, v);
    }
    wave_bits_set(next, v, found);
    wave_bits_set(visited, v, found);
  }
  publish_count<NT>(tally, cnt);
}

// TOCAB pull, per block: flag[l] = 1 when local row l (an unvisited vertex)
// has an in-arc from an active source of this block; a local next array.
__global__ __launch_bounds__(kThreads) void k_bfs_tocab(const int32_t* __restrict__ row_ptr,
                                                        const int32_t* __restrict__ col,
                                                        const int32_t* __restrict__ id_map, int64_t P,
                                                        const uint32_t* __restrict__ visited,
                                                        const uint32_t* __restrict__ front,
                                                        uint8_t* __restrict__ flag, int32_t* __restrict__ stats) {
  __shared__ FrontRows rows[kThreads / kWave];
  stamp_start(stats);
  // the stride is uniform over the work-group, so every wave of it runs the
  // same passes and the wave-wide scans inside stay convergent
  for (int64_t base = static_cast<int64_t>(blockIdx.x) * kThreads; base < P;
       base += static_cast<int64_t>(gridDim.x) * kThreads) {
    const int64_t l = base + threadIdx.x;
    bool active = false;
    int32_t b = 0, e = 0;
    if (l < P && !bit_test(visited, id_map[l])) {
      active = true;
      b = row_ptr[l];
      e = row_ptr[l + 1];
    }
    const bool found = scan_front(col, front, active, b, e, rows[threadIdx.x / kWave]);
    if (l < P) flag[l] = found ? 1 : 0;
  }
}

// Merge of the per-block flags over vertex range j (OR), fused with the
// depth update and the next frontier (Section 3.3: the reduction of next is
// done in the same kernel as that of the partial results).
template <int K, bool kFlat>
__global__ __launch_bounds__(kThreads) void k_bfs_merge(const int32_t* __restrict__ range_ptr, int32_t B,
                                                        const uint16_t* __restrict__ id16,
                                                        const uint8_t* __restrict__ flag, int32_t n,
                                                        int32_t* __restrict__ depth, int32_t level,
                                                        uint32_t* __restrict__ next, uint32_t* __restrict__ visited,
                                                        Tally tally) {
  __shared__ uint8_t hit[K];
  Counted cnt;
  const int32_t v0 = blockIdx.x * K;
  for (int i = threadIdx.x; i < K; i += kThreads) hit[i] = 0;
  gcm::merge_slices<kFlat, kThreads>(range_ptr, B, id16, flag, blockIdx.x, [&](uint32_t v, uint8_t f) {
    if (f) hit[v] = 1;
  });
  for (int i = threadIdx.x; i < K; i += kThreads) {
    const int32_t v = v0 + i;
    const bool found = v < n && hit[i] && !bit_test(visited, v);
    if (found) {
      depth[v] = level + 1;
      cnt.add(tally, v);
    }
    wave_bits_set(next, v, found);
    wave_bits_set(visited, v, found);
  }
  publish_count<kThreads>(tally, cnt);
}

// ---------------------------------------------------------------------------
// SSSP (synchronous Bellman-Ford rounds over the vertices changed last round)

// Minimum of dist[u] + w over in-arcs [b, e) of each lane's row from active
// sources u (kInf if none). *ovf is set when a candidate path length reaches
// INT32_MAX. Shortest paths by pull alone, 10^6 vertices of an R-MAT graph,
// 16 arcs each: 3840 us with a row per lane, 2660 so (4110 without the case
// of one row, whose lanes all met on one LDS word).
struct MinRows : WaveRows {
  int32_t best[kWave];
};
__device__ __forceinline__ int32_t scan_min(const int32_t* __restrict__ col, const int32_t* __restrict__ w,
                                            const uint32_t* __restrict__ front, const int32_t* __restrict__ dist,
                                            bool active, int32_t b, int32_t e, bool* ovf, MinRows& rows) {
  const int lane = gcd::lane_id();
  bool over = false;
  rows.best[lane] = kInf;
  walk_rows<4>(rows, b, active ? e - b : 0, [&](const int(&at)[4], const int32_t(&i)[4], uint32_t in) {
    int32_t u[4], wk[4], du[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) u[k] = (in >> k) & 1u ? col[i[k]] : 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) in &= ~(static_cast<uint32_t>(!bit_test(front, u[k])) << k);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      wk[k] = (in >> k) & 1u ? w[i[k]] : 0;
      du[k] = (in >> k) & 1u ? dist[u[k]] : 0;
    }
    int32_t cand[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const bool on = (in >> k) & 1u, past = wk[k] >= kInf - du[k];  // du[k] + wk[k] >= kInf
      over |= on && past;
      cand[k] = on && !past ? du[k] + wk[k] : kInf;
    }
    if (__builtin_amdgcn_readfirstlane(at[0]) == __builtin_amdgcn_readlane(at[3], kWave - 1)) {  // one row has them all
      int32_t m = min(min(cand[0], cand[1]), min(cand[2], cand[3]));
      for (int o = 32; o > 0; o >>= 1) m = min(m, __shfl_xor(m, o, kWave));
      if (lane == 0 && m != kInf) atomicMin(&rows.best[at[0]], m);
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (cand[k] != kInf) atomicMin(&rows.best[at[k]], cand[k]);
    }
  });
  gcd::wave_lds_fence();
  *ovf = over;
  return rows.best[lane];
}

template <int NT>
__global__ __launch_bounds__(NT, 8) void k_sssp_pull(const int32_t* __restrict__ t_rowptr,
                                                  const int32_t* __restrict__ t_col,
                                                  const int32_t* __restrict__ t_w, int32_t n,
                                                  const uint32_t* __restrict__ front, int32_t* __restrict__ dist,
                                                  uint32_t* __restrict__ next, Tally tally) {
  __shared__ MinRows rows[NT / kWave];
  stamp_start(tally.stats);
  Counted cnt;
  bool any_over = false;
  for (int64_t base = static_cast<int64_t>(blockIdx.x) * NT; base < n; base += static_cast<int64_t>(gridDim.x) * NT) {
    const int32_t v = static_cast<int32_t>(min<int64_t>(base + threadIdx.x, INT32_MAX));
    int32_t b = 0, e = 0;
    if (v < n) {
      b = t_rowptr[v];
      e = t_rowptr[v + 1];
    }
    bool ovf;
    const int32_t best = scan_min(t_col, t_w, front, dist, v < n, b, e, &ovf, rows[threadIdx.x / kWave]);
    any_over |= ovf;
    bool improved = false;
    if (v < n && best < dist[v]) {
      dist[v] = best;
      improved = true;
      cnt.add(tally, v);
    }
    wave_bits_set(next, v, improved);
  }
  if (any_over) tally.stats[kOverflow] = 1;
  publish_count<NT>(tally, cnt);
}

// TOCAB pull, per block: pmin[l] = min over active sources of this block of
// dist[u] + w (INT32_MAX if none; saturated on overflow, which is flagged).
__global__ __launch_bounds__(kThreads) void k_sssp_tocab(const int32_t* __restrict__ row_ptr,
                                                         const int32_t* __restrict__ col,
                                                         const int32_t* __restrict__ w, int64_t P,
                                                         const uint32_t* __restrict__ front,
                                                         const int32_t* __restrict__ dist, int32_t* __restrict__ pmin,
                                                         int32_t* __restrict__ stats) {
  __shared__ MinRows rows[kThreads / kWave];
  stamp_start(stats);
  for (int64_t base = static_cast<int64_t>(blockIdx.x) * kThreads; base < P;
       base += static_cast<int64_t>(gridDim.x) * kThreads) {  // uniform per work-group
    const int64_t l = base + threadIdx.x;
    int32_t b = 0, e = 0;
    if (l < P) {
      b = row_ptr[l];
      e = row_ptr[l + 1];
    }
    bool ovf;
    const int32_t best = scan_min(col, w, front, dist, l < P, b, e, &ovf, rows[threadIdx.x / kWave]);
    if (ovf) stats[kOverflow] = 1;
    if (l < P) pmin[l] = best;
  }
}

// TOCAB pull for SSSP and BFS over the stream layout (blocks up to 2^15 wide,
// the layout the PageRank pull reads): the block's slice of the frontier's
// distances lives in LDS, so the random reads of a round never leave the CU.
// Values are kept as INT32_MAX - distance, 0 for a source outside the
// frontier, so that "none" is 0 and the minimum of a row is a maximum of
// values whose lack is masked, like PageRank's sums: the same tile reduction
// does both (BFS: 1 for a source in the frontier). One work-group per chunk
// of the partition (rows [r0, r1) of block b) fills the slice, then each wave
// walks a contiguous range of 512-arc tiles: a lane holds 8 consecutive arcs
// (16-bit columns, their weights, the head bits of its head word) and takes
// the candidates value[col] - w, saturating at 0. pmin gets every row's
// result at its range-major index. What bounds it is the instruction path of
// the tile reduction, not memory. Measured: 16 M weighted arcs of a uniform
// graph 87 -> 57 us, the 15.6 M arcs of a 4 M-vertex grid's BFS 70 -> 45 us
// (before: a minimum of its own with a store per arc and a walk over the
// position table per tile).
using namespace gcs;

// Weights of a stream-layout partition in its arc order (kW): int32
// (kW32), one byte each when every weight lies in [0, 255] (kW8), or none:
// BFS, whose candidates are the sources' own values.
constexpr int kW32 = 0, kW8 = 1, kWNone = 2;
typedef int32_t ti32x4 __attribute__((ext_vector_type(4)));

// A tile's raw streams for one lane: its 8 columns, its head word and its
// 8 weights (as loaded), so that the loads of later tiles can be issued
// before an earlier tile is reduced.
struct RawTile {
  u32x4 cols;
  u32x4 hw;
  ti32x4 wa, wb;  // int32 weights (kW32)
  uint64_t w8;    // byte weights (kW8)
};

template <int kW>
__device__ __forceinline__ RawTile load_raw_tile(const uint16_t* __restrict__ col16,
                                                 const gc_head_word* __restrict__ heads,
                                                 const void* __restrict__ w_arcs, int64_t q, int lane) {
  RawTile r;
  const int64_t tb = q * kWaveTile;
  r.cols = gcd::ld_stream(reinterpret_cast<const u32x4*>(col16 + tb) + lane);
  r.hw = *reinterpret_cast<const u32x4*>(heads + (tb >> 6) + (lane >> 3));
  if (kW == kW8) {
    r.w8 = gcd::ld_stream(reinterpret_cast<const uint64_t*>(static_cast<const uint8_t*>(w_arcs) + tb) + lane);
  } else if (kW == kW32) {
    const int32_t* w_pad = static_cast<const int32_t*>(w_arcs);
    r.wa = gcd::ld_stream(reinterpret_cast<const ti32x4*>(w_pad + tb) + 2 * lane);
    r.wb = gcd::ld_stream(reinterpret_cast<const ti32x4*>(w_pad + tb) + 2 * lane + 1);
  }
  return r;
}

// Keeps a tile's registers and candidates allocated up to this point.
template <int kW>
__device__ __forceinline__ void hold_raw(const RawTile& t, const uint32_t (&x)[kArcsPerLane]) {
  asm volatile("" ::"v"(t.cols), "v"(t.hw));
  if (kW == kW8) asm volatile("" ::"v"(t.w8));
  if (kW == kW32) asm volatile("" ::"v"(t.wa), "v"(t.wb));
#pragma unroll
  for (int e = 0; e < kArcsPerLane; ++e) asm volatile("" ::"v"(x[e]));
}

// The lane's arcs of tile q (bit e: arc e) that lie in [a0, a1) (indices
// past the layout's end still fit 32 bits).
__device__ __forceinline__ uint32_t arcs_inside(int32_t q, int lane, int32_t a0, int32_t a1) {
  const int32_t b = q * kWaveTile + kArcsPerLane * lane;
  const int32_t lo = min(max(a0 - b, 0), kArcsPerLane), hi = min(max(a1 - b, 0), kArcsPerLane);
  return (0xFFu << lo) & ~(0xFFu << hi);
}

// The lane's candidates from the slice at ad. check (uniform): a path length
// may reach INT32_MAX in this block; *ovf is set when one does over an arc of
// the mask own(). The first and the last tile of a chunk also hold arcs of
// the blocks beside it, whose columns are offsets into other slices: they are
// left out of the mask.
template <int kW, class Own>
__device__ __forceinline__ void gather_min(const RawTile& r, const uint32_t* ad, bool check, Own&& own,
                                           uint32_t (&x)[kArcsPerLane], bool* ovf) {
#pragma unroll
  for (int e = 0; e < kArcsPerLane; ++e) x[e] = ad[(r.cols[e >> 1] >> (16 * (e & 1))) & 0xFFFFu];
  if (kW == kWNone) return;
  uint32_t w[kArcsPerLane];
#pragma unroll
  for (int e = 0; e < kArcsPerLane; ++e)
    w[e] = kW == kW8 ? static_cast<uint32_t>(r.w8 >> (8 * e)) & 0xFFu
                     : static_cast<uint32_t>(e < 4 ? r.wa[e] : r.wb[e - 4]);
  if (check) {
    const uint32_t mine = own();
#pragma unroll
    for (int e = 0; e < kArcsPerLane; ++e) *ovf |= ((mine >> e) & 1u) && x[e] != 0u && w[e] >= x[e];
  }
#pragma unroll
  for (int e = 0; e < kArcsPerLane; ++e) x[e] = __builtin_elementwise_sub_sat(x[e], w[e]);
}

// Largest candidate over the tiles after tile q of the row open at q's end,
// up to its end (the first head bit that follows).
template <int kW>
__device__ uint32_t finish_open_min(const uint16_t* __restrict__ col16, const gc_head_word* __restrict__ heads,
                                    const void* __restrict__ w_arcs, const uint32_t* ad, bool check, int32_t q,
                                    int lane, bool* ovf) {
  uint32_t best = 0;
  for (int64_t qq = static_cast<int64_t>(q) + 1;; ++qq) {
    const RawTile r = load_raw_tile<kW>(col16, heads, w_arcs, qq, lane);
    const uint32_t my8 = static_cast<uint32_t>(word_bits(r.hw) >> (8 * (lane & 7))) & 0xFFu;
    const uint64_t hl = __ballot(my8 != 0u);
    const int first_lane = hl ? __ffsll(static_cast<long long>(hl)) - 1 : kWave;
    // the lane's arcs before the tile's first head
    const int mine = lane < first_lane ? kArcsPerLane : (lane == first_lane ? __ffs(my8) - 1 : 0);
    uint32_t x[kArcsPerLane];
    bool o = false;
    gather_min<kW>(r, ad, check, [&] { return (1u << mine) - 1u; }, x, &o);
    *ovf |= o;
    uint32_t m = 0;
#pragma unroll
    for (int e = 0; e < kArcsPerLane; ++e) m = e < mine ? max(m, x[e]) : m;
    best = max(best, static_cast<uint32_t>(gcd::wave_max(static_cast<int>(m))));  // below 2^31
    if (hl) return best;  // bits past the last arc are set, so this ends
  }
}

template <int kW>
__global__ __launch_bounds__(kLdsThreads) void k_sssp_tocab_lds(
    const int32_t* __restrict__ row_ptr, const uint16_t* __restrict__ col16, const gc_head_word* __restrict__ heads,
    const void* __restrict__ w_arcs, uint32_t max_w, const int32_t* __restrict__ chunk_beg,
    const int32_t* __restrict__ chunk_end, const int32_t* __restrict__ chunk_blk, const int32_t* __restrict__ chunk_j0,
    const int32_t* __restrict__ chunk_ns, const int2* __restrict__ seg, int32_t R, int32_t log2W, int32_t n,
    const uint32_t* __restrict__ front, const int32_t* __restrict__ dist, int32_t* __restrict__ pmin,
    uint32_t pmin_bytes, int32_t* __restrict__ stats) {
  extern __shared__ uint32_t ad[];
  stamp_start(stats);
  const __amdgpu_buffer_rsrc_t out = partial_rsrc(pmin, pmin_bytes);
  const int32_t ch = blockIdx.x;
  const int32_t r0 = chunk_beg[ch], r1 = chunk_end[ch], b = chunk_blk[ch], j0 = chunk_j0[ch], ns = chunk_ns[ch];
  if (r0 >= r1) return;  // padding of the dispatch order (uniform)
  // Each wave streams a contiguous range [qa, qz] of the chunk's tiles. Its
  // bounds and its first tiles depend on the chunk alone, so their loads are
  // issued before the block's LDS fill and overlap it.
  const int lane = threadIdx.x & (kWave - 1);
  const int wid = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
  const int32_t a0 = row_ptr[r0], a1 = row_ptr[r1];  // the chunk's arcs
  const int32_t q0 = a0 / kWaveTile, q1 = (a1 - 1) / kWaveTile;
  const int32_t nt = q1 - q0 + 1;
  const int32_t qa = q0 + static_cast<int32_t>(static_cast<int64_t>(nt) * wid / kLdsWaves);
  const int32_t qz = q0 + static_cast<int32_t>(static_cast<int64_t>(nt) * (wid + 1) / kLdsWaves) - 1;
  // Tiles in registers: four, as in the PageRank pull; two with weights,
  // whose registers would otherwise spill, and a spill's reload waits for
  // every tile load before it (68 -> 57 us on the uniform graph above).
  constexpr int kDepth = kW == kWNone ? 4 : 2;
  int32_t q = qa;
  RawTile t0{}, t1{}, t2{}, t3{};
  if (qa <= qz) {  // uniform over the wave; loads clamped to the wave's last tile
    t0 = load_raw_tile<kW>(col16, heads, w_arcs, q, lane);
    t1 = load_raw_tile<kW>(col16, heads, w_arcs, min(q + 1, qz), lane);
    if (kDepth > 2) {
      t2 = load_raw_tile<kW>(col16, heads, w_arcs, min(q + 2, qz), lane);
      t3 = load_raw_tile<kW>(col16, heads, w_arcs, min(q + 3, qz), lane);
    }
  }
  const int32_t W = 1 << log2W, v0 = b << log2W, cnt = min(W, n - v0);  // cnt >= 1
  uint32_t* stage = ad + W + wid * (kStageRows + kStageSpare);  // this wave's output staging and spare slots
  int32_t* sb = reinterpret_cast<int32_t*>(ad + W + kLdsWaves * (kStageRows + kStageSpare));
  int32_t* sd = sb + ns + kSegPad;
  int32_t* near = sd + ns + kSegPad;  // [kLdsWaves]: the wave filled a value that a weight may exhaust
  // The block's frontier values in LDS: thread t fills vertices t + 1024 u.
  // A wave's vertices need 64 status words, one per lane and one load, handed
  // out by lane reads; then the distances, kFill loads in flight, a vertex
  // outside the frontier reading the block's first one instead (so a sparse
  // frontier costs no slice of distances).
  constexpr int kFill = 16;
  bool exhaust = false;
  const int32_t nu = W / kLdsThreads;  // 1 .. 32
  uint32_t word = 0;
  {
    const int32_t wi = (lane >> 1) * (kLdsThreads / 32) + 2 * wid + (lane & 1);
    if (32 * wi < cnt) word = front[(v0 >> 5) + wi];
  }
  for (int32_t u0 = 0; u0 < nu; u0 += kFill) {
    int32_t dv[kFill];
    uint32_t on = 0;
#pragma unroll
    for (int k = 0; k < kFill; ++k) {
      const int32_t u = min(u0 + k, nu - 1);
      const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(word), 2 * u);
      const uint32_t hi = __builtin_amdgcn_readlane(static_cast<int>(word), 2 * u + 1);
      const uint32_t bit = ((lane < 32 ? lo : hi) >> (lane & 31)) & 1u;
      on |= bit << k;
      if (kW != kWNone) dv[k] = dist[v0 + (bit ? u * kLdsThreads + static_cast<int32_t>(threadIdx.x) : 0)];
    }
#pragma unroll
    for (int k = 0; k < kFill; ++k) {
      const int32_t u = min(u0 + k, nu - 1);
      uint32_t y = (on >> k) & 1u;
      if (kW != kWNone) {
        y = y ? static_cast<uint32_t>(kInf - dv[k]) : 0u;
        exhaust |= y != 0u && y <= max_w;
      }
      ad[u * kLdsThreads + threadIdx.x] = y;
    }
  }
  // the chunk's part of the position table: sb[i] = first row of merge range
  // j0 + i, sd[i] = its shift to the range-major index; sb[ns] lies past the
  // chunk, then sentinels
  {
    const int2* sg = seg + static_cast<int64_t>(b) * (R + 1) + j0;
    for (int32_t i = threadIdx.x; i < ns + kSegPad; i += kLdsThreads) {
      const int2 e = i <= ns ? sg[i] : make_int2(INT32_MAX, 0);
      sb[i] = e.x;
      sd[i] = e.y;
    }
  }
  exhaust = __any(exhaust);
  if (lane == 0) near[wid] = exhaust ? 1 : 0;
  __syncthreads();
  if (qa > qz) return;  // no barrier follows
  const bool check = kW != kWNone && __any(near[lane & (kLdsWaves - 1)] != 0);
  bool ovf = false;
  PullCarry<MaxOp> cr;
  load_window(sb, sd, ns, lane, cr);
  cursor_from_window(cr);
  uint32_t x0[kArcsPerLane], x1[kArcsPerLane];
  // the chunk's arcs of the wave's tile i (clamped to its last)
  auto own = [&](int32_t i) { return [=] { return arcs_inside(min(i, qz), lane, a0, a1); }; };
  gather_min<kW>(t0, ad, check, own(q), x0, &ovf);
#define GC_MIN_STEP(cur, xcur, nxt, xnxt, k)                                       \
  gather_min<kW>(nxt, ad, check, own(q + (k + 1)), xnxt, &ovf);                    \
  reduce_wave_tile<MaxOp>(cur.hw, xcur, lane, sb, sd, ns, r0, r1, cr, out, stage); \
  hold_raw<kW>(cur, xcur);                                                         \
  cur = load_raw_tile<kW>(col16, heads, w_arcs, min(q + (k + kDepth), qz), lane);
  // whole rounds of kDepth tiles in the loop, the rest after it
  const int32_t nw = qz - qa + 1;
  for (int32_t round = 0; round < nw / kDepth; ++round) {
    if constexpr (kDepth == 4) {
      GC_MIN_STEP(t0, x0, t1, x1, 0)
      GC_MIN_STEP(t1, x1, t2, x0, 1)
      GC_MIN_STEP(t2, x0, t3, x1, 2)
      GC_MIN_STEP(t3, x1, t0, x0, 3)
    } else {
      GC_MIN_STEP(t0, x0, t1, x1, 0)
      GC_MIN_STEP(t1, x1, t0, x0, 1)
    }
    q += kDepth;
  }
  const int32_t rest = nw % kDepth;
  if (rest > 0) {
    if (kDepth > 2) gather_min<kW>(t1, ad, check, own(q + 1), x1, &ovf);
    reduce_wave_tile<MaxOp>(t0.hw, x0, lane, sb, sd, ns, r0, r1, cr, out, stage);
  }
  if constexpr (kDepth == 4) {
    if (rest > 1) {
      gather_min<kW>(t2, ad, check, own(q + 2), x0, &ovf);
      reduce_wave_tile<MaxOp>(t1.hw, x1, lane, sb, sd, ns, r0, r1, cr, out, stage);
    }
    if (rest > 2) reduce_wave_tile<MaxOp>(t2.hw, x0, lane, sb, sd, ns, r0, r1, cr, out, stage);
  }
#undef GC_MIN_STEP
  if (cr.open_row >= 0) {  // the range's last row continues past it
    const uint32_t v = max(cr.open, finish_open_min<kW>(col16, heads, w_arcs, ad, check, qz, lane, &ovf));
    if (lane == 0) pmin[cr.open_row + sd[seek_range(sb, cr.jc, cr.open_row)]] = static_cast<int32_t>(v);
  }
  if (kW != kWNone && __any(ovf) && lane == 0) stats[kOverflow] = 1;
}

// Dynamic LDS of k_sssp_tocab_lds for partition t: the PageRank pull's, plus
// a word per wave.
inline size_t tocab_lds_bytes(const gc_tocab_s* t) {
  return sizeof(int32_t) * (static_cast<size_t>(t->W) + 2 * static_cast<size_t>(t->seg_max) + 2 * kSegPad + kLdsWaves) +
         gcx::kLdsStageBytes;
}

// Size in bytes of the partial minima of a stream-layout partition (P + 8
// entries, below 2^31 bytes by the layout's own limit).
inline uint32_t pmin_bytes(const gc_tocab_s* t) { return static_cast<uint32_t>(sizeof(int32_t) * (t->P + 8)); }

// Figure 5 merge of the stream-layout SSSP partial minima, read as streams:
// range j's partials of every block are one contiguous slice [rstart[j],
// rstart[j+1]) of pmin / id16s (the position table's range-major order). A
// persistent work-group (two per CU) walks ranges j = blockIdx.x,
// blockIdx.x + gridDim.x, ...: 16-byte / 8-byte loads of 4 entries, LDS
// maxima of the inverted values, then the range's vertices are updated
// (distance, next status bit, counts) and the maxima reset for the next
// range, whose first loads are issued before that update.
template <int K, int NT, bool kBfs>
__global__ __launch_bounds__(NT) void k_sssp_merge_stream(const int32_t* __restrict__ rstart,
                                                          const uint16_t* __restrict__ id16s,
                                                          const int32_t* __restrict__ pmin, int32_t R, int32_t n,
                                                          int32_t* __restrict__ dist, uint32_t* __restrict__ next,
                                                          Tally tally, int32_t level, uint32_t* __restrict__ visited) {
  __shared__ int32_t best[K];
  Counted cnt;
  for (int i = threadIdx.x; i < K; i += NT) best[i] = 0;
  __syncthreads();
  const ti32x4* p4 = reinterpret_cast<const ti32x4*>(pmin);
  const uint64_t* i4 = reinterpret_cast<const uint64_t*>(id16s);
  constexpr int kU = 4;  // groups of 4 entries per thread and step (two register sets in turn)
  constexpr int32_t kStep = NT * kU;
  ti32x4 pa[kU], pb[kU];
  uint64_t ia[kU], ib[kU];
  int32_t a = 0, z = 0, g0 = 0, g1 = 0;
  auto bounds = [&](int32_t j) {
    a = rstart[j];
    z = rstart[j + 1];
    g0 = a >> 2;
    g1 = (z + 3) >> 2;
  };
  // loads clamped to the range's last group: no branch, so the compiler's
  // count of outstanding loads holds on every path
  auto load = [&](int32_t g, ti32x4 (&p)[kU], uint64_t (&id)[kU]) {
#pragma unroll
    for (int k = 0; k < kU; ++k) {
      const int32_t gg = min(g + k * NT, g1 - 1);
      p[k] = gcd::ld_stream(p4 + gg);
      id[k] = gcd::ld_stream(i4 + gg);
    }
  };
  auto take = [&](int32_t g, const ti32x4 (&p)[kU], const uint64_t (&id)[kU]) {
#pragma unroll
    for (int k = 0; k < kU; ++k) {
      const int32_t e0 = 4 * (g + k * NT);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (e0 + e >= a && e0 + e < z && p[k][e] != 0) atomicMax(&best[(id[k] >> (16 * e)) & 0xFFFFu], p[k][e]);
    }
  };
  const int32_t tid = threadIdx.x;
  int32_t j = blockIdx.x;
  if (j < R) {
    bounds(j);
    if (g0 < g1) load(g0 + tid, pa, ia);  // uniform
  }
  for (; j < R; j += gridDim.x) {
    for (int32_t g = g0 + tid; g < g1; g += 2 * kStep) {
      load(g + kStep, pb, ib);
      take(g, pa, ia);
      load(g + 2 * kStep, pa, ia);
      take(g + kStep, pb, ib);
    }
    __syncthreads();
    const int32_t v0 = j * K;
    static_assert(K % NT == 0 && NT % kWave == 0, "whole waves over the range");
    constexpr int kPer = K / NT;
    // The range's vertices v0 + tid + u NT. Their minima come from LDS and,
    // for those with a candidate, their distance (BFS: their visited word)
    // is loaded into registers before the next range's first minima, so
    // that the update waits for neither those loads nor one load per step;
    // a vertex with no candidate (or past n) reads the range's first vertex
    // instead, one line per wave.
    int32_t bi[kPer], cur[kPer];
    const uint32_t last = static_cast<uint32_t>(n - 1 - v0);
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int32_t i = tid + u * NT;
      bi[u] = best[i];
      best[i] = 0;
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const uint32_t o = static_cast<uint32_t>(tid + u * NT);
      const bool need = o <= last && bi[u] != 0;
      const uint32_t oo = need ? o : 0u;
      cur[u] = kBfs ? static_cast<int32_t>(visited[(static_cast<uint32_t>(v0) + oo) >> 5]) : dist[v0 + oo];
    }
    const int32_t jn = j + gridDim.x;
    if (jn < R) {  // uniform: the next range's first loads, in flight during the update
      bounds(jn);
      if (g0 < g1) load(g0 + tid, pa, ia);
    }
    // distance (or depth) and status bits, with one atomic per 32-bit status
    // word (a wave's 32 lanes hold one word's vertices, the range starts on
    // a word), then the new frontier's degrees, which are counted
    uint32_t took = 0;  // bit u: vertex v0 + tid + u NT entered the next frontier
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int32_t v = v0 + tid + u * NT;
      bool improved;
      if (kBfs) {  // depth: a vertex not yet reached with an in-neighbour in the frontier
        improved = v < n && bi[u] != 0 && !((static_cast<uint32_t>(cur[u]) >> (v & 31)) & 1u);
        if (improved) dist[v] = level + 1;
      } else {
        const int32_t nd = kInf - bi[u];
        improved = v < n && bi[u] != 0 && nd < cur[u];
        if (improved) dist[v] = nd;
      }
      const uint64_t m = __ballot(improved);
      const int lane = tid & (kWave - 1);
      const uint32_t word = static_cast<uint32_t>(m >> (lane & 32));
      if ((lane & 31) == 0 && word != 0u) {
        atomicOr(&next[v >> 5], word);
        if (kBfs) atomicOr(&visited[v >> 5], word);
      }
      took |= static_cast<uint32_t>(improved) << u;
    }
    if (__any(took)) {  // the new frontier's degrees, all loads together (others read the range's first vertex)
      int32_t lo[kPer], hi[kPer];
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        const int32_t o = (took >> u) & 1u ? tid + u * NT : 0;
        lo[u] = tally.rowptr[v0 + o];
        hi[u] = tally.rowptr[v0 + o + 1];
      }
#pragma unroll
      for (int u = 0; u < kPer; ++u) cnt.mine += (took >> u) & 1u ? one_vertex(hi[u] - lo[u]) : 0ull;
      if (tally.t_rowptr) {  // uniform
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
          const int32_t o = (took >> u) & 1u ? tid + u * NT : 0;
          lo[u] = tally.t_rowptr[v0 + o];
          hi[u] = tally.t_rowptr[v0 + o + 1];
        }
#pragma unroll
        for (int u = 0; u < kPer; ++u) cnt.in += (took >> u) & 1u ? static_cast<uint64_t>(hi[u] - lo[u]) : 0ull;
      }
    }
    __syncthreads();
  }
  publish_count<NT>(tally, cnt);
}

template <int K, bool kFlat>
__global__ __launch_bounds__(kThreads) void k_sssp_merge(const int32_t* __restrict__ range_ptr, int32_t B,
                                                         const uint16_t* __restrict__ id16,
                                                         const int32_t* __restrict__ pmin, int32_t n,
                                                         int32_t* __restrict__ dist, uint32_t* __restrict__ next,
                                                         Tally tally) {
  __shared__ int32_t best[K];
  Counted cnt;
  const int32_t v0 = blockIdx.x * K;
  for (int i = threadIdx.x; i < K; i += kThreads) best[i] = kInf;
  gcm::merge_slices<kFlat, kThreads>(range_ptr, B, id16, pmin, blockIdx.x, [&](uint32_t v, int32_t p) {
    if (p != kInf) atomicMin(&best[v], p);
  });
  for (int i = threadIdx.x; i < K; i += kThreads) {
    const int32_t v = v0 + i;
    bool improved = false;
    if (v < n && best[i] < dist[v]) {
      dist[v] = best[i];
      improved = true;
      cnt.add(tally, v);
    }
    wave_bits_set(next, v, improved);
  }
  publish_count<kThreads>(tally, cnt);
}

// ---------------------------------------------------------------------------
// Betweenness centrality (Section 4's BC benchmark): the BFS levels above
// also count shortest paths, sigma[v] = sum of sigma[u] over in-neighbours u
// one level up (Algorithm 3's update); then the dependencies are
// accumulated level by level backwards (Brandes).

// Sum of sigma[u] over in-arcs [b, e) of each lane's row (none unless active)
// from active sources u (FP64). The first pull level of an R-MAT graph of
// 2^20 vertices (16 M arcs) took 186 us with a row per lane, 118 so.
struct SigmaRows : WaveRows {
  double sum[kWave];
};
__device__ __forceinline__ double scan_sigma(const int32_t* __restrict__ col, const uint32_t* __restrict__ front,
                                             const double* __restrict__ sigma, bool active, int32_t b, int32_t e,
                                             SigmaRows& rows) {
  const int lane = gcd::lane_id();
  rows.sum[lane] = 0.0;
  walk_rows<4>(rows, b, active ? e - b : 0, [&](const int(&at)[4], const int32_t(&i)[4], uint32_t in) {
    int32_t u[4];
    double x[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) u[k] = (in >> k) & 1u ? col[i[k]] : 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) in &= ~(static_cast<uint32_t>(!bit_test(front, u[k])) << k);
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = (in >> k) & 1u ? sigma[u[k]] : 0.0;
    if (__builtin_amdgcn_readfirstlane(at[0]) == __builtin_amdgcn_readlane(at[3], kWave - 1)) {  // one row has them all
      const double t = gcd::wave_sum((x[0] + x[1]) + (x[2] + x[3]));
      if (lane == 0 && t != 0.0) atomicAdd(&rows.sum[at[0]], t);
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if ((in >> k) & 1u) atomicAdd(&rows.sum[at[k]], x[k]);
    }
  });
  gcd::wave_lds_fence();
  return rows.sum[lane];
}

// Topology-driven pull: an unvisited vertex with an active in-neighbour
// joins the next level with the sum of their path counts. Rows of more than
// kHugeRow arcs (kHuges of them at most) are left for the whole work-group:
// one wave would walk a hub's row for longer than the level's other rows
// take together.
constexpr int kHugeRow = 4096, kHuges = 64;
template <int NT>
__global__ __launch_bounds__(NT, 8) void k_bc_pull(const int32_t* __restrict__ t_rowptr,
                                                const int32_t* __restrict__ t_col, int32_t n,
                                                const uint32_t* __restrict__ front, int32_t* __restrict__ depth,
                                                int32_t level, double* __restrict__ sigma,
                                                uint32_t* __restrict__ next, uint32_t* __restrict__ visited,
                                                Tally tally) {
  __shared__ SigmaRows rows[NT / kWave];
  __shared__ int32_t huge[kHuges], huges;
  if (threadIdx.x == 0) huges = 0;
  __syncthreads();
  Counted cnt;
  for (int64_t base = static_cast<int64_t>(blockIdx.x) * NT; base < n; base += static_cast<int64_t>(gridDim.x) * NT) {
    const int32_t v = static_cast<int32_t>(min<int64_t>(base + threadIdx.x, INT32_MAX));
    uint32_t vw = ~0u;
    int32_t b = 0, e = 0;
    if (v < n) {
      vw = visited[v >> 5];
      b = t_rowptr[v];
      e = t_rowptr[v + 1];
    }
    bool active = !((vw >> (v & 31)) & 1u);
    if (active && e - b > kHugeRow) {
      const int at = atomicAdd(&huges, 1);
      if (at < kHuges) {
        huge[at] = v;
        active = false;
      }
    }
    const double sum = scan_sigma(t_col, front, sigma, active, b, e, rows[threadIdx.x / kWave]);
    const bool found = active && sum > 0.0;  // every active vertex has sigma >= 1
    if (found) {
      depth[v] = level + 1;
      sigma[v] = sum;
      cnt.add(tally, v);
    }
    wave_bits_set(next, v, found);
    wave_bits_set(visited, v, found);
  }
  __syncthreads();
  const int left = min(huges, kHuges);
  for (int i = 0; i < left; ++i) {  // uniform
    const int32_t v = huge[i];
    const int32_t b = t_rowptr[v], e = t_rowptr[v + 1];
    double part = 0.0;
    for (int64_t a0 = b; a0 < e; a0 += 4 * NT) {
      int32_t u[4];
      bool on[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) u[k] = t_col[static_cast<int32_t>(min<int64_t>(a0 + threadIdx.x + k * NT, e - 1))];
#pragma unroll
      for (int k = 0; k < 4; ++k) on[k] = a0 + threadIdx.x + k * NT < e && bit_test(front, u[k]);
#pragma unroll
      for (int k = 0; k < 4; ++k) part += on[k] ? sigma[u[k]] : 0.0;
    }
    part = gcd::wave_sum(part);
    __syncthreads();  // rows[] is read no more
    if (gcd::lane_id() == 0) rows[threadIdx.x / kWave].sum[0] = part;
    __syncthreads();
    if (threadIdx.x == 0) {
      double sum = 0.0;
      for (int w = 0; w < NT / kWave; ++w) sum += rows[w].sum[0];
      if (sum > 0.0) {
        depth[v] = level + 1;
        sigma[v] = sum;
        cnt.add(tally, v);
        atomicOr(&next[v >> 5], 1u << (v & 31));
        atomicOr(&visited[v >> 5], 1u << (v & 31));
      }
    }
  }
  publish_count<NT>(tally, cnt);
}

// TOCAB pull, per block: part[l] = sum of sigma over the active sources of
// this block among the in-arcs of local row l (0 when its vertex is visited).
__global__ __launch_bounds__(kThreads) void k_bc_tocab(const int32_t* __restrict__ row_ptr,
                                                       const int32_t* __restrict__ col,
                                                       const int32_t* __restrict__ id_map, int64_t P,
                                                       const uint32_t* __restrict__ visited,
                                                       const uint32_t* __restrict__ front,
                                                       const double* __restrict__ sigma, double* __restrict__ part) {
  __shared__ SigmaRows rows[kThreads / kWave];
  for (int64_t base = static_cast<int64_t>(blockIdx.x) * kThreads; base < P;
       base += static_cast<int64_t>(gridDim.x) * kThreads) {  // uniform per work-group
    const int64_t l = base + threadIdx.x;
    bool active = false;
    int32_t b = 0, e = 0;
    if (l < P && !bit_test(visited, id_map[l])) {
      active = true;
      b = row_ptr[l];
      e = row_ptr[l + 1];
    }
    const double sum = scan_sigma(col, front, sigma, active, b, e, rows[threadIdx.x / kWave]);
    if (l < P) part[l] = sum;
  }
}

// Merge of the per-block path counts over vertex range j (FP64 LDS sums),
// fused with the depth / sigma update and the next frontier.
template <int K, bool kFlat>
__global__ __launch_bounds__(kThreads) void k_bc_merge(const int32_t* __restrict__ range_ptr, int32_t B,
                                                       const uint16_t* __restrict__ id16,
                                                       const double* __restrict__ part, int32_t n,
                                                       int32_t* __restrict__ depth, int32_t level,
                                                       double* __restrict__ sigma, uint32_t* __restrict__ next,
                                                       uint32_t* __restrict__ visited, Tally tally) {
  __shared__ double acc[K];
  Counted cnt;
  gcm::merge_accumulate<K, kFlat, kThreads>(range_ptr, B, id16, part, blockIdx.x, acc);
  const int32_t v0 = blockIdx.x * K;
  for (int i = threadIdx.x; i < K; i += kThreads) {
    const int32_t v = v0 + i;
    const bool found = v < n && acc[i] > 0.0 && !bit_test(visited, v);
    if (found) {
      depth[v] = level + 1;
      sigma[v] = acc[i];
      cnt.add(tally, v);
    }
    wave_bits_set(next, v, found);
    wave_bits_set(visited, v, found);
  }
  publish_count<kThreads>(tally, cnt);
}

// ---------------------------------------------------------------------------
// Data-driven push, balanced over arcs. The queue's arc prefix cuts the
// concatenated out-arcs of the frontier into equal pieces, one per
// work-group, so a hub's arcs spread over many work-groups and a frontier of
// any shape takes one launch. A work-group finds its first vertex with a
// wave-wide search (64 probes per step), stages a window of the queue in
// LDS, and every thread locates its kA arcs there. What bounds a small level
// is the chain of dependent accesses (queue, row, column, value, atomic), so
// each step is issued for all of a thread's arcs before the next; what
// bounds a large one is the append, an atomic on one address, so a
// work-group takes tiles in turn and collects what they find in LDS until
// its buffer is full.
// The relaxation is a functor: src(u) loads what u passes along its arcs, and
// relax<kA>() does the atomics and returns the arcs whose target enters the
// next frontier.

struct BfsRelax {  // Algorithm 3's CAS on depth
  using Src = int32_t;
  int32_t* depth;
  int32_t level;
  __device__ Src src(int32_t) const { return 0; }
  template <int kA>
  __device__ uint32_t relax(uint32_t in, const int32_t (&v)[kA], const int32_t (&)[kA], const Src (&)[kA],
                            int32_t*) const {
    int32_t old[kA];
#pragma unroll
    for (int k = 0; k < kA; ++k) old[k] = (in >> k) & 1u ? depth[v[k]] : 0;
#pragma unroll
    for (int k = 0; k < kA; ++k) {
      const bool open = old[k] == kInf;
      old[k] = 0;
      if (open) old[k] = atomicCAS(&depth[v[k]], kInf, level + 1);
    }
    uint32_t took = 0;
#pragma unroll
    for (int k = 0; k < kA; ++k) took |= static_cast<uint32_t>(old[k] == kInf) << k;
    return took;
  }
};

struct SsspRelax {  // atomicMin on dist; a vertex is queued once per round (stamp in mark)
  using Src = int32_t;
  const int32_t* w;
  int32_t* dist;
  int32_t round;
  int32_t* mark;
  __device__ Src src(int32_t u) const { return dist[u]; }
  template <int kA>
  __device__ uint32_t relax(uint32_t in, const int32_t (&v)[kA], const int32_t (&e)[kA], const Src (&du)[kA],
                            int32_t* stats) const {
    int32_t nd[kA], old[kA];
    bool over = false;
#pragma unroll
    for (int k = 0; k < kA; ++k) {
      nd[k] = (in >> k) & 1u ? w[e[k]] : 0;
      old[k] = (in >> k) & 1u ? dist[v[k]] : 0;
    }
#pragma unroll
    for (int k = 0; k < kA; ++k) {
      const int64_t d = static_cast<int64_t>(du[k]) + nd[k];
      const bool on = (in >> k) & 1u;
      over |= on && d >= kInf;
      nd[k] = on && d < kInf ? static_cast<int32_t>(d) : kInf;
    }
    if (over) stats[kOverflow] = 1;
#pragma unroll
    for (int k = 0; k < kA; ++k) {
      const bool better = nd[k] < old[k];
      old[k] = INT32_MIN;
      if (better) old[k] = atomicMin(&dist[v[k]], nd[k]);
    }
#pragma unroll
    for (int k = 0; k < kA; ++k) {
      const bool won = nd[k] < old[k];
      old[k] = round;
      if (won) old[k] = atomicExch(&mark[v[k]], round);
    }
    uint32_t took = 0;
#pragma unroll
    for (int k = 0; k < kA; ++k) took |= static_cast<uint32_t>(old[k] != round) << k;
    return took;
  }
};

struct BcRelax {  // the BFS CAS plus sigma[v] += sigma[u] (FP64 atomic) for arcs that land one level down
  using Src = double;
  int32_t* depth;
  int32_t level;
  double* sigma;
  __device__ Src src(int32_t u) const { return sigma[u]; }
  template <int kA>
  __device__ uint32_t relax(uint32_t in, const int32_t (&v)[kA], const int32_t (&)[kA], const Src (&su)[kA],
                            int32_t*) const {
    int32_t old[kA];
    uint32_t took = 0;
#pragma unroll
    for (int k = 0; k < kA; ++k) old[k] = (in >> k) & 1u ? depth[v[k]] : 0;
#pragma unroll
    for (int k = 0; k < kA; ++k)
      if (old[k] == kInf) {
        old[k] = atomicCAS(&depth[v[k]], kInf, level + 1);
        if (old[k] == kInf) took |= 1u << k;
      }
#pragma unroll
    for (int k = 0; k < kA; ++k)
      if (((in >> k) & 1u) && (old[k] == kInf || old[k] == level + 1)) atomicAdd(&sigma[v[k]], su[k]);
    return took;
  }
};

// The last i in [0, qn) with pre[i] <= a (pre ascends, pre[0] <= a), by the
// whole wave.
__device__ __forceinline__ int32_t wave_owner(const int32_t* __restrict__ pre, int32_t qn, int32_t a) {
  const int lane = gcd::lane_id();
  int32_t lo = 0, hi = qn - 1;
  while (lo < hi) {  // uniform
    const int32_t step = (hi - lo + kWave - 1) / kWave;
    const int32_t idx = static_cast<int32_t>(min<int64_t>(hi, lo + static_cast<int64_t>(lane + 1) * step));
    const int cnt = __popcll(__ballot(pre[idx] <= a));  // a prefix of the lanes
    const int32_t fail = static_cast<int32_t>(min<int64_t>(hi, lo + static_cast<int64_t>(cnt + 1) * step));
    lo = static_cast<int32_t>(min<int64_t>(hi, lo + static_cast<int64_t>(cnt) * step));
    if (cnt < kWave) hi = fail - 1;
  }
  return lo;
}

// One arc per thread up to 64 tiles of them (the latency of a level is
// least, and so few appends cost little), four beyond.
constexpr int64_t kPushOneArc = 64 * kThreads;

template <class Relax, int kA>
__global__ __launch_bounds__(kThreads) void k_push(const int32_t* __restrict__ queue_in,
                                                   const int32_t* __restrict__ pre, int32_t qn, int32_t arcs,
                                                   const int32_t* __restrict__ rowptr,
                                                   const int32_t* __restrict__ colidx, Relax r, Sink sink) {
  constexpr int kWin = kA == 1 ? kThreads : 2 * kThreads;  // queue entries staged at a time
  constexpr int kTile = kThreads * kA;                     // arcs
  constexpr int kPer = kA == 1 ? 1 : 12;                   // buffered vertices per thread
  constexpr int kBuf = kThreads * kPer;
  static_assert(kBuf >= kTile, "a tile's vertices fit the empty buffer");
  __shared__ int32_t w_pre[kWin], w_row[kWin], buf[kBuf];
  __shared__ typename Relax::Src w_src[kWin];
  __shared__ int32_t first, held;
  const int tid = threadIdx.x;
  stamp_start(sink.stats);
  if (tid == 0) held = 0;
  for (int64_t t0 = static_cast<int64_t>(blockIdx.x) * kTile; t0 < arcs;
       t0 += static_cast<int64_t>(gridDim.x) * kTile) {  // uniform
    const int32_t a0 = static_cast<int32_t>(t0);
    const int32_t a1 = static_cast<int32_t>(min<int64_t>(arcs, t0 + kTile));
    if (tid < kWave) {
      const int32_t i = wave_owner(pre, qn, a0);
      if (tid == 0) first = i;
    }
    __syncthreads();
    int32_t v[kA];
    uint32_t took = 0;
#pragma unroll
    for (int k = 0; k < kA; ++k) v[k] = 0;
    // one window nearly always; more where vertices without out-arcs stand between
    for (int32_t base = first; base < qn; base += kWin) {  // uniform
#pragma unroll
      for (int t = tid; t < kWin; t += kThreads) {
        const int32_t i = base + t;
        int32_t p = INT32_MAX, row = 0;
        typename Relax::Src x{};
        if (i < qn) {
          const int32_t u = queue_in[i];
          p = pre[i];
          row = rowptr[u] - p;
          x = r.src(u);
        }
        w_pre[t] = p;
        w_row[t] = row;
        w_src[t] = x;
      }
      const int32_t next = base + kWin < qn ? pre[base + kWin] : arcs;
      __syncthreads();
      const int32_t from = w_pre[0];
      int32_t e[kA];
      typename Relax::Src x[kA];
      uint32_t in = 0;
#pragma unroll
      for (int k = 0; k < kA; ++k) {
        const int64_t a = t0 + tid + k * kThreads;
        const bool here = a >= from && a < next && a < a1;
        int lo = 0;  // the last entry with w_pre <= a
#pragma unroll
        for (int step = kWin / 2; step > 0; step >>= 1)
          if (w_pre[lo + step] <= a) lo += step;
        e[k] = here ? static_cast<int32_t>(a) + w_row[lo] : 0;
        x[k] = w_src[lo];
        in |= static_cast<uint32_t>(here) << k;
      }
      int32_t to[kA];
#pragma unroll
      for (int k = 0; k < kA; ++k) to[k] = (in >> k) & 1u ? colidx[e[k]] : 0;
      took |= r.template relax<kA>(in, to, e, x, sink.stats);
#pragma unroll
      for (int k = 0; k < kA; ++k) v[k] = (in >> k) & 1u ? to[k] : v[k];
      if (next >= a1) break;
      __syncthreads();  // the window is refilled
    }
    // what the tile found goes to the buffer, one LDS atomic per wave
    int32_t total = 0, before[kA];
#pragma unroll
    for (int k = 0; k < kA; ++k) {
      const uint64_t m = __ballot((took >> k) & 1u);
      before[k] = total + __popcll(m & gcd::lanemask_lt());
      total += __popcll(m);
    }
    if (total) {  // uniform over the wave
      int32_t at = 0;
      if (gcd::lane_id() == 0) at = atomicAdd(&held, total);
      at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
      for (int k = 0; k < kA; ++k)
        if ((took >> k) & 1u) buf[at + before[k]] = v[k];
    }
    __syncthreads();
    const int32_t c = held;
    const bool last = t0 + static_cast<int64_t>(gridDim.x) * kTile >= arcs;
    if (c > 0 && (last || c + kTile > kBuf)) {  // uniform
      int32_t u[kPer], deg[kPer];
#pragma unroll
      for (int j = 0; j < kPer; ++j) u[j] = buf[min(tid + j * kThreads, c - 1)];
#pragma unroll
      for (int j = 0; j < kPer; ++j) deg[j] = sink.rowptr[u[j] + 1] - sink.rowptr[u[j]];
      uint64_t mine = 0, in = 0;
#pragma unroll
      for (int j = 0; j < kPer; ++j) mine += tid + j * kThreads < c ? one_vertex(deg[j]) : 0ull;
      if (sink.t_rowptr) {  // uniform
        int32_t di[kPer];
#pragma unroll
        for (int j = 0; j < kPer; ++j) di[j] = sink.t_rowptr[u[j] + 1] - sink.t_rowptr[u[j]];
#pragma unroll
        for (int j = 0; j < kPer; ++j) in += tid + j * kThreads < c ? static_cast<uint64_t>(di[j]) : 0ull;
      }
      uint64_t at = wg_count<kThreads, true>(mine, in, sink.t_rowptr != nullptr, sink.stats, sink.counter);
#pragma unroll
      for (int j = 0; j < kPer; ++j) {
        if (tid + j * kThreads < c) {
          sink_put(sink, at, u[j]);
          at += one_vertex(deg[j]);
        }
      }
      if (tid == 0) held = 0;  // added to again after the next tile's barriers
    }
  }
}

__global__ void k_order_degree(const int32_t* __restrict__ order, int32_t cnt, const int32_t* __restrict__ rowptr,
                               int32_t* __restrict__ deg) {
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < cnt) {
    const int32_t v = order[i];
    deg[i] = rowptr[v + 1] - rowptr[v];
  }
}

// Backward sweep. coef[v] = (1 + delta[v]) / sigma[v]; two arrays alternate
// from level to level. When depth d is processed, the array it reads holds
// the coefficients of depth d + 1 and zero for depth d and every depth above
// (an arc from depth d reaches depth d + 1 at most), so the sum over all
// out-arcs of coef needs no depth test; the array it writes is zero at the
// vertices of depth d.
//
// A step walks the arcs of the vertices order[lo, hi), concatenated in level
// order (pre = their prefix), in tiles of one work-group, cut like k_push's:
// the tile's first vertex by a wave-wide search, a window of the level in
// LDS, every thread's arcs located there.
//
// kPush false: over the out-arcs of the level at depth d, coef_in of the
// targets is added up per vertex in LDS and stored, or added with one FP64
// atomic where the vertex's arcs go on in another tile.
// kPush true, chosen where the next level's in-arcs are few: over the
// in-arcs v -> w of the vertices at depth d + 1, coef_in[w] is added into
// coef_out[v] for every v of depth d (FP64 atomic).
// The sums are bound by the gathers (110 G arcs/s: 11.7 M arcs of an R-MAT
// graph of 2^20 vertices 106 us), the pushes by the atomics on hubs (4.2 M
// arcs 194 us). 1.5 M arcs of 255 K vertices took 75 us when each lane
// searched the level for its eight arcs alone and loaded their vertices one
// after the other, 19 us so.
template <bool kPush, int kA>
__global__ __launch_bounds__(kThreads) void k_bc_back(const int32_t* __restrict__ rowptr,
                                                      const int32_t* __restrict__ colidx,
                                                      const int32_t* __restrict__ order,
                                                      const int32_t* __restrict__ pre, int32_t qn, int32_t arcs,
                                                      const int32_t* __restrict__ depth, int32_t d,
                                                      const double* __restrict__ coef_in,
                                                      double* __restrict__ coef_out) {
  constexpr int kWin = kA == 1 ? kThreads : 2 * kThreads;
  constexpr int kTile = kThreads * kA;
  constexpr int kPad = kPush ? 1 : kTile + kTile / 32;  // a word apart every 32: a thread's kA are neighbours
  __shared__ int32_t w_pre[kWin], w_row[kWin];
  __shared__ double w_sum[kWin];  // kPush: coefficient of the entry, else its sum
  __shared__ double val[kPad];
  __shared__ int16_t own[kPad];
  __shared__ int32_t first;
  const int tid = threadIdx.x;
  const int32_t off = pre[0];
  const int64_t t0 = static_cast<int64_t>(blockIdx.x) * kTile;  // the tile's arcs, from the level's first
  const int32_t a0 = static_cast<int32_t>(t0);
  const int32_t a1 = static_cast<int32_t>(min<int64_t>(arcs, t0 + kTile));
  if (tid < kWave) {
    const int32_t i = wave_owner(pre, qn, a0 + off);
    if (tid == 0) first = i;
  }
  __syncthreads();
  for (int32_t base = first; base < qn; base += kWin) {  // uniform; one window nearly always
#pragma unroll
    for (int t = tid; t < kWin; t += kThreads) {
      const int32_t i = base + t;
      int32_t p = INT32_MAX, row = 0;
      double x = 0.0;
      if (i < qn) {
        const int32_t u = order[i];
        p = pre[i] - off;
        row = rowptr[u] - p;
        if constexpr (kPush) x = coef_in[u];
      }
      w_pre[t] = p;
      w_row[t] = row;
      w_sum[t] = x;
    }
    const int32_t next = base + kWin < qn ? pre[base + kWin] - off : arcs;
    __syncthreads();
    const int32_t from = w_pre[0];
    int32_t e[kA], at[kA];
    uint32_t in = 0;
#pragma unroll
    for (int k = 0; k < kA; ++k) {
      const int64_t a = t0 + tid + k * kThreads;
      const bool here = a >= from && a < next && a < a1;
      int lo = 0;  // the last entry with w_pre <= a
#pragma unroll
      for (int step = kWin / 2; step > 0; step >>= 1)
        if (w_pre[lo + step] <= a) lo += step;
      at[k] = lo;
      e[k] = here ? static_cast<int32_t>(a) + w_row[lo] : 0;
      in |= static_cast<uint32_t>(here) << k;
    }
    int32_t to[kA];
#pragma unroll
    for (int k = 0; k < kA; ++k) to[k] = (in >> k) & 1u ? colidx[e[k]] : 0;
    if constexpr (kPush) {
      int32_t dv[kA];
#pragma unroll
      for (int k = 0; k < kA; ++k) dv[k] = (in >> k) & 1u ? depth[to[k]] : d + 1;
#pragma unroll
      for (int k = 0; k < kA; ++k)
        if (dv[k] == d) atomicAdd(&coef_out[to[k]], w_sum[at[k]]);
    } else {
      double c[kA];
#pragma unroll
      for (int k = 0; k < kA; ++k) c[k] = (in >> k) & 1u ? coef_in[to[k]] : 0.0;
#pragma unroll
      for (int k = 0; k < kA; ++k) {
        const int i = tid + k * kThreads;
        val[i + i / 32] = c[k];
        own[i + i / 32] = (in >> k) & 1u ? static_cast<int16_t>(at[k]) : int16_t{-1};
      }
      __syncthreads();
      // kA neighbouring arcs per thread: one LDS atomic per run of a vertex,
      // one per wave where a vertex has all its arcs
      double sum = 0.0;
      const int l0 = tid * kA + tid * kA / 32;
      int who = own[l0];
      bool one = who >= 0;
#pragma unroll
      for (int k = 0; k < kA; ++k) {
        const int i = tid * kA + k;
        const int o = own[i + i / 32];
        if (o != who) {
          if (who >= 0) atomicAdd(&w_sum[who], sum);
          sum = 0.0;
          who = o;
          one = false;
        }
        sum += val[i + i / 32];
      }
      const int lead = __builtin_amdgcn_readfirstlane(who);
      if (__all(one && who == lead)) {
        sum = gcd::wave_sum(sum);
        if (gcd::lane_id() == 0) atomicAdd(&w_sum[who], sum);
      } else if (who >= 0) {
        atomicAdd(&w_sum[who], sum);
      }
      __syncthreads();
#pragma unroll
      for (int t = tid; t < kWin; t += kThreads) {
        const int32_t i = base + t;
        if (i >= qn) break;
        const int32_t p = w_pre[t], q = t + 1 < kWin && i + 1 < qn ? w_pre[t + 1] : next;
        if (p >= a1 || q <= a0 || p == q) continue;  // no arc in the tile
        if (p >= a0 && q <= a1) coef_out[order[i]] = w_sum[t];
        else if (w_sum[t] != 0.0) atomicAdd(&coef_out[order[i]], w_sum[t]);
      }
    }
    if (next >= a1) break;
    __syncthreads();  // the window is refilled
  }
}

// The step of depth d is pushed where the in-arcs below are fewer than a
// sixth of the level's out-arcs: an arc costs 50 to 70 ps pushed, 9 ps pulled
// (4.2 M against 11.7 M: 194 us pushed, 106 pulled; 0.9 M against 13.6 M: 62
// and 114; 41 K against 4.1 M: 14 and 43).
inline bool back_pushes(int64_t in_next, int64_t out_arcs) { return 6 * in_next < out_arcs; }

// One step: the arcs of the qn vertices at `order`, one per thread up to
// kPushOneArc of them (k_push's reason), four beyond.
template <bool kPush>
hipError_t bc_back(const int32_t* rowptr, const int32_t* colidx, const int32_t* order, const int32_t* pre, int32_t qn,
                   int64_t arcs, const int32_t* depth, int32_t d, const double* coef_in, double* coef_out,
                   hipStream_t s) {
  const int32_t m = static_cast<int32_t>(arcs);
  if (m == 0) return hipSuccess;
  if (arcs <= kPushOneArc)
    k_bc_back<kPush, 1><<<(m + kThreads - 1) / kThreads, kThreads, 0, s>>>(rowptr, colidx, order, pre, qn, m, depth, d,
                                                                           coef_in, coef_out);
  else
    k_bc_back<kPush, 4><<<static_cast<int32_t>((arcs + 4 * kThreads - 1) / (4 * kThreads)), kThreads, 0, s>>>(
        rowptr, colidx, order, pre, qn, m, depth, d, coef_in, coef_out);
  return hipGetLastError();
}

// delta[v] = sigma[v] * (sum held in coef[v]) is added into bc[v], and
// coef[v] becomes (1 + delta[v]) / sigma[v].
__global__ void k_bc_finish(const int32_t* __restrict__ order, int32_t cnt, const double* __restrict__ sigma,
                            double* __restrict__ coef, double* __restrict__ bc) {
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < cnt) {
    const int32_t v = order[i];
    const double sg = sigma[v];
    const double d = sg * coef[v];
    bc[v] += d;
    coef[v] = (1.0 + d) / sg;
  }
}

template <int K>
struct BcMerge {
  template <class... A>
  static void run(int32_t R, hipStream_t s, const int32_t* range_ptr, int32_t B, A... a) {
    if (B <= gcm::kFlatB) k_bc_merge<K, true><<<R, kThreads, 0, s>>>(range_ptr, B, a...);
    else k_bc_merge<K, false><<<R, kThreads, 0, s>>>(range_ptr, B, a...);
  }
};

// Work-groups for one item per thread. Item counts here are vertex, queue
// or arc counts below 2^31, so the grid never needs a cap.
inline int grid_for(int64_t items, int threads) {
  return static_cast<int>(std::max<int64_t>(1, (items + threads - 1) / threads));
}

// Work-groups of the grid-stride TOCAB row kernels: at most kRowGrid, so
// partitions with more than kRowGrid * kThreads local rows take several
// passes (RMAT-24 partitions do).
constexpr int64_t kRowGrid = 1 << 16;
inline int row_grid(int64_t rows) {
  return static_cast<int>(std::max<int64_t>(1, std::min<int64_t>((rows + kThreads - 1) / kThreads, kRowGrid)));
}

enum class Mode { kPull, kTocab, kPush };

// Direction choice (Section 3.3): with the direction-optimising rule of
// Beamer et al. (the paper's [Direction] reference; alpha = 14, beta = 24)
// a level pulls when the frontier's out-arcs exceed the unexplored arcs /
// alpha and returns to push when the frontier shrinks below n / beta. A
// pull level is blocked (TOCAB) when its working set exceeds the cache: the
// frontier must be large (4 bytes per frontier out-arc above one XCD's L2,
// the paper's test) and the array its random reads land in must not fit in
// that L2 either. With one status bit per vertex a BFS pull reads only the
// bitmap (n / 8 bytes: 2 MB at 2^24 vertices, so plain pull's reads already
// hit L2 and blocking only adds its local rows); an SSSP pull also gathers
// the 4-byte distances of active sources.
struct Heuristic {
  static constexpr double kAlpha = 14.0, kBeta = 24.0;
  static constexpr double kCacheBytes = 4.0 * 1024 * 1024;  // one XCD's L2
  // BFS over a stream-layout partition: TOCAB pull on graphs with at most
  // kBfsTocabVertices vertices and kBfsTocabDegree arcs per vertex, while at
  // least 1/64 of the arcs still end at unvisited vertices; else plain pull.
  // The plain pull is the faster since a wave walks its rows end to end
  // (early exit, status bits in L2). A whole BFS with the TOCAB arm and
  // without: grids of 160,000, 10^6, 4 and 8 M vertices 501, 668, 1052, 1616
  // us against 453, 553, 772, 1163; uniform of 8 arcs per vertex 229, 317, 604,
  // 879 against 209, 273, 525, 758; R-MAT of 8 194, 252, 370, 440 against 174,
  // 201, 300, 340. So the arm is not the faster form at any size: up to 2^18
  // vertices, where it costs some 10 us per level, it stays as the header
  // describes it and traversal_trace shows it; beyond, its cost grows with n.
  static constexpr int64_t kBfsTocabVertices = int64_t{1} << 18;
  static constexpr double kBfsTocabShare = 1.0 / 64.0;
  static constexpr double kBfsTocabDegree = 10.0;
  bool pulling = false;
  // m_u: unexplored out-arcs (the direction test); m_u_in: in-arcs of the
  // unvisited vertices; stream: the TOCAB partition has the stream layout
  Mode pick(int64_t n, int64_t n_f, int64_t m_f, int64_t m_u, bool have_tocab, bool bfs, int64_t m = 0,
            int64_t m_u_in = 0, bool stream = false) {
    if (!pulling && static_cast<double>(m_f) > static_cast<double>(m_u) / kAlpha) pulling = true;
    else if (pulling && static_cast<double>(n_f) < static_cast<double>(n) / kBeta) pulling = false;
    if (!pulling) return Mode::kPush;
    if (bfs && have_tocab && stream)
      return n <= kBfsTocabVertices && static_cast<double>(m) <= kBfsTocabDegree * static_cast<double>(n) &&
                     static_cast<double>(m_u_in) >= kBfsTocabShare * static_cast<double>(m)
                 ? Mode::kTocab
                 : Mode::kPull;
    const double gathered = static_cast<double>(n) / 8.0 + (bfs ? 0.0 : 4.0 * static_cast<double>(n));
    const bool large = 4.0 * static_cast<double>(m_f) > kCacheBytes && gathered > kCacheBytes;
    return (have_tocab && large) ? Mode::kTocab : Mode::kPull;
  }
};

using gcx::kLearnedGate;

template <template <int> class Kern, class... Args>
hipError_t launch_by_k(int32_t k, int32_t R, hipStream_t s, Args... args) {
  switch (k) {
    case 256: Kern<256>::run(R, s, args...); break;
    case 512: Kern<512>::run(R, s, args...); break;
    case 1024: Kern<1024>::run(R, s, args...); break;
    case 2048: Kern<2048>::run(R, s, args...); break;
    case 4096: Kern<4096>::run(R, s, args...); break;
    case 8192: Kern<8192>::run(R, s, args...); break;
    case 16384: Kern<16384>::run(R, s, args...); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int K>
struct BfsMerge {
  template <class... A>
  static void run(int32_t R, hipStream_t s, const int32_t* range_ptr, int32_t B, A... a) {
    if (B <= gcm::kFlatB) k_bfs_merge<K, true><<<R, kThreads, 0, s>>>(range_ptr, B, a...);
    else k_bfs_merge<K, false><<<R, kThreads, 0, s>>>(range_ptr, B, a...);
  }
};

template <int K>
struct SsspMerge {
  template <class... A>
  static void run(int32_t R, hipStream_t s, const int32_t* range_ptr, int32_t B, A... a) {
    if (B <= gcm::kFlatB) k_sssp_merge<K, true><<<R, kThreads, 0, s>>>(range_ptr, B, a...);
    else k_sssp_merge<K, false><<<R, kThreads, 0, s>>>(range_ptr, B, a...);
  }
};

// Compute units of the GPU (read once).
int32_t device_cus() {
  static const int32_t cus = [] {
    int dev = 0, c = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) !=
                                                 hipSuccess || c <= 0)
      c = 256;
    return c;
  }();
  return cus;
}

template <int K>
struct SsspMergeStream {
  // LDS minima of K int32: two work-groups per CU; no more threads than K
  static constexpr int kNT = K >= 8192 ? 1024 : (K >= 512 ? 512 : K);
  template <class... A>
  static void run(int32_t R, hipStream_t s, A... a) {
    const int32_t grid = std::max(1, std::min(R, 2 * device_cus()));
    k_sssp_merge_stream<K, kNT, false><<<grid, kNT, 0, s>>>(a...);
  }
};

template <int K>
struct BfsMergeStream {
  static constexpr int kNT = SsspMergeStream<K>::kNT;
  template <class... A>
  static void run(int32_t R, hipStream_t s, A... a) {
    const int32_t grid = std::max(1, std::min(R, 2 * device_cus()));
    k_sssp_merge_stream<K, kNT, true><<<grid, kNT, 0, s>>>(a...);
  }
};

// *flag = 1 if a weight lies outside [0, 255].
__global__ void k_weight_range(const int32_t* __restrict__ w, int64_t m, int32_t* __restrict__ flag) {
  bool wide = false;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < m;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    wide |= static_cast<uint32_t>(w[i]) > 255u;
  if (__any(wide) && gcd::lane_id() == 0) *flag = 1;
}

// Weights as bytes in arc order, zero past m.
__global__ void k_weight_bytes(const int32_t* __restrict__ w, int64_t m, int64_t m_pad, uint8_t* __restrict__ w8) {
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < m_pad;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    w8[i] = i < m ? static_cast<uint8_t>(w[i]) : 0;
}

// One device int32 for the weight check (per process, allocated once).
int32_t* g_range_flag() {
  static int32_t* flag = [] {
    void* p = nullptr;
    return hipMalloc(&p, sizeof(int32_t)) == hipSuccess ? static_cast<int32_t*>(p) : nullptr;
  }();
  return flag;
}

// The LDS limit of the stream-layout traversal pull (a block's values and
// its chunk's position table).
hipError_t stream_pull_setup() {
  static const hipError_t attr = [] {
    const int lds = gcx::lds_budget(gcx::kLdsMaxWidth) + static_cast<int>(sizeof(int32_t)) * kLdsWaves;
    hipError_t e = hipSuccess;
    for (const void* k : {reinterpret_cast<const void*>(&k_sssp_tocab_lds<kW32>),
                          reinterpret_cast<const void*>(&k_sssp_tocab_lds<kW8>),
                          reinterpret_cast<const void*>(&k_sssp_tocab_lds<kWNone>)})
      if (e == hipSuccess) e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    return e;
  }();
  return attr;
}

// Integer weights of a stream-layout partition in its arc order, padded with
// zeros to the layout's length (built by the first SSSP round over it), and
// the LDS limit of the kernel that reads them.
hipError_t stream_weights(gc_tocab t, hipStream_t s) {
  GC_HIP_TRY(stream_pull_setup());
  if (t->w_pad || t->w8) return hipSuccess;
  if (!t->w) return hipErrorInvalidValue;
  // one byte per weight when every weight fits (checked once, on the device)
  int32_t* flag = g_range_flag();
  if (!flag) return hipErrorOutOfMemory;
  GC_HIP_TRY(hipMemsetAsync(flag, 0, sizeof(int32_t), s));
  if (t->m > 0) k_weight_range<<<grid_for(t->m, kThreads), kThreads, 0, s>>>(t->w, t->m, flag);
  GC_HIP_TRY(hipGetLastError());
  int32_t wide = 0;
  GC_HIP_TRY(hipMemcpyAsync(&wide, flag, sizeof(int32_t), hipMemcpyDeviceToHost, s));
  GC_HIP_TRY(hipStreamSynchronize(s));
  if (!wide) {
    t->w8 = static_cast<uint8_t*>(gcx::dev_alloc(static_cast<size_t>(t->m_pad), s));
    if (!t->w8) return hipErrorOutOfMemory;
    t->bytes += t->m_pad;
    k_weight_bytes<<<grid_for(t->m_pad, kThreads), kThreads, 0, s>>>(t->w, t->m, t->m_pad, t->w8);
    return hipGetLastError();
  }
  t->w_pad = static_cast<int32_t*>(gcx::dev_alloc(sizeof(int32_t) * static_cast<size_t>(t->m_pad), s));
  if (!t->w_pad) return hipErrorOutOfMemory;
  t->bytes += static_cast<int64_t>(sizeof(int32_t)) * t->m_pad;
  if (t->m > 0) GC_HIP_TRY(hipMemcpyAsync(t->w_pad, t->w, sizeof(int32_t) * t->m, hipMemcpyDeviceToDevice, s));
  return hipMemsetAsync(t->w_pad + t->m, 0, sizeof(int32_t) * (t->m_pad - t->m), s);
}

// Waits until the pinned mirror holds level `seq`'s counters.
hipError_t wait_stats(gc_graph g, int32_t seq, hipStream_t s) {
  return gcx::wait_mirror(g->stats_host + gcx::kStatSeq, seq, s);
}

// Work-groups for a pass over `items`, each thread striding over them.
inline int stride_grid(int64_t items) {
  return static_cast<int>(std::max<int64_t>(1, std::min<int64_t>((items + kThreads - 1) / kThreads, 8 * device_cus())));
}

// Per-level bookkeeping: the frontier's queue and status words, and the
// counters of the next one.
struct Frontier {
  gc_graph g;
  hipStream_t s;
  int32_t* q[2];  // queues and their arc prefixes, the current and the next level's in turn
  int32_t* p[2];
  int cur = 0;
  int32_t n_f = 1;
  int64_t m_f = 0;
  int64_t m_f_in = 0;  // in-arcs of the frontier when count_in (the source's are not counted)
  bool count_in = false;
  bool queue_ok = true;            // queue and pre hold the current frontier
  bool bits_ok = false;            // front (and visited) hold the current frontier
  bool dirty[2] = {false, false};  // status words of [cur] / [cur ^ 1] may be set
  bool clearing = false;           // the last level's end zeroes status words, which nothing has waited for
  Frontier(gc_graph gr, hipStream_t st)
      : g(gr), s(st), q{gr->queue[0], gr->queue[1]}, p{gr->arc_pre, gr->arc_deg} {}
  uint32_t* front() { return cur == 0 ? g->front : g->next; }
  uint32_t* next() { return cur == 0 ? g->next : g->front; }
  int32_t* queue() { return q[cur]; }
  int32_t* pre() { return p[cur]; }
  int32_t* queue_next() { return q[cur ^ 1]; }
  int64_t words() const { return (static_cast<int64_t>(g->n) + 31) / 32; }
  Sink sink() {
    return Sink{q[cur ^ 1], p[cur ^ 1], g->rowptr, count_in ? g->t_rowptr : nullptr, g->stats};
  }
  Tally tally() { return Tally{g->rowptr, count_in ? g->t_rowptr : nullptr, g->stats}; }

  // Start of a traversal from `src`: the value array (and what else is
  // given), the frontier {src}; m_f = its out-degree.
  hipError_t start(int32_t src, int32_t* value, int32_t* mark, double* sigma, double* coef) {
    if (!g->bits_clean) {
      k_fill_i32<<<stride_grid(words()), kThreads, 0, s>>>(reinterpret_cast<int32_t*>(g->front), words(), 0);
      k_fill_i32<<<stride_grid(words()), kThreads, 0, s>>>(reinterpret_cast<int32_t*>(g->next), words(), 0);
    }
    g->bits_clean = false;  // until the traversal has ended well
    const int32_t seq = static_cast<int32_t>(++g->level_seq);
    k_start<<<stride_grid(g->n), kThreads, 0, s>>>(g->n, src, g->rowptr, value, mark, sigma, coef, q[0], p[0], g->stats,
                                                   g->stats_host, seq);
    GC_HIP_TRY(hipGetLastError());
    GC_HIP_TRY(wait_stats(g, seq, s));
    m_f = static_cast<uint32_t>(g->stats_host[gcx::kStatArcs]);
    return hipSuccess;
  }

  // Before a pull level: the status words of the frontier (and, for BFS and
  // BC, of the visited vertices) when the previous level was a push.
  hipError_t need_bits(const int32_t* depth, int32_t level) {
    if (bits_ok) return hipSuccess;
    if (depth)
      k_bits_from_depth<<<grid_for(g->n, kThreads), kThreads, 0, s>>>(depth, g->n, level, front(), g->visited);
    else
      k_bits_from_queue<<<grid_for(n_f, kThreads), kThreads, 0, s>>>(queue(), n_f, front());
    dirty[cur] = true;
    bits_ok = true;
    return hipGetLastError();
  }

  // Before a push level: the queue, when the previous level was a pull.
  hipError_t need_queue() {
    if (queue_ok) return hipSuccess;
    Sink to{q[cur], p[cur], g->rowptr, nullptr, g->stats, gcx::kStatBuild};
    // up to 512 work-groups, an atomic each, at 2^22 vertices and 2^24
    if (words() <= 512 * kThreads)
      k_queue_from_bits<1><<<grid_for(words(), kThreads), kThreads, 0, s>>>(front(), words(), to);
    else
      k_queue_from_bits<4><<<grid_for(words(), 4 * kThreads), kThreads, 0, s>>>(front(), words(), to);
    queue_ok = true;
    return hipGetLastError();
  }

  // Device time of the level just ended (its relaxation kernels), in ms,
  // from the clock stamps in the host mirror.
  double level_ms() const {
    const uint64_t t0 = *reinterpret_cast<const uint64_t*>(g->stats_host + gcx::kStatT0);
    const uint64_t t1 = *reinterpret_cast<const uint64_t*>(g->stats_host + gcx::kStatT1);
    return t1 > t0 ? static_cast<double>(t1 - t0) / g->clock_khz : 0.0;
  }

  // Ends a level (pull: it set the next frontier's status words): queues the
  // learned scheduler's decision for the next level when `decide` is given
  // (read back with the counters, so it costs no synchronisation of its
  // own), and reads the counters.
  hipError_t end_level(bool pull, bool* overflow, gc_sched decide = nullptr, int32_t next_level = 0,
                       LevelDecide dec = LevelDecide()) {
    size_t lds = 0;
    if (decide) {
      dec.params = gcx::sched_params(decide);
      dec.frange = gcx::sched_range(decide);
      dec.K = gcx::sched_actions(decide);
      dec.n = g->n;
      dec.m = g->m;
      dec.level = next_level;
      dec.prior_arcs = m_f;
      dec.clock_khz = g->clock_khz;
      lds = level_decide_lds(dec.K);
    }
    const int32_t seq = static_cast<int32_t>(++g->level_seq);
    const bool clear = dirty[cur];
    const int grid = clear && words() > kClearFirst ? stride_grid(words()) : 1;
    clearing = grid > 1;
    k_level_end<<<grid, kThreads, lds, s>>>(g->stats, g->stats_host, seq, dec, clear ? front() : nullptr, words());
    dirty[cur] = false;
    if (pull) dirty[cur ^ 1] = true;
    bits_ok = pull;
    queue_ok = !pull;
    GC_HIP_TRY(hipGetLastError());
    GC_HIP_TRY(wait_stats(g, seq, s));
    n_f = g->stats_host[gcx::kStatQLen];
    m_f = static_cast<uint32_t>(g->stats_host[gcx::kStatArcs]);
    m_f_in = static_cast<int64_t>(static_cast<uint32_t>(g->stats_host[gcx::kStatInDegLo])) |
             (static_cast<int64_t>(g->stats_host[gcx::kStatInDegLo + 1]) << 32);
    if (overflow && g->stats_host[kOverflow]) *overflow = true;
    cur ^= 1;
    return hipSuccess;
  }

  // End of a traversal: no status bit is set when its last level found
  // nothing. A level's end tells the host its counts while other work-groups
  // may still zero status words, so a traversal that ends there waits for
  // them: the handle's next user may come on another stream.
  hipError_t finish() {
    if (clearing) GC_HIP_TRY(gcx::wait_queued(g, s));
    g->bits_clean = n_f == 0;
    return hipSuccess;
  }
};

// Push of one level with relaxation r, in at most four work-groups per CU.
template <class Relax>
hipError_t push_level(gc_graph g, Frontier& f, Relax r, hipStream_t s) {
  if (f.m_f == 0) return hipSuccess;
  GC_HIP_TRY(f.need_queue());
  const int32_t arcs = static_cast<int32_t>(f.m_f);
  if (f.m_f <= kPushOneArc)
    k_push<Relax, 1><<<grid_for(arcs, kThreads), kThreads, 0, s>>>(f.queue(), f.pre(), f.n_f, arcs, g->rowptr, g->colidx,
                                                                   r, f.sink());
  else
    k_push<Relax, 4><<<std::min(grid_for(arcs, 4 * kThreads), 4 * device_cus()), kThreads, 0, s>>>(
        f.queue(), f.pre(), f.n_f, arcs, g->rowptr, g->colidx, r, f.sink());
  return hipGetLastError();
}

// Grid of a pull over all vertices: two work-groups of 1024 threads per CU
// (the most that are resident), smaller ones for graphs that would not give
// every CU one.
constexpr int kPullThreads = 1024;
inline bool wide_pull(int32_t n) { return n >= 2 * kPullThreads * device_cus(); }
inline int pull_grid(int32_t n) {
  return wide_pull(n) ? std::min(grid_for(n, kPullThreads), 2 * device_cus())
                      : std::min(grid_for(n, kThreads), 4 * device_cus());
}

// Enqueues one level (BFS depth `level` -> level+1, or SSSP round `level`)
// in the given mode; t is the partition used by a TOCAB level.
hipError_t run_level(gc_graph g, Frontier& f, bool bfs, int32_t* value, int32_t level, Mode mode, gc_tocab t,
                     hipStream_t s) {
  const int32_t n = g->n;
  const Tally tally = f.tally();
  if (mode != Mode::kPush) GC_HIP_TRY(f.need_bits(bfs ? value : nullptr, level));
  if (bfs) {
    if (mode == Mode::kPush) {
      ProfScope prof("bfs_push", s);
      GC_HIP_TRY(push_level(g, f, BfsRelax{value, level}, s));
    } else if (mode == Mode::kPull) {
      ProfScope prof("bfs_pull", s);
      if (wide_pull(n))
        k_bfs_pull<kPullThreads><<<pull_grid(n), kPullThreads, 0, s>>>(g->t_rowptr, g->t_colidx, n, f.front(), value,
                                                                       level, f.next(), g->visited, tally);
      else
        k_bfs_pull<kThreads><<<pull_grid(n), kThreads, 0, s>>>(g->t_rowptr, g->t_colidx, n, f.front(), value, level,
                                                               f.next(), g->visited, tally);
    } else if (t->col16) {
      // stream layout: the block's frontier bits (as 1 or 0) in LDS,
      // per-(row, block) maxima stored range-major (1: an in-neighbour of
      // the row is in the frontier), merged as one stream per range
      GC_HIP_TRY(stream_pull_setup());
      {
        ProfScope prof("bfs_tocab", s);
        if (t->n_chunks > 0)
          k_sssp_tocab_lds<kWNone><<<t->n_chunks, kLdsThreads, tocab_lds_bytes(t), s>>>(
              t->row_ptr, t->col16, t->heads, nullptr, 0u, t->chunk_beg, t->chunk_end, t->chunk_blk, t->chunk_j0,
              t->chunk_ns, t->seg, t->mR, t->log2W, n, f.front(), nullptr, t->pmin, pmin_bytes(t), g->stats);
      }
      ProfScope prof("bfs_merge", s);
      GC_HIP_TRY((launch_by_k<BfsMergeStream>(t->mk, t->mR, s, static_cast<const int32_t*>(t->rstart),
                                              static_cast<const uint16_t*>(t->id16s),
                                              static_cast<const int32_t*>(t->pmin), t->mR, n, value, f.next(),
                                              tally, level, g->visited)));
    } else {
      uint8_t* flag = reinterpret_cast<uint8_t*>(t->pmin);
      {
        ProfScope prof("bfs_tocab", s);
        k_bfs_tocab<<<row_grid(t->P), kThreads, 0, s>>>(t->row_ptr, t->col, t->id_map, t->P, g->visited,
                                                                   f.front(), flag, g->stats);
      }
      ProfScope prof("bfs_merge", s);
      GC_HIP_TRY((launch_by_k<BfsMerge>(t->mk, t->mR, s, static_cast<const int32_t*>(t->mrange), t->B,
                                        static_cast<const uint16_t*>(t->id16),
                                        static_cast<const uint8_t*>(flag), n, value, level, f.next(), g->visited,
                                        tally)));
    }
  } else {
    if (mode == Mode::kPush) {
      ProfScope prof("sssp_push", s);
      GC_HIP_TRY(push_level(g, f, SsspRelax{g->w, value, level, g->mark}, s));
    } else if (mode == Mode::kPull) {
      ProfScope prof("sssp_pull", s);
      if (wide_pull(n))
        k_sssp_pull<kPullThreads><<<pull_grid(n), kPullThreads, 0, s>>>(g->t_rowptr, g->t_colidx, g->t_w, n, f.front(),
                                                                        value, f.next(), tally);
      else
        k_sssp_pull<kThreads><<<pull_grid(n), kThreads, 0, s>>>(g->t_rowptr, g->t_colidx, g->t_w, n, f.front(), value,
                                                                f.next(), tally);
    } else {
      if (t->col16) {  // stream layout: the block's distances in LDS, partial minima range-major
        GC_HIP_TRY(stream_weights(t, s));
        {
          ProfScope prof("sssp_tocab", s);
          const size_t lds = tocab_lds_bytes(t);
          if (t->n_chunks > 0 && t->w8)
            k_sssp_tocab_lds<kW8><<<t->n_chunks, kLdsThreads, lds, s>>>(
                t->row_ptr, t->col16, t->heads, t->w8, 255u, t->chunk_beg, t->chunk_end, t->chunk_blk, t->chunk_j0,
                t->chunk_ns, t->seg, t->mR, t->log2W, n, f.front(), value, t->pmin, pmin_bytes(t), g->stats);
          else if (t->n_chunks > 0)
            k_sssp_tocab_lds<kW32><<<t->n_chunks, kLdsThreads, lds, s>>>(
                t->row_ptr, t->col16, t->heads, t->w_pad, static_cast<uint32_t>(kInf), t->chunk_beg, t->chunk_end, t->chunk_blk, t->chunk_j0,
                t->chunk_ns, t->seg, t->mR, t->log2W, n, f.front(), value, t->pmin, pmin_bytes(t), g->stats);
        }
        ProfScope prof("sssp_merge", s);
        GC_HIP_TRY((launch_by_k<SsspMergeStream>(t->mk, t->mR, s, static_cast<const int32_t*>(t->rstart),
                                                 static_cast<const uint16_t*>(t->id16s),
                                                 static_cast<const int32_t*>(t->pmin), t->mR, n, value, f.next(),
                                                 tally, level, g->visited)));
        return hipGetLastError();
      } else {
        ProfScope prof("sssp_tocab", s);
        k_sssp_tocab<<<row_grid(t->P), kThreads, 0, s>>>(t->row_ptr, t->col, t->w, t->P, f.front(), value,
                                                         t->pmin, g->stats);
      }
      ProfScope prof("sssp_merge", s);
      GC_HIP_TRY((launch_by_k<SsspMerge>(t->mk, t->mR, s, static_cast<const int32_t*>(t->mrange), t->B,
                                         static_cast<const uint16_t*>(t->id16),
                                         static_cast<const int32_t*>(t->pmin), n, value, f.next(), tally)));
    }
  }
  return hipGetLastError();
}

double now_ms() {
  return std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now().time_since_epoch()).count();
}

// Two HIP events released on scope exit.
struct EventPair {
  hipEvent_t e[2] = {nullptr, nullptr};
  hipError_t create() {
    GC_HIP_TRY(hipEventCreate(&e[0]));
    return hipEventCreate(&e[1]);
  }
  ~EventPair() {
    for (hipEvent_t x : e)
      if (x) (void)hipEventDestroy(x);
  }
};

// Action k of the learned scheduler: 0 push, 1 plain pull, 2 + i TOCAB pull
// over the i-th attached partition.
void action_mode(int32_t a, gc_tocab* parts, Mode* mode, gc_tocab* t) {
  *t = nullptr;
  if (a == 0) *mode = Mode::kPush;
  else if (a == 1) *mode = Mode::kPull;
  else {
    *mode = Mode::kTocab;
    *t = parts[a - 2];
  }
}

int32_t mode_action(Mode m) { return m == Mode::kPush ? 0 : (m == Mode::kPull ? 1 : 2); }

// One forward BC level (depth `level` -> level+1): depth, sigma and the next
// frontier, in the given mode.
hipError_t run_bc_level(gc_graph g, Frontier& f, int32_t level, Mode mode, gc_tocab t, hipStream_t s) {
  const int32_t n = g->n;
  const Tally tally = f.tally();
  if (mode != Mode::kPush) GC_HIP_TRY(f.need_bits(g->bc_depth, level));
  if (mode == Mode::kPush) {
    ProfScope prof("bc_push", s);
    GC_HIP_TRY(push_level(g, f, BcRelax{g->bc_depth, level, g->bc_sigma}, s));
  } else if (mode == Mode::kPull) {
    ProfScope prof("bc_pull", s);
    if (wide_pull(n))
      k_bc_pull<kPullThreads><<<pull_grid(n), kPullThreads, 0, s>>>(g->t_rowptr, g->t_colidx, n, f.front(), g->bc_depth,
                                                                    level, g->bc_sigma, f.next(), g->visited, tally);
    else
      k_bc_pull<kThreads><<<pull_grid(n), kThreads, 0, s>>>(g->t_rowptr, g->t_colidx, n, f.front(), g->bc_depth, level,
                                                            g->bc_sigma, f.next(), g->visited, tally);
  } else {
    {
      ProfScope prof("bc_tocab", s);
      k_bc_tocab<<<row_grid(t->P), kThreads, 0, s>>>(t->row_ptr, t->col, t->id_map, t->P, g->visited,
                                                                f.front(), g->bc_sigma, t->bc_part);
    }
    ProfScope prof("bc_merge", s);
    GC_HIP_TRY((launch_by_k<BcMerge>(t->mk, t->mR, s, static_cast<const int32_t*>(t->mrange), t->B,
                                     static_cast<const uint16_t*>(t->id16), static_cast<const double*>(t->bc_part),
                                     n, g->bc_depth, level, g->bc_sigma, f.next(), g->visited, tally)));
  }
  return hipGetLastError();
}

}  // namespace

namespace gcx {

void sched_features(int64_t n, int64_t m, int64_t n_f, int64_t m_f, int32_t level, double prior_ms,
                    int64_t prior_arcs, float* f) {
  level_features(n, m, n_f, m_f, level, prior_ms, prior_arcs, f);
}

hipError_t traverse(gc_graph g, gc_tocab t, int32_t source, int32_t* value, int32_t* count, uint32_t policy,
                    hipStream_t s, bool bfs, bool* overflow) {
  const int32_t n = g->n;
  Frontier f(g, s);
  GC_HIP_TRY(f.start(source, value, bfs ? nullptr : g->mark, nullptr, nullptr));
  int64_t m_u = g->m - f.m_f;
  int64_t m_u_in = g->m;  // in-arcs of the unvisited vertices (the source's own few left in)
  Heuristic h;
  int32_t level = 0;
  g->trace_action.clear();
  g->trace_ms.clear();
  if (overflow) *overflow = false;
  // Learned policy: the network's decision for every level after the first
  // is computed on the device from the level counters at the end of the
  // previous level and read back with them; the first level's from host
  // features. Its working-set fallback uses the attached partition nearest
  // the paper's 2^18 when the call gives none.
  const gc_sched net = sched_for(g, bfs ? 0 : 1);
  const bool learned = policy == GC_POLICY_LEARNED && net;
  const int32_t K = learned ? sched_actions(net) : 0;
  gc_tocab fall_t = t;
  int32_t fall_action = -1;  // action index of TOCAB over fall_t
  if (learned) {
    const int32_t np = static_cast<int32_t>(g->sched_parts.size());
    int32_t best = INT32_MAX;
    for (int32_t j = 0; j < np && 2 + j < K; ++j) {
      const int32_t d = std::abs(g->sched_parts[j]->log2W - 18);
      if (d < best) {
        best = d;
        fall_action = 2 + j;
      }
    }
    if (!t && fall_action >= 0) fall_t = g->sched_parts[fall_action - 2];
    if (t) fall_action = -1;  // the caller's partition is not among the network's actions
  }
  // the working-set rule's BFS arm over a stream-layout partition reads the
  // unvisited vertices' in-arcs
  f.count_in = bfs && (policy == GC_POLICY_HEURISTIC || policy == GC_POLICY_LEARNED) && fall_t != nullptr &&
               fall_t->col16 != nullptr && n <= Heuristic::kBfsTocabVertices &&
               static_cast<double>(g->m) <= Heuristic::kBfsTocabDegree * n;
  std::vector<float> outs(static_cast<size_t>(std::max(K, 1)));
  while (f.n_f > 0) {
    if (!bfs && level > n) return hipErrorInvalidValue;  // cannot happen with positive weights
    // SSSP revisits vertices, so the unexplored-arc count of BFS does not
    // apply; the whole arc set stands in for it.
    const int64_t unexplored = bfs ? m_u : g->m;
    // the working-set rule's choice: the policy itself, the fallback of the
    // learned one, and the reference its decision is gated against
    Mode hmode;
    if (policy == GC_POLICY_PUSH) hmode = Mode::kPush;
    else if (policy == GC_POLICY_PULL) hmode = t ? Mode::kTocab : Mode::kPull;
    else
      hmode = h.pick(n, f.n_f, f.m_f, unexplored, fall_t != nullptr, bfs, g->m, m_u_in,
                     fall_t != nullptr && fall_t->col16 != nullptr);
    Mode mode = hmode;
    gc_tocab lt = fall_t;
    int32_t action = -1;
    if (learned) {
      int32_t a = -1;
      if (level == 0) {
        if (hmode != Mode::kPush) {
          float feats[GC_SCHED_INPUTS];
          sched_features(n, g->m, f.n_f, f.m_f, level, 0.0, 0, feats);
          GC_HIP_TRY(sched_decide(net, feats, s, &a, outs.data()));
        }
      } else {
        a = g->stats_host[gcx::kStatChoice];
        std::memcpy(outs.data(), g->stats_host + gcx::kStatOut, sizeof(float) * K);
      }
      if (a >= 0 && a < K && hmode != Mode::kPush) {
        // The rule keeps the direction (its push / pull switch is the
        // direction-optimising test, close to the best on every graph
        // measured); on a pull level the network picks the form: plain pull
        // or TOCAB pull over one of the attached widths, the rule's own form
        // kept unless the network predicts its pick faster by more than the
        // gate.
        a = 1;
        for (int32_t k = 2; k < K; ++k)
          if (outs[k] < outs[a]) a = k;
        const int32_t ha = hmode == Mode::kPull ? 1 : fall_action;
        if (ha >= 1 && ha < K && outs[ha] <= outs[a] + kLearnedGate) a = ha;
        action_mode(a, g->sched_parts.data(), &mode, &lt);
        action = a;
      }
    }
    if (action < 0) {
      mode = hmode;
      lt = mode == Mode::kTocab ? fall_t : t;
      action = mode_action(mode);
    }
    const double t0 = now_ms();
    GC_HIP_TRY(run_level(g, f, bfs, value, level, mode, lt, s));
    LevelDecide dec;
    if (learned) {
      dec.pulling = h.pulling;
      dec.sub_next = bfs;
      dec.unexplored = bfs ? m_u : g->m;
      dec.alpha = Heuristic::kAlpha;
      dec.beta = Heuristic::kBeta;
    }
    GC_HIP_TRY(f.end_level(mode != Mode::kPush, overflow, learned ? net : nullptr, level + 1, dec));
    const double wall_ms = now_ms() - t0;
    g->trace_action.push_back(action);
    g->trace_ms.push_back(static_cast<float>(wall_ms));
    if (overflow && *overflow) break;
    if (bfs) {
      m_u -= f.m_f;
      m_u_in -= f.m_f_in;
    }
    ++level;
  }
  GC_HIP_TRY(f.finish());
  if (count) *count = level;
  return hipSuccess;
}

hipError_t bfs_run(gc_graph g, gc_tocab t, int32_t source, int32_t* depth, int32_t* levels, uint32_t policy,
                   hipStream_t s) {
  return traverse(g, t, source, depth, levels, policy, s, true, nullptr);
}

hipError_t sssp_run(gc_graph g, gc_tocab t, int32_t source, int32_t* dist, int32_t* rounds, uint32_t policy,
                    hipStream_t s, bool* overflow) {
  return traverse(g, t, source, dist, rounds, policy, s, false, overflow);
}

// Betweenness centrality from the given sources (Brandes): per source, the
// forward levels count shortest paths (push, pull or TOCAB pull per level,
// chosen as for BFS), then the backward steps accumulate the dependencies
// deepest level first into bc. The per-graph sigma / delta / depth arrays
// and the partition's FP64 partials are allocated by the first call.
hipError_t bc_run(gc_graph g, gc_tocab t, const int32_t* sources, int32_t n_src, double* bc, uint32_t policy,
                  hipStream_t s) {
  const int32_t n = g->n;
  if (!g->bc_sigma) {
    g->bc_sigma = static_cast<double*>(dev_alloc(sizeof(double) * n, s));
    g->bc_coef = static_cast<double*>(dev_alloc(sizeof(double) * 2 * static_cast<size_t>(n), s));
    g->bc_depth = static_cast<int32_t*>(dev_alloc(sizeof(int32_t) * n, s));
    g->bc_order = static_cast<int32_t*>(dev_alloc(sizeof(int32_t) * n, s));
    if (!g->bc_sigma || !g->bc_coef || !g->bc_depth || !g->bc_order) {
      for (void* p : {static_cast<void*>(g->bc_sigma), static_cast<void*>(g->bc_coef),
                      static_cast<void*>(g->bc_depth), static_cast<void*>(g->bc_order)})
        if (p) dev_free(p, s);
      g->bc_sigma = g->bc_coef = nullptr;
      g->bc_depth = g->bc_order = nullptr;
      return hipErrorOutOfMemory;
    }
  }
  if (t && !t->bc_part) {
    t->bc_part = static_cast<double*>(dev_alloc(sizeof(double) * std::max<int64_t>(t->P, 1), s));
    if (!t->bc_part) return hipErrorOutOfMemory;
  }
  Buf pre_in(sizeof(int32_t) * (static_cast<size_t>(n) + 1), s);
  if (!pre_in.p) return hipErrorOutOfMemory;
  g->trace_action.clear();
  g->trace_ms.clear();
  for (int32_t si = 0; si < n_src; ++si) {
    const int32_t src = sources[si];
    // order holds the vertices level by level (the source first); level d
    // occupies [lv_off[d], lv_off[d + 1]), and arc_pre each level's own arc
    // prefix: both are the forward levels' queues
    std::vector<int32_t> lv_off{0, 1};
    std::vector<int64_t> lv_arcs;     // out-arcs of each level's vertices
    std::vector<int64_t> lv_in{0};    // in-arcs (the source's are not needed)
    Frontier f(g, s);
    f.count_in = true;
    f.q[0] = g->bc_order;
    f.p[0] = g->arc_pre;
    GC_HIP_TRY(f.start(src, g->bc_depth, nullptr, g->bc_sigma, g->bc_coef));
    int64_t m_u = g->m - f.m_f;
    lv_arcs.push_back(f.m_f);
    Heuristic h;
    int32_t level = 0;
    while (f.n_f > 0) {
      Mode mode;
      if (policy == GC_POLICY_PUSH) mode = Mode::kPush;
      else if (policy == GC_POLICY_PULL) mode = t ? Mode::kTocab : Mode::kPull;
      else mode = h.pick(n, f.n_f, f.m_f, m_u, t != nullptr, true);
      const double t0 = now_ms();
      f.q[f.cur ^ 1] = g->bc_order + lv_off.back();
      f.p[f.cur ^ 1] = g->arc_pre + lv_off.back();
      GC_HIP_TRY(run_bc_level(g, f, level, mode, t, s));
      GC_HIP_TRY(f.end_level(mode != Mode::kPush, nullptr));
      g->trace_action.push_back(mode_action(mode));
      g->trace_ms.push_back(static_cast<float>(now_ms() - t0));
      if (f.n_f > 0) {
        GC_HIP_TRY(f.need_queue());  // the level order is its queues
        lv_off.push_back(lv_off.back() + f.n_f);
        lv_arcs.push_back(f.m_f);
        lv_in.push_back(f.m_f_in);
      }
      m_u -= f.m_f;
      ++level;
    }
    f.clearing = false;  // the steps below follow on the same stream, and the call ends in a wait for it
    GC_HIP_TRY(f.finish());
    // depths run 0 .. level-1 (level = lv_off.size() - 1). Each step d runs
    // in the cheaper direction: pull over the out-arcs of depth d
    // (arc_pre) or push over the in-arcs of depth d + 1 (pre_in = exclusive
    // scan of the in-degrees along order). The deepest level's step only sets
    // coef = 1 / sigma; the source (depth 0) takes no share.
    ProfScope prof("bc_back", s);
    const int32_t reached = lv_off.back();
    bool push_any = false;
    for (int32_t d = 1; d + 1 < level; ++d) push_any |= back_pushes(lv_in[d + 1], lv_arcs[d]);
    if (push_any) {
      k_order_degree<<<grid_for(reached, kThreads), kThreads, 0, s>>>(g->bc_order, reached, g->t_rowptr, g->arc_deg);
      GC_HIP_TRY(hipGetLastError());
      GC_HIP_TRY(scan_exclusive(g->arc_deg, pre_in.as<int32_t>(), reached, s));
    }
    for (int32_t d = level - 1; d >= 1; --d) {
      const int32_t lo = lv_off[d], hi = lv_off[d + 1];
      double* coef_out = g->bc_coef + static_cast<size_t>(d & 1) * n;
      const double* coef_in = g->bc_coef + static_cast<size_t>((d + 1) & 1) * n;
      const int64_t out_arcs = lv_arcs[d];
      const int64_t in_next = d + 1 < level ? lv_in[d + 1] : 0;
      if (d + 1 < level && back_pushes(in_next, out_arcs))
        GC_HIP_TRY(bc_back<true>(g->t_rowptr, g->t_colidx, g->bc_order + hi, pre_in.as<int32_t>() + hi,
                                 lv_off[d + 2] - hi, in_next, g->bc_depth, d, coef_in, coef_out, s));
      else if (d + 1 < level)
        GC_HIP_TRY(bc_back<false>(g->rowptr, g->colidx, g->bc_order + lo, g->arc_pre + lo, hi - lo, out_arcs,
                                  g->bc_depth, d, coef_in, coef_out, s));
      k_bc_finish<<<grid_for(hi - lo, kThreads), kThreads, 0, s>>>(g->bc_order + lo, hi - lo, g->bc_sigma, coef_out,
                                                                    bc);
    }
    GC_HIP_TRY(hipGetLastError());
  }
  return hipStreamSynchronize(s);
}

// Training data for the scheduler: at every level of a traversal from each
// source, the level is run once per action from the same state (snapshot
// and restore of the frontier state), each run timed with HIP events; the
// traversal then continues with the fastest action. One row per level:
// 6 features and K = 2 + n_parts times in ms.
hipError_t collect(gc_graph g, gc_tocab* parts, int32_t n_parts, bool bfs, const int32_t* sources, int32_t n_src,
                   float* features, float* times, int32_t max_rows, int32_t* rows, hipStream_t s) {
  const int32_t n = g->n;
  const int32_t K = 2 + n_parts;
  const size_t words = (static_cast<size_t>(n) + 31) / 32;
  Buf value(sizeof(int32_t) * n, s), sv(sizeof(int32_t) * n, s), sfront(sizeof(uint32_t) * words, s),
      snext(sizeof(uint32_t) * words, s),
      svis(sizeof(uint32_t) * words, s), smark(sizeof(int32_t) * n, s), squeue(sizeof(int32_t) * n, s);
  if (!value.p || !sv.p || !sfront.p || !snext.p || !svis.p || !smark.p || !squeue.p) return hipErrorOutOfMemory;
  hipEvent_t e0, e1;
  GC_HIP_TRY(hipEventCreate(&e0));
  GC_HIP_TRY(hipEventCreate(&e1));
  int32_t r = 0;
  hipError_t err = hipSuccess;
  for (int32_t si = 0; si < n_src && err == hipSuccess; ++si) {
    Frontier f(g, s);
    err = f.start(sources[si], value.as<int32_t>(), bfs ? nullptr : g->mark, nullptr, nullptr);
    int32_t level = 0;
    double prior_ms = 0.0;  // device time of the previous level (its fastest action), from the clock stamps
    int64_t prior_arcs = 0;
    bool overflow = false;
    std::vector<double> stamp_ms(static_cast<size_t>(K));
    while (err == hipSuccess && f.n_f > 0 && r < max_rows && !overflow) {
      err = f.need_queue();
      if (err != hipSuccess) break;
      sched_features(n, g->m, f.n_f, f.m_f, level, prior_ms, prior_arcs,
                     features + static_cast<size_t>(r) * GC_SCHED_INPUTS);
      // snapshot the state this level starts from
      const hipMemcpyKind dd = hipMemcpyDeviceToDevice;
      err = hipMemcpyAsync(sv.p, value.p, sizeof(int32_t) * n, dd, s);
      if (err == hipSuccess) err = hipMemcpyAsync(sfront.p, f.front(), sizeof(uint32_t) * words, dd, s);
      if (err == hipSuccess) err = hipMemcpyAsync(snext.p, f.next(), sizeof(uint32_t) * words, dd, s);
      if (err == hipSuccess) err = hipMemcpyAsync(svis.p, g->visited, sizeof(uint32_t) * words, dd, s);
      if (err == hipSuccess && !bfs) err = hipMemcpyAsync(smark.p, g->mark, sizeof(int32_t) * n, dd, s);
      if (err == hipSuccess) err = hipMemcpyAsync(squeue.p, f.queue(), sizeof(int32_t) * f.n_f, dd, s);
      const Frontier start = f;
      auto restore = [&]() -> hipError_t {
        f = start;
        GC_HIP_TRY(hipMemcpyAsync(value.p, sv.p, sizeof(int32_t) * n, dd, s));
        GC_HIP_TRY(hipMemcpyAsync(f.front(), sfront.p, sizeof(uint32_t) * words, dd, s));
        GC_HIP_TRY(hipMemcpyAsync(f.next(), snext.p, sizeof(uint32_t) * words, dd, s));
        GC_HIP_TRY(hipMemcpyAsync(g->visited, svis.p, sizeof(uint32_t) * words, dd, s));
        if (!bfs) GC_HIP_TRY(hipMemcpyAsync(g->mark, smark.p, sizeof(int32_t) * n, dd, s));
        return hipMemcpyAsync(f.queue(), squeue.p, sizeof(int32_t) * f.n_f, dd, s);
      };
      float* row_t = times + static_cast<size_t>(r) * K;
      int32_t best = 0;
      for (int32_t a = 0; a < K && err == hipSuccess; ++a) {
        Mode mode;
        gc_tocab lt;
        action_mode(a, parts, &mode, &lt);
        if (a > 0) err = restore();
        if (err == hipSuccess) err = hipEventRecord(e0, s);
        if (err == hipSuccess) err = run_level(g, f, bfs, value.as<int32_t>(), level, mode, lt, s);
        if (err == hipSuccess) err = hipEventRecord(e1, s);
        if (err == hipSuccess) err = f.end_level(mode != Mode::kPush, &overflow);
        float ms = 0.0f;
        if (err == hipSuccess) err = hipEventSynchronize(e1);
        if (err == hipSuccess) err = hipEventElapsedTime(&ms, e0, e1);
        row_t[a] = ms;
        stamp_ms[a] = f.level_ms();
        if (ms < row_t[best]) best = a;
      }
      if (err != hipSuccess) break;
      // continue the traversal with the fastest action
      if (best != K - 1) {
        Mode mode;
        gc_tocab lt;
        action_mode(best, parts, &mode, &lt);
        err = restore();
        if (err == hipSuccess) err = run_level(g, f, bfs, value.as<int32_t>(), level, mode, lt, s);
        if (err == hipSuccess) err = f.end_level(mode != Mode::kPush, &overflow);
      }
      prior_ms = stamp_ms[best];
      prior_arcs = start.m_f;
      ++r;
      ++level;
    }
    if (err == hipSuccess && !overflow) err = f.finish();
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  *rows = r;
  if (err == hipSuccess) err = hipStreamSynchronize(s);
  return err;
}

}  // namespace gcx
