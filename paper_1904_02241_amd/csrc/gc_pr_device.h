// Device code shared by the PageRank kernels and the batched persistent
// kernel: the fused per-vertex update, pull tiles and the merge of the
// partial sums of one vertex range.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "gc_device.h"
#include "gc_internal.h"
#include "gc_merge.h"

namespace {


using gcd::kWave;
using gcd::wave_lds_fence;

constexpr int kThreads = 256;

constexpr int kTileArcs = 2048;                  // arcs per pull tile (tile table granularity)
constexpr int kStageCap = 4096;                  // arcs a tile may stage in LDS
constexpr int kPerThread = kStageCap / kThreads;  // staged arcs per thread
constexpr int kFlatB = gcm::kFlatB;              // merges over at most this many blocks flatten their slices

static_assert(kTileArcs <= kStageCap, "a tile's short rows must fit the stage");

// Convergence mode queues an iteration before it knows the change of the one
// before; the kernels of an iteration past the last do nothing. The word
// (null: never) holds the number of the last call that has ended, and calls
// are numbered upwards, so the kernels that a call leaves behind stay stopped
// when the next one runs, on whichever stream. (32 bits, and the number in
// what was padding of the kernels' arguments: beyond 128 bytes of them, or
// with a 64-bit comparison, each kernel of an iteration took 0.1 to 0.2 us
// more, 6 of 353 us for 300,007 vertices.)
__device__ __forceinline__ bool stopped(const int32_t* word, int32_t call) {
  return word && static_cast<int32_t>(static_cast<uint32_t>(*word) - static_cast<uint32_t>(call)) >= 0;
}

struct Update {
  double base;      // (1 - d) / n
  double d;         // damping
  double inv_n;     // 1 / n, applied to D in uniform mode (0 in leak mode)
  const double* din;  // D of this iteration: the sum of din[0 .. dcount)
  int32_t dcount;
  int32_t call = 0;  // convergence mode: the call's number, for `stop`
  double* dpart;    // one dangling partial per work-group of the update kernel
  const int32_t* rowptr;  // out-arc CSR: outdeg(v) = rowptr[v+1] - rowptr[v]
  float* contrib;         // written for the next iteration
  float* rank_out;        // written on the last iteration only (else null)
  const float* rank_prev = nullptr;  // convergence mode: the previous iterate
  double* lpart = nullptr;           // convergence mode: L1 change per work-group
  const int32_t* stop = nullptr;     // convergence mode
  int32_t n;
};

// r'[v] from the neighbour sum; writes c'[v] (and r'[v] on the last pass),
// returns r'[v] when v has no out-arcs (its share of the next D), else 0.
// In convergence mode also adds |r'[v] - r[v]| (FP64 over the FP32
// iterates) to dl.
// The new contribution is also returned in cv (u.contrib may be null when
// the caller keeps it elsewhere). update_vertex_loaded takes v's out-degree
// and previous rank (read only in convergence mode) from the caller.
__device__ __forceinline__ double update_vertex_loaded(const Update& u, int32_t v, double sum, double D, double& dl,
                                                       float& cv, int32_t deg, float prev) {
  const double r = u.base + u.d * (sum + D * u.inv_n);
  const float r32 = static_cast<float>(r);
  cv = deg ? static_cast<float>(static_cast<double>(r32) / deg) : 0.0f;
  if (u.contrib) u.contrib[v] = cv;
  if (u.rank_out) u.rank_out[v] = r32;
  if (u.rank_prev) dl += fabs(static_cast<double>(r32) - static_cast<double>(prev));
  return deg ? 0.0 : static_cast<double>(r32);
}

__device__ __forceinline__ double update_vertex(const Update& u, int32_t v, double sum, double D, double& dl,
                                                float& cv) {
  return update_vertex_loaded(u, v, sum, D, dl, cv, u.rowptr[v + 1] - u.rowptr[v], u.rank_prev ? u.rank_prev[v] : 0.0f);
}

__device__ __forceinline__ double update_vertex(const Update& u, int32_t v, double sum, double D, double& dl) {
  float cv;
  return update_vertex(u, v, sum, D, dl, cv);
}

__device__ __forceinline__ double update_vertex(const Update& u, int32_t v, double sum, double D) {
  double dl = 0.0;
  return update_vertex(u, v, sum, D, dl);
}

// Work-group sum of one double per thread (fixed reduction tree), returned
// to every thread.
template <int NT = kThreads>
__device__ __forceinline__ double wg_sum(double x) {
  __shared__ double part[NT / kWave];
  x = gcd::wave_sum(x);
  if ((threadIdx.x & (kWave - 1)) == 0) part[threadIdx.x / kWave] = x;
  __syncthreads();
  double t = 0.0;
#pragma unroll
  for (int w = 0; w < NT / kWave; ++w) t += part[w];
  __syncthreads();
  return t;
}

// This thread's share of D (its loads are issued before the caller's own),
// and D itself, to every thread: up to kDangFused partials of the previous
// update are added by each work-group in one fixed order, which costs a
// few loads in the shadow of the tile's, where a reduction kernel between
// two iterations costs its launch and two memory round trips (4.3 us each
// on a 1000-vertex graph, more than the rest of its iteration needs).
// Larger counts come reduced (dcount = 1): at 1024 partials and as many
// work-groups the repeated reads are 8 MB of L2 traffic, and they grow with
// the square.
constexpr int32_t kDangFused = gcx::kDangSlots;

template <int NT = kThreads>
__device__ __forceinline__ double dangling_share(const Update& u) {
  double x = 0.0;
  for (int32_t i = threadIdx.x; i < u.dcount; i += NT) x += u.din[i];
  return x;
}

template <int NT = kThreads>
__device__ __forceinline__ double dangling_total(const Update& u, double share) {
  return u.dcount == 1 ? *u.din : wg_sum<NT>(share);  // uniform
}

template <int NT = kThreads>
__device__ __forceinline__ void publish_dangling(const Update& u, double mine) {
  const double t = wg_sum<NT>(mine);
  if (threadIdx.x == 0) u.dpart[blockIdx.x] = t;
}

// publish_dangling plus, in convergence mode, the work-group's L1 change.
template <int NT = kThreads>
__device__ __forceinline__ void publish_update(const Update& u, double mine, double dl) {
  publish_dangling<NT>(u, mine);
  if (u.lpart) {  // uniform
    const double t = wg_sum<NT>(dl);
    if (threadIdx.x == 0) u.lpart[blockIdx.x] = t;
  }
}

// The value an arc contributes to its row's sum, given its index i in the
// arc array and the gathered source value x: x itself (PageRank, where the
// source value is already c[u] = r[u] / outdeg(u)), or x times the arc's
// value (SpMV: FP32 values stored as their bits, or integer weights).
// load(i) fetches the arc's value, so that it is in flight with the columns
// and gathers; apply multiplies it in.
struct PlainArc {
  struct Value {};
  __device__ __forceinline__ Value load(int32_t) const { return {}; }
  __device__ __forceinline__ float apply(Value, float x) const { return x; }
};
struct ValuedArc {
  const int32_t* val;  // null: every value is 1
  bool f32;            // val holds FP32 bit patterns (else integers)
  using Value = int32_t;
  __device__ __forceinline__ Value load(int32_t i) const { return val ? gcd::ld_stream(val + i) : 0; }
  __device__ __forceinline__ float apply(Value b, float x) const {
    if (!val) return x;
    return x * (f32 ? __int_as_float(b) : static_cast<float>(b));
  }
};

// Arcs kFirst * kThreads + [0, kCount * kThreads) of a tile of len arcs
// starting at a0: the columns (coalesced across the work-group, streamed
// past the cache), then the gathers, times the arcs' values into `vals` (LDS);
// between() runs while the gathers are in flight. Indices past
// the end are clamped to the last arc instead of branched around, which
// keeps the loads free of control flow (a branch per load would make each
// one wait for the previous).
template <int kFirst, int kCount, class Arc, class Between>
__device__ __forceinline__ void stage_part(const int32_t* __restrict__ col, const float* __restrict__ c, int32_t a0,
                                           int32_t len, float* vals, Arc arc, Between&& between) {
  int32_t idx[kCount];
  typename Arc::Value val[kCount];
#pragma unroll
  for (int k = 0; k < kCount; ++k) {
    const int32_t i = min(static_cast<int32_t>(threadIdx.x) + (kFirst + k) * kThreads, len - 1);
    idx[k] = gcd::ld_stream(col + a0 + i);
    val[k] = arc.load(a0 + i);
  }
  float x[kCount];
#pragma unroll
  for (int k = 0; k < kCount; ++k) x[k] = c[idx[k]];
  between();
#pragma unroll
  for (int k = 0; k < kCount; ++k) {
    const int32_t i = threadIdx.x + (kFirst + k) * kThreads;
    if (i < len) vals[i] = arc.apply(val[k], x[k]);
  }
}

// Gathers c[col[i]] times the arc's value for i = a0 + [0, len) (len <= kStageCap) into
// LDS. Most tiles hold about kTileArcs arcs, a last row's few arcs more or
// less, so the first kTileArcs are always loaded and the rest only where a
// tile has them, two loads per thread or all of them (uniform branches,
// taken while the first gathers are in flight): loading every tile as if it
// held kStageCap arcs issued twice the memory instructions, and the gathers
// are what bounds the tile (L2 address rate).
template <class Arc = PlainArc>
__device__ __forceinline__ void stage_gather(const int32_t* __restrict__ col, const float* __restrict__ c,
                                             int32_t a0, int32_t len, float* vals, Arc arc = Arc()) {
  if (len <= 0) return;
  constexpr int kBase = kTileArcs / kThreads, kFew = 2;
  auto nothing = [] {};
  stage_part<0, kBase>(col, c, a0, len, vals, arc, [&] {
    if (len > (kBase + kFew) * kThreads) stage_part<kBase, kPerThread - kBase>(col, c, a0, len, vals, arc, nothing);
    else if (len > kBase * kThreads) stage_part<kBase, kFew>(col, c, a0, len, vals, arc, nothing);
  });
}

// Sum of the arcs' values times c[col[i]] over arcs [b, e) (b < e) by the whole
// work-group (hub rows).
template <class Arc = PlainArc>
__device__ double wg_row_sum(const int32_t* __restrict__ col, const float* __restrict__ c, int32_t b, int32_t e,
                             Arc arc = Arc()) {
  double s = 0.0;
  for (int32_t base = b; base < e; base += kStageCap) {
    int32_t idx[kPerThread];
    typename Arc::Value val[kPerThread];
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) {
      const int32_t i = min(base + static_cast<int32_t>(threadIdx.x) + k * kThreads, e - 1);
      idx[k] = gcd::ld_stream(col + i);
      val[k] = arc.load(i);
    }
    float x[kPerThread];
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) x[k] = c[idx[k]];
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) {
      const int32_t i = base + static_cast<int32_t>(threadIdx.x) + k * kThreads;
      if (i < e) s += static_cast<double>(arc.apply(val[k], x[k]));
    }
  }
  return wg_sum(s);
}

// One pull tile (coarse-grained load balancing of the pull direction,
// Section 3.2): the tile owns the rows whose first arc lies in its
// kTileArcs-wide slice of the arc array. Their arcs are gathered into LDS
// together; then each thread sums whole short rows serially in FP64, rows of
// more than kThreadRow arcs are summed by a wave (a thread walking a hub's row
// of up to 4096 arcs kept the tile waiting), and a last row too long for the
// stage is summed by the whole work-group. No atomics. emit(row, sum) is
// called once per owned row. Measured before and after (with stage_gather's
// skipped loads): plain pull of a 1000-vertex R-MAT graph 17.8 -> 11.4 us,
// pull over 2^18-wide blocks of a uniform graph of 2.5 M vertices and 38 M
// arcs 203 -> 184 us (206 G gathers/s of the 274 an L2-resident slice gives).
// Where a tile's rows are about as long as that line, some threads walk theirs
// and the wave then takes the others: so a tile of more than kMeanRow arcs per
// row leaves its rows of more than kMeanWaveRow to the waves, all four of them.
// PageRank by plain pull, 20 iterations, 100,000 vertices of 112, 136, 200
// arcs: threads alone 1214, 1428, 2090 us; the one line for every tile and the
// first wave 1216, 1624, 1914; so 1124, 1309, 1836 (of 64: 758, 744, 747).
constexpr int kThreadRow = 128, kMeanRow = 80, kMeanWaveRow = 32;
template <class Emit, class Arc = PlainArc>
__device__ __forceinline__ void pull_tile(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
                                          const float* __restrict__ c, int32_t r0, int32_t r1, float* vals,
                                          Emit&& emit, Arc arc = Arc()) {
  const int32_t a0 = row_ptr[r0];
  const int32_t last_b = row_ptr[r1 - 1];
  const int32_t a_end = row_ptr[r1];
  const bool long_last = (a_end - a0) > kStageCap;
  const int lane = threadIdx.x & (kWave - 1);
  // up to 64 rows go to the waves in turn, so that rows summed by a wave
  // spread over all of them; more go to the threads in order (coalesced)
  const bool few = r1 - r0 <= kWave;  // uniform
  const int32_t slot =
      few ? lane * (kThreads / kWave) + static_cast<int32_t>(threadIdx.x) / kWave : static_cast<int32_t>(threadIdx.x);
  // the bounds of the thread's first row, in flight with the tile's loads
  const int32_t r_short_end = long_last ? r1 - 1 : r1;
  int32_t rb = 0, re = 0;
  if (r0 + slot < r_short_end) {
    rb = row_ptr[r0 + slot];
    re = row_ptr[r0 + slot + 1];
  }
  const int32_t arcs = (long_last ? last_b : a_end) - a0;
  const int32_t by_wave = arcs > kMeanRow * (r_short_end - r0) ? kMeanWaveRow : kThreadRow;
  stage_gather(col, c, a0, arcs, vals, arc);
  __syncthreads();
  for (int32_t base = r0; base < r_short_end; base += kThreads) {  // uniform
    const int32_t r = base + slot;
    const bool mine = r < r_short_end;
    if (base != r0 && mine) {
      rb = row_ptr[r];
      re = row_ptr[r + 1];
    }
    const int32_t b = mine ? rb - a0 : 0, e = mine ? re - a0 : 0;
    const bool whole_wave = e - b > by_wave;
    double s = 0.0;
    if (mine && !whole_wave)
      for (int32_t i = b; i < e; ++i) s += static_cast<double>(vals[i]);
    uint64_t pending = __ballot(whole_wave);
    while (pending) {
      const int owner = __ffsll(static_cast<long long>(pending)) - 1;
      pending &= pending - 1;
      const int32_t wb = __builtin_amdgcn_readlane(b, owner), we = __builtin_amdgcn_readlane(e, owner);
      double t = 0.0;
      for (int32_t i = wb + lane; i < we; i += kWave) t += static_cast<double>(vals[i]);
      t = gcd::wave_sum(t);
      if (lane == owner) s = t;
    }
    if (mine) emit(r, s);
  }
  if (long_last) {
    const double s = wg_row_sum(col, c, last_b, a_end, arc);
    if (threadIdx.x == 0) emit(r1 - 1, s);
  }
}

// Figure 5 merge, accumulation part, for vertex range j (FP64 LDS sums).
template <int K, bool kFlat, class T>
__device__ __forceinline__ void merge_accumulate(const int32_t* __restrict__ range_ptr, int32_t B,
                                                 const uint16_t* __restrict__ id16, const T* __restrict__ partial,
                                                 int32_t j, double* acc) {
  gcm::merge_accumulate<K, kFlat, kThreads>(range_ptr, B, id16, partial, j, acc);
}

}  // namespace
