// PageRank of small graphs: every iteration in one launch of one work-group,
// the whole graph in its LDS.
//
// A graph whose transposed columns (16 bits each), offsets, out-degrees and
// two contribution vectors fit the LDS of a compute unit is bound by launches
// and memory round trips, not by bytes: the tile kernels take about 16 us per
// iteration of a 1000-vertex graph, four dependent loads deep, whatever its
// arcs. Here the loads happen once, an iteration touches LDS alone and ends
// in one barrier. What bounds it then is the instruction rate of the one CU
// (a wave instruction every four cycles on each of four SIMDs), so rows are
// sorted by length once and taken by the least lanes that hold them with
// eight arcs each (1, 2, 4, 8, 16, or the whole wave in several steps): 64 to
// 1 rows per wave step, with the vertex update (an FP64 division) on lanes
// that mostly have one to do. Row
// sums are FP64, ranks and contributions FP32, as in the other forms, and
// every form of the iteration (pull, push, blocked) has the same result, so
// all of them may come here. Measured (20 iterations of the plain pull, us
// per call, tile kernels -> this one): R-MAT of 1000 vertices and 7,400 arcs
// 247 -> 54, of 2500 / 18,000 275 -> 109, of 2000 / 27,000 240 -> 124; uniform
// graphs of 1000 / 8,000 107 -> 46, 3000 / 24,000 124 -> 112, 5000 / 20,000
// 132 -> 142 (these stay with the tile kernels). pr_small_pays says which
// calls take this form; a graph must fit the LDS: 18 n + 2 m + 1028 bytes
// (22 n in convergence mode) of 158 KB, 3,200 vertices at 16 arcs each.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>

#include "gc_device.h"
#include "gc_internal.h"

namespace {

using gcd::kWave;

constexpr int kSmallThreads = 1024;
constexpr int kSmallWaves = kSmallThreads / kWave;

struct SmallArgs {
  int32_t n, m;
  const int32_t* t_rowptr;
  const int32_t* t_col;
  const int32_t* rowptr;
  const float* rank_in;
  float* rank_out;
  double base, d, inv_n;
  int32_t iters;
  double tol;      // convergence mode: stop at the first L1 change <= tol
  double* result;  // convergence mode: the last change, the iterations run
};

// The value a DPP control moves into each lane, both halves.
template <int kCtrl>
__device__ __forceinline__ double dpp_f64(double x) {
  const uint64_t b = static_cast<uint64_t>(__double_as_longlong(x));
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(b), kCtrl, 0xF, 0xF, false);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(b >> 32), kCtrl, 0xF, 0xF, false);
  return __longlong_as_double(static_cast<long long>(lo | (static_cast<uint64_t>(hi) << 32)));
}

// Sum over aligned groups of VW lanes (1 .. 16), to every lane of the group:
// exchanges with the lane at distance 1, 2 (quad_perm), then the mirrored
// lane of the half row and of the row.
template <int VW>
__device__ __forceinline__ double group_sum(double x) {
  if (VW > 1) x += dpp_f64<0xB1>(x);
  if (VW > 2) x += dpp_f64<0x4E>(x);
  if (VW > 4) x += dpp_f64<0x141>(x);
  if (VW > 8) x += dpp_f64<0x140>(x);
  return x;
}

// Sum over the wave, to every lane (the four rows of 16 through scalars).
__device__ __forceinline__ double wave_total(double x) {
  x = group_sum<16>(x);
  const uint64_t b = static_cast<uint64_t>(__double_as_longlong(x));
  double t = 0.0;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(b), 16 * r);
    const uint32_t hi = __builtin_amdgcn_readlane(static_cast<int>(b >> 32), 16 * r);
    t += __longlong_as_double(static_cast<long long>(lo | (static_cast<uint64_t>(hi) << 32)));
  }
  return t;
}

constexpr int kArcs = 8;     // arcs per lane and step
constexpr int kClasses = 6;  // rows by length: lanes 1, 2, 4, 8, 16, 64
constexpr int kColPad = kArcs * kWave;  // columns read past the last arc (and left out)

__device__ __forceinline__ int row_class(int32_t len) {
  return (len > kArcs) + (len > 2 * kArcs) + (len > 4 * kArcs) + (len > 8 * kArcs) + (len > 16 * kArcs);
}

// Sum of cur[cols[i]] over i = b, b + VW, ... < e (FP64), kArcs columns, then
// their contributions, in flight together. Columns past e are read (the next
// rows', or the padding) and left out.
template <int VW>
__device__ __forceinline__ double row_step(const uint16_t* cols, const float* cur, int32_t b, int32_t e) {
  uint32_t u[kArcs];
  float x[kArcs];
  double s = 0.0;
#pragma unroll
  for (int k = 0; k < kArcs; ++k) u[k] = cols[b + k * VW];
#pragma unroll
  for (int k = 0; k < kArcs; ++k) x[k] = cur[u[k]];
#pragma unroll
  for (int k = 0; k < kArcs; ++k) s += static_cast<double>(b + k * VW < e ? x[k] : 0.0f);
  return s;
}

template <bool kConv>
__global__ __launch_bounds__(kSmallThreads) void k_pr_small(SmallArgs a) {
  extern __shared__ float lds[];
  __shared__ double part[2][kSmallWaves], lpart[2][kSmallWaves];
  __shared__ int32_t class_at[kClasses + 1], op_at[kClasses + 1];
  const int32_t n = a.n, m = a.m;
  float* c = lds;                                        // [2][n]
  int32_t* off = reinterpret_cast<int32_t*>(c + 2 * n);  // [n + 1]
  int32_t* deg = off + n + 1;                            // [n]
  float* prev = reinterpret_cast<float*>(deg + n);       // [n], convergence mode
  uint16_t* order = reinterpret_cast<uint16_t*>(prev + (kConv ? n : 0));  // [n]: rows by class
  uint16_t* cols = order + n;                                            // [m + kColPad]
  const int lane = threadIdx.x & (kWave - 1);
  const int wid = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
#pragma unroll 8
  for (int32_t i = threadIdx.x; i < m; i += kSmallThreads) cols[i] = static_cast<uint16_t>(a.t_col[i]);
  for (int32_t i = threadIdx.x; i < kColPad; i += kSmallThreads) cols[m + i] = 0;
  double mine = 0.0;
  for (int32_t v = threadIdx.x; v < n; v += kSmallThreads) {
    off[v] = a.t_rowptr[v];
    const int32_t dg = a.rowptr[v + 1] - a.rowptr[v];
    const float r = a.rank_in[v];
    deg[v] = dg;
    c[v] = dg ? static_cast<float>(static_cast<double>(r) / dg) : 0.0f;
    if (kConv) prev[v] = r;
    if (!dg) mine += static_cast<double>(r);
  }
  if (threadIdx.x == 0) off[n] = m;
  mine = wave_total(mine);
  if (lane == 0) part[0][wid] = mine;
  // rows by class, ascending inside a class (so every sum has one order):
  // wave w lists class w
  __syncthreads();
  if (wid < kClasses) {
    int32_t cnt = 0;
    for (int32_t v0 = 0; v0 < n; v0 += kWave) {
      const int32_t v = v0 + lane;
      cnt += __popcll(__ballot(v < n && row_class(off[min(v, n - 1) + 1] - off[min(v, n - 1)]) == wid));
    }
    if (lane == 0) class_at[wid + 1] = cnt;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    class_at[0] = op_at[0] = 0;
    for (int k = 0; k < kClasses; ++k) {
      const int32_t rows = class_at[k + 1], per = k < kClasses - 1 ? kWave >> k : 1;
      class_at[k + 1] = class_at[k] + rows;
      op_at[k + 1] = op_at[k] + (rows + per - 1) / per;
    }
  }
  __syncthreads();
  if (wid < kClasses) {
    int32_t at = class_at[wid];
    for (int32_t v0 = 0; v0 < n; v0 += kWave) {
      const int32_t v = v0 + lane;
      const bool in = v < n && row_class(off[min(v, n - 1) + 1] - off[min(v, n - 1)]) == wid;
      const uint64_t mask = __ballot(in);
      if (in) order[at + __popcll(mask & gcd::lanemask_lt())] = static_cast<uint16_t>(v);
      at += __popcll(mask);
    }
  }
  __syncthreads();
  // the class bounds in scalar registers
  int32_t row0[kClasses + 1], op0[kClasses + 1];
#pragma unroll
  for (int k = 0; k <= kClasses; ++k) {
    row0[k] = __builtin_amdgcn_readfirstlane(class_at[k]);
    op0[k] = __builtin_amdgcn_readfirstlane(op_at[k]);
  }
  const int32_t ops = op0[kClasses];
  int32_t it = 0;
  double change = 0.0;
  for (; it < a.iters; ++it) {
    const float* cur = c + (it & 1) * n;
    float* nxt = c + ((it & 1) ^ 1) * n;
    const bool last = it == a.iters - 1;
    double D = 0.0;
#pragma unroll
    for (int w = 0; w < kSmallWaves; ++w) D += part[it & 1][w];
    mine = 0.0;
    double dl = 0.0;
    // wave steps, the longest rows first
    for (int32_t q = wid; q < ops; q += kSmallWaves) {  // uniform
      const int32_t op = ops - 1 - q;
      int k = 0;
      int32_t first = row0[0], end = row0[1], o = op;
#pragma unroll
      for (int j = 1; j < kClasses; ++j) {
        if (op >= op0[j]) {
          k = j;
          first = row0[j];
          end = row0[j + 1];
          o = op - op0[j];
        }
      }
      const int32_t rows = end - first;
      int32_t v = 0;
      bool lead = false;  // the lane that updates row v
      double s = 0.0;
      auto take = [&](auto vw) {
        constexpr int VW = decltype(vw)::value;
        const int32_t i = o * (kWave / VW) + lane / VW;
        v = order[first + min(i, rows - 1)];
        lead = i < rows && (lane & (VW - 1)) == 0;
        s = group_sum<VW>(row_step<VW>(cols, cur, off[v] + (lane & (VW - 1)), off[v + 1]));
      };
      switch (k) {  // uniform
        case 0: take(std::integral_constant<int, 1>()); break;
        case 1: take(std::integral_constant<int, 2>()); break;
        case 2: take(std::integral_constant<int, 4>()); break;
        case 3: take(std::integral_constant<int, 8>()); break;
        case 4: take(std::integral_constant<int, 16>()); break;
        default: {
          v = order[first + o];
          lead = lane == 0;
          const int32_t e = off[v + 1];
          for (int32_t b = off[v] + lane; b - lane < e; b += kArcs * kWave) s += row_step<kWave>(cols, cur, b, e);
          s = wave_total(s);
        }
      }
      if (lead) {
        const float r32 = static_cast<float>(a.base + a.d * (s + D * a.inv_n));
        const int32_t dg = deg[v];
        nxt[v] = dg ? static_cast<float>(static_cast<double>(r32) / dg) : 0.0f;
        if (!dg) mine += static_cast<double>(r32);
        if (kConv) {
          dl += fabs(static_cast<double>(r32) - static_cast<double>(prev[v]));
          prev[v] = r32;
        } else if (last) {
          a.rank_out[v] = r32;
        }
      }
    }
    const int slot = (it & 1) ^ 1;  // read by the next iteration, written again after its barrier
    mine = wave_total(mine);
    if (kConv) dl = wave_total(dl);
    if (lane == 0) {
      part[slot][wid] = mine;
      if (kConv) lpart[slot][wid] = dl;
    }
    __syncthreads();
    if (kConv) {
      change = 0.0;
#pragma unroll
      for (int w = 0; w < kSmallWaves; ++w) change += lpart[slot][w];
      if (change <= a.tol) {  // uniform
        ++it;
        break;
      }
    }
  }
  if (kConv) {
    for (int32_t v = threadIdx.x; v < n; v += kSmallThreads) a.rank_out[v] = prev[v];
    if (threadIdx.x == 0) {
      a.result[0] = change;
      a.result[1] = static_cast<double>(it);
    }
  }
}

size_t small_lds(int64_t n, int64_t m, bool conv) {
  return sizeof(float) * static_cast<size_t>(4 * n + 1 + (conv ? n : 0)) +
         sizeof(uint16_t) * static_cast<size_t>(n + m + kColPad);
}

constexpr size_t kSmallLds = 158 * 1024;  // of a compute unit's 160 KB, beside the static arrays

template <bool kConv>
hipError_t launch(const SmallArgs& a, size_t lds, hipStream_t s) {
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_pr_small<kConv>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize,
                                                     static_cast<int>(kSmallLds));
  GC_HIP_TRY(attr);
  k_pr_small<kConv><<<1, kSmallThreads, lds, s>>>(a);
  return hipGetLastError();
}

}  // namespace

namespace gcx {

bool pr_small_fits(int64_t n, int64_t m, bool conv) { return n <= 65536 && small_lds(n, m, conv) <= kSmallLds; }

// Microseconds of both sides, fitted to graphs of 64 to 8,500 vertices and
// 0.1 to 160 arcs each, uniform and R-MAT, in every form (a call's time is
// within a quarter of these but for the plain push of hub graphs). This form
// loads and sorts once per call (5 us per 1000 vertices), then pays per
// vertex and arc with one CU's instructions; a row of more than 128 arcs
// takes a whole wave's steps of 512, so beyond 112 arcs per row on average
// rows count as such. The tile kernels cost their launches (one to start and
// one to three per iteration) and little per arc, but for a tile's rows, one
// thread each (where arcs are few, a tile has many), a row of more than 128
// arcs, and the push's atomics. Calls at both sides of the line (this form,
// tiles): plain pull, 20 iterations of 2000 / 32,000 122, 119; of 3000 /
// 48,000 180, 121; of 8,500 / 850 207, 386; one iteration of 1000 / 8,000 10,
// 10, of 3000 / 24,000 23, 11; push of 8,500 / 850 207, 125; pull over blocks,
// 400 / 64,000 549, 351, 3000 / 48,000 180, 245.
bool pr_small_pays(gc_graph g, PrForm form, bool conv, int32_t iters) {
  if (!pr_small_fits(g->n, g->m, conv)) return false;
  const double n = g->n * 1e-3, m = static_cast<double>(g->m) * 1e-3, deg = m / n;
  const double it = conv ? std::min(iters, 20) : iters;  // (a run until convergence takes some 10 to 20)
  const double arcs = deg > 112.0 ? n * 512.0 * std::ceil(deg / 512.0) : m;
  const double small = 5.0 * n + it * (0.5 + (conv ? 1.2 : 0.9) * n + 0.11 * arcs);
  double step = 0.0;
  switch (form) {
    case PrForm::kPull:
      step = g->longest_in > 128 ? 10.0
                                 : std::max(6.7, 3.5 + 1.8 * n / static_cast<double>(g->m / pull_tile_arcs() + 1));
      break;
    case PrForm::kPush: step = 5.6 + 0.75 * deg; break;
    case PrForm::kTocabPull: step = 10.0; break;
    case PrForm::kTocabPush: step = 16.0 + 0.5 * m; break;
    default: step = 8.0 + 0.16 * m; break;  // kTocabPushInner
  }
  return small <= 5.0 + it * (step + (conv ? 4.5 : 0.0));
}

hipError_t pr_small_run(gc_graph g, float damping, int32_t dangling, const float* rank_in, float* rank_out,
                        int32_t iters, hipStream_t s, Converge* cv) {
  SmallArgs a;
  a.n = g->n;
  a.m = static_cast<int32_t>(g->m);
  a.t_rowptr = g->t_rowptr;
  a.t_col = g->t_colidx;
  a.rowptr = g->rowptr;
  a.rank_in = rank_in;
  a.rank_out = rank_out;
  a.d = damping;
  a.base = (1.0 - static_cast<double>(damping)) / g->n;
  a.inv_n = dangling == GC_DANGLING_UNIFORM ? 1.0 / g->n : 0.0;
  a.iters = iters;
  a.tol = cv ? cv->tol : 0.0;
  a.result = cv ? g->ltotal : nullptr;
  const size_t lds = small_lds(g->n, g->m, cv != nullptr);
  ProfScope prof("pr_small", s);
  if (!cv) return launch<false>(a, lds, s);
  GC_HIP_TRY(launch<true>(a, lds, s));
  double got[2] = {0.0, 0.0};
  GC_HIP_TRY(hipMemcpyAsync(got, g->ltotal, sizeof(got), hipMemcpyDeviceToHost, s));
  GC_HIP_TRY(hipStreamSynchronize(s));
  cv->delta = got[0];
  cv->iters = static_cast<int32_t>(got[1]);
  return hipSuccess;
}

}  // namespace gcx
