// Graph construction on the GPU: exclusive scan, CSR transpose with sorted
// rows, and the TOCAB static partition (Section 3.1, preprocessing phase).
// Runs once per graph / per block width; timed apart from the iterations.

#include <algorithm>
#include <climits>
#include <vector>

#include "gc_device.h"
#include "gc_internal.h"

namespace {

using gcd::kWave;

// ---------------------------------------------------------------------------
// Exclusive scan (reduce tiles -> scan tile totals -> rescan tiles).

constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;
constexpr int kScanTile = kScanThreads * kScanItems;

// Work-group exclusive scan of one int per thread; *total gets the sum.
__device__ int wg_excl_scan(int v, int* total) {
  __shared__ int wave_tot[kScanThreads / kWave];
  const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
  const int incl = gcd::wave_incl_scan(v);
  if (lane == kWave - 1) wave_tot[wid] = incl;
  __syncthreads();
  int off = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < kScanThreads / kWave; ++w) {
    const int x = wave_tot[w];
    off += (w < wid) ? x : 0;
    tot += x;
  }
  __syncthreads();
  *total = tot;
  return off + incl - v;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_reduce(const int32_t* __restrict__ in, int64_t n,
                                                              int32_t* __restrict__ tile_sum) {
  const int64_t base = static_cast<int64_t>(blockIdx.x) * kScanTile;
  int s = 0;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    const int64_t idx = base + i * kScanThreads + threadIdx.x;
    if (idx < n) s += in[idx];
  }
  int tot;
  wg_excl_scan(s, &tot);
  if (threadIdx.x == 0) tile_sum[blockIdx.x] = tot;
}

// One work-group scans all tile sums in place (exclusive).
__global__ __launch_bounds__(kScanThreads) void k_scan_top(int32_t* __restrict__ tile_sum, int64_t nt) {
  int carry = 0;
  for (int64_t base = 0; base < nt; base += kScanTile) {
    int vals[kScanItems];
    int local = 0;
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
      const int64_t idx = base + static_cast<int64_t>(threadIdx.x) * kScanItems + i;
      vals[i] = idx < nt ? tile_sum[idx] : 0;
      local += vals[i];
    }
    int tot;
    int run = carry + wg_excl_scan(local, &tot);
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
      const int64_t idx = base + static_cast<int64_t>(threadIdx.x) * kScanItems + i;
      if (idx < nt) tile_sum[idx] = run;
      run += vals[i];
    }
    carry += tot;
  }
}

__global__ __launch_bounds__(kScanThreads) void k_scan_apply(const int32_t* __restrict__ in,
                                                             int32_t* __restrict__ out, int64_t n,
                                                             const int32_t* __restrict__ tile_off) {
  const int64_t base = static_cast<int64_t>(blockIdx.x) * kScanTile +
                       static_cast<int64_t>(threadIdx.x) * kScanItems;
  int vals[kScanItems];
  int local = 0;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    const int64_t idx = base + i;
    vals[i] = idx < n ? in[idx] : 0;
    local += vals[i];
  }
  int tot;
  int run = tile_off[blockIdx.x] + wg_excl_scan(local, &tot);
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    const int64_t idx = base + i;
    if (idx < n) out[idx] = run;
    if (idx == n - 1) out[n] = run + vals[i];
    run += vals[i];
  }
}

// ---------------------------------------------------------------------------
// Stable partition of arcs by a digit of their key, the one pass that the
// transpose (digits of the destination, low to high) and the TOCAB partition
// (the block of the column) are made of. Arcs (key, row, weight) keep their
// order within a digit, so a transposed row comes out with its sources
// ascending and a block with its rows ascending: no sort of rows, no atomics
// on global memory. A pass is bound by memory: it counts digits per tile of
// kRadixTile arcs (k_radix_count), scans the counts digit-major, then ranks
// each tile's arcs in LDS and writes every digit's run to its place
// (k_radix_move), so writes leave in runs of kRadixTile / digits arcs on
// average. Digits have at most kRadixBits bits (1024 runs per tile of 4096
// arcs: 16-byte runs); the transpose takes at most 8 (64-byte runs: a pass
// more, but whole sectors), the block of a column one pass of its own width
// up to 1024 blocks. Measured on an R-MAT graph of 1.5 M vertices and 23 M
// weighted arcs: a pass 0.20 ms (move 0.16, 3.4 TB/s; count 0.04), so the
// transpose takes 0.62 ms (random scatter through atomics, in-degree atomics
// and per-row sorts: 5.4 ms) and the partition into 46 blocks of 2^15 with
// its local rows 0.38 ms (one wave per merge range walking its rows' blocks
// in order, twice, and a copy per row: 8.3 ms); loading, partitioning and
// exporting the graph 14.4 -> 1.9 ms. Tile shapes tried (move, per pass):
// 512 threads x 16 arcs 0.228 (132 registers: one work-group per CU), 1024 x
// 8 0.180, 512 x 8 0.163, the last held to 80 registers 0.204 (spills).

constexpr int kRadixThreads = 512;
constexpr int kRadixWaves = kRadixThreads / kWave;
constexpr int kRadixItems = 8;  // arcs per thread
constexpr int kRadixTile = kRadixThreads * kRadixItems;
constexpr int kRadixBits = 10;
constexpr int kTransposeBits = 8;
// Rows that a tile marks one by one; over more of them (long runs of empty
// rows) its arcs search for theirs: 10^6 arcs at both ends of 16 M vertices
// in blocks, push, 14.4 ms with one work-group marking the rows between, 0.18
// so; 2 M arcs spread over them (32,000 rows a tile) 229 marked, 251 searched,
// 10^6 spread 216 and 231, 500,000 269 and 218 us.
constexpr int32_t kMarkRows = 24 * kRadixTile;

// Digit counts of every tile, digit-major: counts[d * tiles + tile]. A
// thread reads kRadixItems consecutive keys and adds each run of equal
// digits once (the columns of a row are ascending, so neighbours share a
// block).
__global__ __launch_bounds__(kRadixThreads) void k_radix_count(const int32_t* __restrict__ key, int64_t m, int shift,
                                                               int32_t bins, int32_t tiles,
                                                               int32_t* __restrict__ counts) {
  __shared__ int32_t hist[1 << kRadixBits];
  for (int32_t d = threadIdx.x; d < bins; d += kRadixThreads) hist[d] = 0;
  __syncthreads();
  const int64_t i0 = static_cast<int64_t>(blockIdx.x) * kRadixTile + static_cast<int64_t>(threadIdx.x) * kRadixItems;
  if (i0 < m) {
    const int cnt = static_cast<int>(min<int64_t>(kRadixItems, m - i0));
    int32_t k[kRadixItems];
#pragma unroll
    for (int j = 0; j < kRadixItems; ++j) k[j] = key[i0 + min(j, cnt - 1)];
    int32_t d = (k[0] >> shift) & (bins - 1), run = 1;
#pragma unroll
    for (int j = 1; j < kRadixItems; ++j) {
      const int32_t e = (k[j] >> shift) & (bins - 1);
      if (j < cnt) {
        if (e != d) {
          atomicAdd(&hist[d], run);
          d = e;
          run = 0;
        }
        ++run;
      }
    }
    atomicAdd(&hist[d], run);
  }
  __syncthreads();
  for (int32_t d = threadIdx.x; d < bins; d += kRadixThreads)
    counts[static_cast<int64_t>(d) * tiles + blockIdx.x] = hist[d];
}

// Row owning arc e: the last r in [0, n] with rowptr[r] <= e, by the whole
// wave (64 probes per step: four dependent loads for 2^24 rows).
__device__ __forceinline__ int32_t wave_owner_row(const int32_t* __restrict__ rowptr, int32_t n, int64_t e) {
  const int lane = gcd::lane_id();
  int32_t lo = 0, hi = n;
  while (lo < hi) {  // uniform
    const int32_t step = (hi - lo + kWave - 1) / kWave;
    const int32_t idx = static_cast<int32_t>(min<int64_t>(hi, lo + static_cast<int64_t>(lane + 1) * step));
    const int cnt = __popcll(__ballot(rowptr[idx] <= e));  // a prefix of the lanes
    const int32_t fail = static_cast<int32_t>(min<int64_t>(hi, lo + static_cast<int64_t>(cnt + 1) * step));
    lo = static_cast<int32_t>(min<int64_t>(hi, lo + static_cast<int64_t>(cnt) * step));
    if (cnt < kWave) hi = fail - 1;
  }
  return lo;
}

// Tile of this work-group of k_radix_move: consecutive tiles run on one XCD
// (the GPU hands consecutive work-groups to its kXcds XCDs in turn), since a
// digit's runs of consecutive tiles share cache lines, which one L2 can put
// together and several write back in parts.
constexpr int kXcds = 8;
__device__ __forceinline__ int32_t xcd_tile(int32_t tiles) {
  const int32_t per = (tiles + kXcds - 1) / kXcds;
  return static_cast<int32_t>(blockIdx.x % kXcds) * per + static_cast<int32_t>(blockIdx.x / kXcds);
}
inline int32_t xcd_grid(int32_t tiles) { return (tiles + kXcds - 1) / kXcds * kXcds; }

// LDS bytes of k_radix_move.
constexpr size_t radix_lds(int32_t bins) {
  return sizeof(int32_t) * (kRadixTile + static_cast<size_t>(bins) * (kRadixWaves + 1));
}

struct RadixArgs {
  const int32_t* key;
  const int32_t* row;     // null: the arc's row in rowptr (first pass over a CSR)
  const int32_t* rowptr;
  int32_t n_rows;
  const int32_t* w;       // null: no weights
  int64_t m;
  int32_t shift, bits, tiles;
  const int32_t* base;    // exclusive scan of the counts
  int32_t* key_out;       // null: not wanted
  int32_t* row_out;
  int32_t* w_out;
  uint16_t* low_out;      // null, or: key & low_mask of every arc
  int32_t low_mask;
};

// One pass. Lane l of wave v holds the arcs 512 v + 64 r + l, r < 8, of its
// tile (eight arcs per thread keep two work-groups per CU resident). Ranks: lanes with equal digits find each other with
// one ballot per digit bit, the wave's counter of the digit (LDS) gives the
// arcs of earlier rounds. The three arrays then go through one LDS stage,
// one after another, into digit order, and out in that order.
__global__ __launch_bounds__(kRadixThreads) void k_radix_move(RadixArgs a) {
  extern __shared__ int32_t stage[];  // kRadixTile arcs, then the counters
  const int32_t bins = 1 << a.bits;
  int32_t* cnt = stage + kRadixTile;            // [kRadixWaves][bins]
  int32_t* off = cnt + kRadixWaves * bins;      // [bins]: a digit's place minus its first position in the stage
  __shared__ int32_t wave_tot[kRadixWaves];
  __shared__ int32_t row_first, row_last;
  const int lane = threadIdx.x & (kWave - 1);
  const int wid = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
  const int32_t tile = xcd_tile(a.tiles);
  if (tile >= a.tiles) return;  // uniform
  const int64_t e0 = static_cast<int64_t>(tile) * kRadixTile;
  const int32_t len = static_cast<int32_t>(min<int64_t>(kRadixTile, a.m - e0));  // >= 1
  const int32_t p0 = wid * (kRadixTile / kRadixWaves) + lane;  // position of the thread's arc of round 0
  int32_t key[kRadixItems], row[kRadixItems];  // row: filled here only when it comes from rowptr
#pragma unroll
  for (int r = 0; r < kRadixItems; ++r) key[r] = gcd::ld_stream(a.key + e0 + min(p0 + r * kWave, len - 1));
  if (!a.row) {  // uniform
    // rows of the tile's arcs: each row that starts inside the tile marks its
    // first arc (the last of several starting there wins), then a running
    // maximum
    if (wid == 0) {
      const int32_t r = wave_owner_row(a.rowptr, a.n_rows, e0);
      if (lane == 0) row_first = r;
    } else if (wid == 1) {
      const int32_t r = wave_owner_row(a.rowptr, a.n_rows, e0 + len - 1);
      if (lane == 0) row_last = r;
    }
    __syncthreads();
    const int32_t rf = row_first, rl = row_last;
    if (rl - rf > kMarkRows) {  // uniform
      // mostly empty rows: every arc searches them
      int64_t e[kRadixItems];
#pragma unroll
      for (int r = 0; r < kRadixItems; ++r) {
        e[r] = e0 + min(p0 + r * kWave, len - 1);
        row[r] = rf;
      }
      for (int32_t step = 1 << (31 - __builtin_clz(rl - rf)); step > 0; step >>= 1) {
#pragma unroll
        for (int r = 0; r < kRadixItems; ++r)
          if (step <= rl - row[r] && a.rowptr[row[r] + step] <= e[r]) row[r] += step;
      }
    } else {
      for (int32_t i = threadIdx.x; i < kRadixTile; i += kRadixThreads) stage[i] = 0;
      __syncthreads();
      for (int32_t r = rf + 1 + static_cast<int32_t>(threadIdx.x); r <= rl; r += kRadixThreads) {
        atomicMax(&stage[a.rowptr[r] - e0], r - rf);  // e0 < rowptr[r] < e0 + len
      }
      __syncthreads();
      int32_t v[kRadixItems];
      const int32_t s0 = threadIdx.x * kRadixItems;
#pragma unroll
      for (int j = 0; j < kRadixItems; ++j) {
        v[j] = stage[s0 + j];
        if (j) v[j] = max(v[j], v[j - 1]);
      }
      int32_t incl = v[kRadixItems - 1];
#pragma unroll
      for (int o = 1; o < kWave; o <<= 1) {
        const int32_t t = __shfl_up(incl, o, kWave);
        if (lane >= o) incl = max(incl, t);
      }
      if (lane == kWave - 1) wave_tot[wid] = incl;
      const int32_t up = __shfl_up(incl, 1, kWave);
      __syncthreads();
      int32_t before = lane ? up : 0;
      for (int w = 0; w < wid; ++w) before = max(before, wave_tot[w]);
#pragma unroll
      for (int j = 0; j < kRadixItems; ++j) stage[s0 + j] = rf + max(before, v[j]);
      __syncthreads();
#pragma unroll
      for (int r = 0; r < kRadixItems; ++r) row[r] = stage[p0 + r * kWave];
    }
  }
  for (int32_t i = threadIdx.x; i < kRadixWaves * bins; i += kRadixThreads) cnt[i] = 0;
  __syncthreads();
  // rank of every arc among those of its digit in its wave
  int32_t* mine = cnt + wid * bins;
  int32_t pos[kRadixItems];
#pragma unroll
  for (int r = 0; r < kRadixItems; ++r) {
    const bool in = p0 + r * kWave < len;
    const int32_t d = (key[r] >> a.shift) & (bins - 1);
    uint64_t same = __ballot(in);
    for (int b = 0; b < a.bits; ++b) {  // uniform
      const bool bit = (d >> b) & 1;
      const uint64_t bal = __ballot(bit);
      same &= bit ? bal : ~bal;
    }
    const int32_t old = mine[d];
    gcd::wave_lds_fence();
    if (in && (same & gcd::lanemask_lt()) == 0) mine[d] = old + __popcll(same);
    gcd::wave_lds_fence();
    pos[r] = old + __popcll(same & gcd::lanemask_lt());
  }
  __syncthreads();
  // first stage position of every (digit, wave): exclusive scan over the
  // digits, then over the waves of a digit
  int32_t carry = 0;
  for (int32_t b0 = 0; b0 < bins; b0 += kRadixThreads) {  // uniform
    const int32_t d = b0 + static_cast<int32_t>(threadIdx.x);
    int32_t tot = 0;
    if (d < bins)
      for (int w = 0; w < kRadixWaves; ++w) tot += cnt[w * bins + d];
    const int32_t incl = gcd::wave_incl_scan(tot);
    if (lane == kWave - 1) wave_tot[wid] = incl;
    __syncthreads();
    int32_t start = carry + incl - tot;
    int32_t all = 0;
#pragma unroll
    for (int w = 0; w < kRadixWaves; ++w) {
      start += w < wid ? wave_tot[w] : 0;
      all += wave_tot[w];
    }
    carry += all;
    if (d < bins) {
      off[d] = a.base[static_cast<int64_t>(d) * a.tiles + tile] - start;
      for (int w = 0; w < kRadixWaves; ++w) {
        const int32_t c = cnt[w * bins + d];
        cnt[w * bins + d] = start;
        start += c;
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int r = 0; r < kRadixItems; ++r) pos[r] += mine[(key[r] >> a.shift) & (bins - 1)];
  // keys into digit order, and every stage position's place
  int32_t to[kRadixItems];
#pragma unroll
  for (int r = 0; r < kRadixItems; ++r)
    if (p0 + r * kWave < len) stage[pos[r]] = key[r];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kRadixItems; ++r) {
    const int32_t i = static_cast<int32_t>(threadIdx.x) + r * kRadixThreads;
    to[r] = 0;
    if (i < len) {
      const int32_t k = stage[i];
      to[r] = i + off[(k >> a.shift) & (bins - 1)];
      if (a.key_out) a.key_out[to[r]] = k;
      if (a.low_out) a.low_out[to[r]] = static_cast<uint16_t>(k & a.low_mask);
    }
  }
  if (a.row) {  // uniform
#pragma unroll
    for (int r = 0; r < kRadixItems; ++r) row[r] = gcd::ld_stream(a.row + e0 + min(p0 + r * kWave, len - 1));
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kRadixItems; ++r)
    if (p0 + r * kWave < len) stage[pos[r]] = row[r];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kRadixItems; ++r) {
    const int32_t i = static_cast<int32_t>(threadIdx.x) + r * kRadixThreads;
    if (i < len) a.row_out[to[r]] = stage[i];
  }
  if (!a.w) return;  // uniform
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kRadixItems; ++r)
    if (p0 + r * kWave < len) stage[pos[r]] = gcd::ld_stream(a.w + e0 + p0 + r * kWave);
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kRadixItems; ++r) {
    const int32_t i = static_cast<int32_t>(threadIdx.x) + r * kRadixThreads;
    if (i < len) a.w_out[to[r]] = stage[i];
  }
}

__device__ __forceinline__ int32_t first_at_least(const int32_t* a, int32_t lo, int32_t hi, int64_t key) {
  while (lo < hi) {
    const int32_t mid = lo + ((hi - lo) >> 1);
    if (static_cast<int64_t>(a[mid]) < key) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// First arc in [0, m) with key >= v (m if none), by the whole wave.
__device__ __forceinline__ int32_t wave_first_at_least(const int32_t* __restrict__ key, int64_t m, int32_t v) {
  const int lane = gcd::lane_id();
  int64_t lo = 0, hi = m;
  while (lo < hi) {  // uniform
    const int64_t step = (hi - lo + kWave - 1) / kWave;
    const int64_t at = min(hi - 1, lo + (lane + 1) * step - 1);
    const int cnt = __popcll(__ballot(key[at] < v));  // a prefix of the lanes
    if (cnt == kWave) return static_cast<int32_t>(hi);
    hi = min(hi - 1, lo + (cnt + 1) * step - 1);
    lo += cnt * step;
  }
  return static_cast<int32_t>(lo);
}

// Row offsets of arcs sorted by row: rowptr[v] = first arc with key >= v. A
// work-group stages kOffsetTile keys in LDS and writes the offsets of the
// rows after the previous tile's last key up to its own last key (the last
// tile: up to n), each by a binary search in LDS, if they are at most
// kWideRows. Where arcs are few or leave long runs of rows empty, one
// work-group would walk most of the graph (16 M vertices, 10^6 arcs into the
// last 65,536 of them: 62 ms to load): the rows of wider tiles are written by
// the work-groups after those of the tiles, one per kOffsetTile rows, each by
// a binary search in memory (0.29 ms). One of them meets two wide tiles at
// most, with its first row and with its last. Arcs spread over 16 M vertices,
// load with half this line and with this: 4 M 440, 398 us; 2 M 372, 380;
// 250,000 309, 314 (1425 by tiles alone).
constexpr int kOffsetTile = 4096;
constexpr int32_t kWideRows = 8 * kOffsetTile;

__global__ __launch_bounds__(256) void k_row_offsets(const int32_t* __restrict__ key, int64_t m, int32_t n,
                                                     int32_t tiles, int32_t* __restrict__ rowptr) {
  auto first_row = [&](int64_t t) { return t ? key[t * kOffsetTile - 1] + 1 : 0; };
  auto last_row = [&](int64_t t) { return t == tiles - 1 ? n : key[(t + 1) * kOffsetTile - 1]; };
  const int32_t tile = blockIdx.x;
  if (tile < tiles) {
    __shared__ int32_t k[kOffsetTile];
    const int32_t v0 = first_row(tile), v1 = last_row(tile);
    if (v1 - v0 >= kWideRows) return;  // uniform
    const int64_t i0 = static_cast<int64_t>(tile) * kOffsetTile;
    const int32_t len = static_cast<int32_t>(min<int64_t>(kOffsetTile, m - i0));
    for (int32_t i = threadIdx.x; i < len; i += 256) k[i] = key[i0 + i];
    __syncthreads();
    for (int64_t v = static_cast<int64_t>(v0) + threadIdx.x; v <= v1; v += 256)
      rowptr[v] = static_cast<int32_t>(i0) + first_at_least(k, 0, len, v);
    return;
  }
  __shared__ int32_t end[2];  // arcs at which the first and the last row start
  const int64_t c0 = static_cast<int64_t>(tile - tiles) * kOffsetTile, c1 = min<int64_t>(n, c0 + kOffsetTile - 1);
  const int wid = static_cast<int>(threadIdx.x) / kWave;
  if (wid < 2) {
    const int32_t a = wave_first_at_least(key, m, static_cast<int32_t>(wid ? c1 : c0));
    if (gcd::lane_id() == 0) end[wid] = a;
  }
  __syncthreads();
  const int32_t a0 = end[0], a1 = end[1];
  auto tile_of = [&](int32_t a) { return min(a / kOffsetTile, tiles - 1); };
  const int32_t t0 = tile_of(a0), t1 = tile_of(a1);
  const bool wide0 = last_row(t0) - first_row(t0) >= kWideRows, wide1 = last_row(t1) - first_row(t1) >= kWideRows;
  if (!wide0 && !wide1) return;  // uniform
  for (int64_t v = c0 + threadIdx.x; v <= c1; v += 256) {
    const int32_t a = first_at_least(key, a0, a1, v);
    const int32_t t = tile_of(a);
    if ((t == t0 && wide0) || (t == t1 && wide1)) rowptr[v] = a;
  }
}

// ---------------------------------------------------------------------------
// TOCAB partition: the arcs partitioned by block (rows ascending inside a
// block), then the local rows, which begin where the row or the block
// changes.

// Head bits of 64 arcs (one per wave and step) and their number.
__global__ __launch_bounds__(256) void k_head_bits(const int32_t* __restrict__ row, const int32_t* __restrict__ col,
                                                   int64_t m, int32_t log2W, int64_t words,
                                                   uint64_t* __restrict__ bits, int32_t* __restrict__ cnt) {
  const int lane = gcd::lane_id();
  const int64_t stride = static_cast<int64_t>(gridDim.x) * (256 / kWave);
  for (int64_t w = static_cast<int64_t>(blockIdx.x) * (256 / kWave) + threadIdx.x / kWave; w < words; w += stride) {
    const int64_t i = (w << 6) + lane;
    bool head = false;
    if (i < m) head = i == 0 || row[i] != row[i - 1] || ((col[i] ^ col[i - 1]) >> log2W) != 0;
    const uint64_t b = __ballot(head);
    if (lane == 0) {
      bits[w] = b;
      cnt[w] = __popcll(b);
    }
  }
}

// Local rows: id_map, row_ptr and id16 of every head arc (wrow = exclusive
// scan of the head counts), and, with heads given, the head words of the
// stream layouts: bits at and past arc m are set, so a row walk always stops
// at the end; the word's row count; bit 0 of the word after it.
__global__ __launch_bounds__(256) void k_local_rows(const int32_t* __restrict__ row, int64_t m, int64_t words,
                                                    const uint64_t* __restrict__ bits,
                                                    const int32_t* __restrict__ wrow, int32_t kmask,
                                                    int32_t* __restrict__ id_map, int32_t* __restrict__ row_ptr,
                                                    uint16_t* __restrict__ id16, gc_head_word* __restrict__ heads,
                                                    int64_t head_words) {
  const int lane = gcd::lane_id();
  const int64_t stride = static_cast<int64_t>(gridDim.x) * (256 / kWave);
  const int32_t P = wrow[words];
  auto padded = [&](int64_t w) {  // the bits of word w with those past m set
    const int64_t lo = w << 6;
    if (lo >= m) return ~0ull;
    const uint64_t b = bits[w];
    return lo + 64 > m ? b | (~0ull << (m - lo)) : b;
  };
  const int64_t top = heads ? max(words, head_words) : words;
  for (int64_t w = static_cast<int64_t>(blockIdx.x) * (256 / kWave) + threadIdx.x / kWave; w < top; w += stride) {
    const int32_t before = w < words ? wrow[w] : P;
    if (w < words) {
      const uint64_t b = bits[w];
      if ((b >> lane) & 1ull) {
        const int64_t i = (w << 6) + lane;
        const int32_t l = before + __popcll(b & gcd::lanemask_lt());
        const int32_t v = row[i];
        id_map[l] = v;
        row_ptr[l] = static_cast<int32_t>(i);
        if (id16) id16[l] = static_cast<uint16_t>(v & kmask);
      }
    }
    if (heads && w < head_words && lane == 0) {
      gc_head_word h;
      h.bits = padded(w);
      h.row = before;
      h.next = w + 1 < head_words ? static_cast<int32_t>(padded(w + 1) & 1ull) : 1;
      heads[w] = h;
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) row_ptr[P] = static_cast<int32_t>(m);
}

// First local row of every block: the heads before its first arc.
__global__ void k_block_rows(const int32_t* __restrict__ col, int64_t m, int32_t log2W, int32_t B,
                             const uint64_t* __restrict__ bits, const int32_t* __restrict__ wrow, int64_t words,
                             int32_t* __restrict__ blk_rowoff) {
  const int32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s > B) return;
  int64_t lo = 0, hi = m;  // first arc whose block is s or later
  if (s == B) lo = m;
  else
    while (lo < hi) {
      const int64_t mid = lo + ((hi - lo) >> 1);
      if ((col[mid] >> log2W) < s) lo = mid + 1;
      else hi = mid;
    }
  const int64_t w = lo >> 6;
  blk_rowoff[s] = w < words ? wrow[w] + __popcll(bits[w] & ((1ull << (lo & 63)) - 1ull)) : wrow[words];
}

// range_ptr[j*B + s] = first local row of block s whose row is >= j*k (j = R: block end)
__global__ void k_range_rows(const int32_t* __restrict__ id_map, const int32_t* __restrict__ blk_rowoff, int32_t B,
                             int32_t R, int32_t log2k, int32_t* __restrict__ range_ptr) {
  const int64_t total = static_cast<int64_t>(R + 1) * B;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < total; i += stride) {
    const int32_t s = static_cast<int32_t>(i / (R + 1)), j = static_cast<int32_t>(i - static_cast<int64_t>(s) * (R + 1));
    const int32_t a = blk_rowoff[s], z = blk_rowoff[s + 1];
    range_ptr[static_cast<int64_t>(j) * B + s] = j == R ? z : first_at_least(id_map, a, z, static_cast<int64_t>(j) << log2k);
  }
}

// Structural check that keeps later kernels in bounds: rowptr[0] = 0,
// rowptr[n] = m, rowptr non-decreasing, every column in [0, n).
__global__ void k_check_csr(const int32_t* __restrict__ rowptr, int32_t n, const int32_t* __restrict__ colidx,
                            int64_t m, int32_t* __restrict__ bad) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  const int64_t top = m > n ? m : n;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < top; i += stride) {
    if (i < n) {
      const int32_t a = rowptr[i], b = rowptr[i + 1];
      if (b < a || a < 0 || b > m) atomicOr(bad, 1);
      if (i == 0 && a != 0) atomicOr(bad, 1);
      if (i == n - 1 && b != m) atomicOr(bad, 1);
    }
    if (i < m) {
      const int32_t v = colidx[i];
      if (v < 0 || v >= n) atomicOr(bad, 2);
    }
  }
}

__global__ __launch_bounds__(256) void k_tile_rows(const int32_t* __restrict__ row_ptr, int32_t rows,
                                                   int32_t tile_arcs, int32_t n_tiles, int32_t* __restrict__ tile_row,
                                                   int32_t* __restrict__ longest) {
  const int32_t t = blockIdx.x * 256 + threadIdx.x;
  if (t < n_tiles) tile_row[t] = first_at_least(row_ptr, 0, rows, static_cast<int64_t>(t) * tile_arcs);
  if (t == n_tiles) tile_row[t] = rows;
  if (!longest || blockIdx.x != 0) return;  // uniform
  __shared__ int32_t top[256 / kWave];
  int32_t x = 0;
  for (int32_t r = threadIdx.x; r < rows; r += 256) x = max(x, row_ptr[r + 1] - row_ptr[r]);
  x = gcd::wave_max(x);
  if (gcd::lane_id() == 0) top[threadIdx.x / kWave] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 256 / kWave; ++w) x = max(x, top[w]);
    __hip_atomic_store(longest, x, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// Low 16 bits of (value & mask): a column inside its block, or a row inside
// its merge range.
__global__ void k_col16(const int32_t* __restrict__ col, int64_t m, int32_t mask, uint16_t* __restrict__ col16) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < m; i += stride)
    col16[i] = static_cast<uint16_t>(col[i] & mask);
}

// Rows of block b in merge range j, from the j-major range table.
__global__ void k_seg_counts(const int32_t* __restrict__ range_ptr, int32_t B, int32_t R, int32_t* __restrict__ cnt) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;  // i = j*B + b
  if (i >= static_cast<int64_t>(B) * R) return;
  cnt[i] = range_ptr[i + B] - range_ptr[i];
}

// seg[b][j] = (first local row of block b in range j, shift that moves the
// block-major row index to its range-major index); rstart[j] = first
// range-major index of range j.
__global__ void k_seg_table(const int32_t* __restrict__ range_ptr, const int32_t* __restrict__ rm_start, int32_t B,
                            int32_t R, int64_t P, int2* __restrict__ seg, int32_t* __restrict__ rstart) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;  // i = b*(R+1) + j
  if (i >= static_cast<int64_t>(B) * (R + 1)) return;
  const int32_t b = static_cast<int32_t>(i / (R + 1)), j = static_cast<int32_t>(i % (R + 1));
  const int64_t jb = static_cast<int64_t>(j) * B + b;
  const int32_t first = range_ptr[jb];
  seg[i] = make_int2(first, j < R ? rm_start[jb] - first : 0);
  if (b == 0) rstart[j] = j < R ? rm_start[jb] : static_cast<int32_t>(P);
}

// Arcs per chunk, of kSizes sizes from `base` up in steps of 1/16: the one
// that costs least. The pull runs a round of 256 chunks (one per CU) in its
// longest chunk's time and `fill` (in arcs: loading the slice, and the waves
// that end early), so a few chunks past a multiple of 256 cost as much as 256
// more: 300,007 vertices of 16 arcs took 487 us for 20 iterations in 264
// chunks, 389 in 248. Lane i of each wave counts size i's chunks over the
// wave's share of the blocks; a block has at least one chunk per cap ranges.
constexpr int kSizes = 64;
__global__ __launch_bounds__(1024) void k_chunk_size(const int32_t* __restrict__ range_ptr,
                                                     const int32_t* __restrict__ row_ptr, int32_t B, int32_t R,
                                                     int32_t cap, int32_t base, int32_t fill,
                                                     int32_t* __restrict__ out) {
  __shared__ int32_t count[kSizes], longest[kSizes];
  const int lane = gcd::lane_id(), wave = static_cast<int>(threadIdx.x) / kWave;
  if (wave == 0) count[lane] = longest[lane] = 0;
  __syncthreads();
  const uint32_t size = static_cast<uint32_t>(fminf(base * exp2f(lane * 0.0875f), 2147483647.f));
  int32_t mine = 0;
  uint32_t top = 0;
  const uint32_t least = static_cast<uint32_t>((R + cap - 1) / cap);
  for (int32_t b0 = wave * kWave; b0 < B; b0 += 1024) {
    const int32_t b = min(b0 + lane, B - 1);
    const int32_t arcs =
        b0 + lane < B ? row_ptr[range_ptr[static_cast<int64_t>(R) * B + b]] - row_ptr[range_ptr[b]] : 0;
    for (int l = 0; l < kWave; ++l) {
      const uint32_t a = __shfl(arcs, l);
      const uint32_t pieces = a ? max((a + size - 1) / size, least) : 0u;
      mine += pieces;
      top = max(top, pieces ? (a + pieces - 1) / pieces : 0u);
    }
  }
  atomicAdd(&count[lane], mine);
  atomicMax(&longest[lane], static_cast<int32_t>(top));
  __syncthreads();
  if (wave == 0) {
    float best = static_cast<float>((count[lane] + 255) / 256) * (static_cast<float>(longest[lane]) + fill);
    int at = lane;
    for (int d = 1; d < kWave; d *= 2) {
      const float o = __shfl_xor(best, d);
      const int oa = __shfl_xor(at, d);
      if (o < best || (o == best && oa < at)) best = o, at = oa;
    }
    if (lane == at) out[1] = static_cast<int32_t>(size);
  }
}

// Chunks of the stream-layout pull, one wave per block: a block's ranges are
// cut into chunks of about equal arc counts (at most out[1], at most `cap`
// ranges each). From range j0 a chunk runs to the first boundary that gives
// it its share of the block's arcs, found with 64 probes per step. out[0]
// counts the chunks; chunk i follows at out + kChunkInts (i + 1): first row,
// end row, block, first range, ranges, arcs.
constexpr int kChunkInts = 8;
__global__ __launch_bounds__(256) void k_cut_chunks(const int32_t* __restrict__ range_ptr,
                                                    const int32_t* __restrict__ row_ptr, int32_t B, int32_t R,
                                                    int32_t cap, int32_t most, int32_t* __restrict__ out) {
  const int32_t b = static_cast<int32_t>(blockIdx.x) * (256 / kWave) + static_cast<int32_t>(threadIdx.x) / kWave;
  if (b >= B) return;  // uniform over the wave
  const int lane = gcd::lane_id();
  auto arc_at = [&](int32_t j) { return row_ptr[range_ptr[static_cast<int64_t>(j) * B + b]]; };
  const int64_t mb = arc_at(R) - arc_at(0), target = out[1];
  if (mb == 0) return;
  const int64_t pieces = max<int64_t>((R + cap - 1) / cap, (mb + target - 1) / target);
  const int64_t per = (mb + pieces - 1) / pieces;  // arcs per chunk of this block
  for (int32_t ja = 0; ja < R;) {
    const int32_t a0 = arc_at(ja), top = min(R, ja + cap);
    int32_t lo = ja + 1, hi = top;  // first j in (ja, top] with per arcs or more, else top
    while (lo < hi) {  // uniform
      const int32_t step = (hi - lo + kWave - 1) / kWave;
      const int32_t j = min(hi, lo + lane * step);
      const int cnt = __popcll(__ballot(arc_at(j) - a0 < per));  // a prefix of the lanes
      const int32_t fail = lo + cnt * step;  // the first probe with enough (past hi: none)
      if (cnt == 0) {
        hi = lo;
      } else {
        lo = min(hi, lo + (cnt - 1) * step + 1);
        hi = min(hi, fail);
      }
    }
    if (lane == 0) {
      const int32_t r0 = range_ptr[static_cast<int64_t>(ja) * B + b], r1 = range_ptr[static_cast<int64_t>(lo) * B + b];
      if (r1 > r0) {
        const int32_t i = atomicAdd(out, 1);
        if (i < most) {
          int32_t* c = out + kChunkInts * (static_cast<int64_t>(i) + 1);
          c[0] = r0;
          c[1] = r1;
          c[2] = b;
          c[3] = ja;
          c[4] = lo - ja;
          c[5] = arc_at(lo) - a0;
        }
      }
    }
    ja = lo;
  }
}

// id16 of every local row, scattered to the row's range-major index.
__global__ void k_id16_stream(const int32_t* __restrict__ id_map, int64_t P, const int32_t* __restrict__ blk_rowoff,
                              int32_t B, int32_t R, int32_t log2k, const int2* __restrict__ seg,
                              uint16_t* __restrict__ id16s) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t r = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; r < P; r += stride) {
    const int32_t v = id_map[r];
    const int32_t j = v >> log2k;
    int32_t lo = 0, hi = B;  // block: last b with blk_rowoff[b] <= r
    while (hi - lo > 1) {
      const int32_t mid = (lo + hi) >> 1;
      if (blk_rowoff[mid] <= r) lo = mid;
      else hi = mid;
    }
    id16s[r + seg[static_cast<int64_t>(lo) * (R + 1) + j].y] = static_cast<uint16_t>(v & ((1 << log2k) - 1));
  }
}

// cap: only for kernels that stride over their items; others get one thread per item.
inline int grid_for(int64_t items, int threads, int cap = INT_MAX) {
  const int64_t g = (items + threads - 1) / threads;
  return static_cast<int>(std::max<int64_t>(1, std::min<int64_t>(g, cap)));
}

// Entries of the tile sums a scan of n entries needs, and the scan itself
// with the caller's tile sums (it only queues work).
inline int64_t scan_tiles(int64_t n) { return (n + kScanTile - 1) / kScanTile; }

hipError_t scan_queue(const int32_t* in, int32_t* out, int64_t n, int32_t* tile, hipStream_t s) {
  if (n == 0) return hipMemsetAsync(out, 0, sizeof(int32_t), s);
  const int64_t tiles = scan_tiles(n);
  k_scan_reduce<<<tiles, kScanThreads, 0, s>>>(in, n, tile);
  k_scan_top<<<1, kScanThreads, 0, s>>>(tile, tiles);
  k_scan_apply<<<tiles, kScanThreads, 0, s>>>(in, out, n, tile);
  return hipGetLastError();
}

// Digits of a key of `bits` bits: passes of at most `most` bits, of equal
// width as far as that goes.
struct Digits {
  int passes, width;
  Digits(int bits, int most) {
    bits = std::max(bits, 1);
    passes = (bits + most - 1) / most;
    width = (bits + passes - 1) / passes;
  }
};

inline int key_bits(int64_t values) {  // bits of the largest of `values` values
  int b = 0;
  while ((int64_t{1} << b) < values) ++b;
  return b;
}

// Scratch of a radix pass in a slab: digit counts, their scan and its tile
// sums.
struct RadixScratch {
  size_t i_counts, i_base, i_tile;
  int32_t *counts = nullptr, *base = nullptr, *tile = nullptr;
  int32_t tiles;
  RadixScratch(int64_t m, int width, gcx::Slab& slab) {
    tiles = static_cast<int32_t>((m + kRadixTile - 1) / kRadixTile);
    const int64_t entries = static_cast<int64_t>(tiles) << width;
    i_counts = slab.reserve(sizeof(int32_t) * entries);
    i_base = slab.reserve(sizeof(int32_t) * (entries + 1));
    i_tile = slab.reserve(sizeof(int32_t) * scan_tiles(entries));
  }
  void take(const gcx::Slab& slab, void* p) {
    counts = slab.take<int32_t>(p, i_counts);
    base = slab.take<int32_t>(p, i_base);
    tile = slab.take<int32_t>(p, i_tile);
  }
};

// Queues one pass (m > 0).
hipError_t radix_pass(RadixArgs a, const RadixScratch& r, hipStream_t s) {
  const int32_t bins = 1 << a.bits;
  a.tiles = r.tiles;
  a.base = r.base;
  k_radix_count<<<r.tiles, kRadixThreads, 0, s>>>(a.key, a.m, a.shift, bins, r.tiles, r.counts);
  GC_HIP_TRY(hipGetLastError());
  GC_HIP_TRY(scan_queue(r.counts, r.base, static_cast<int64_t>(r.tiles) << a.bits, r.tile, s));
  k_radix_move<<<xcd_grid(r.tiles), kRadixThreads, radix_lds(bins), s>>>(a);
  return hipGetLastError();
}

// The LDS limit of the pass kernel.
hipError_t radix_setup() {
  static const hipError_t attr =
      hipFuncSetAttribute(reinterpret_cast<const void*>(&k_radix_move), hipFuncAttributeMaxDynamicSharedMemorySize,
                          static_cast<int>(radix_lds(1 << kRadixBits)));
  return attr;
}

}  // namespace

namespace gcx {

hipError_t check_csr(int32_t n, int64_t m, const int32_t* rowptr, const int32_t* colidx, int32_t* bad_out,
                     hipStream_t s) {
  Buf bad(sizeof(int32_t), s);
  if (!bad.p) return hipErrorOutOfMemory;
  GC_HIP_TRY(hipMemsetAsync(bad.p, 0, sizeof(int32_t), s));
  k_check_csr<<<grid_for(std::max<int64_t>(n, m), 256, 65536), 256, 0, s>>>(rowptr, n, colidx, m,
                                                                              bad.as<int32_t>());
  GC_HIP_TRY(hipGetLastError());
  GC_HIP_TRY(hipMemcpyAsync(bad_out, bad.p, sizeof(int32_t), hipMemcpyDeviceToHost, s));
  return hipStreamSynchronize(s);
}

hipError_t build_tiles(const int32_t* row_ptr, int64_t rows, int64_t arcs, int32_t tile_arcs, int32_t** out,
                       int32_t* n_tiles, hipStream_t s, int32_t* longest) {
  const int64_t nt = arcs / tile_arcs + 1;  // arc index `arcs` (trailing empty rows) falls in the last tile
  *n_tiles = static_cast<int32_t>(nt);
  *out = static_cast<int32_t*>(dev_alloc(sizeof(int32_t) * (nt + 1), s));
  if (!*out) return hipErrorOutOfMemory;
  k_tile_rows<<<grid_for(nt + 1, 256, INT_MAX), 256, 0, s>>>(row_ptr, static_cast<int32_t>(rows), tile_arcs,
                                                             static_cast<int32_t>(nt), *out, longest);
  return hipGetLastError();
}

hipError_t scan_exclusive(const int32_t* in, int32_t* out, int64_t n, hipStream_t s) {
  Buf tile(sizeof(int32_t) * std::max<int64_t>(scan_tiles(n), 1), s);
  if (!tile.p) return hipErrorOutOfMemory;
  GC_HIP_TRY(scan_queue(in, out, n, tile.as<int32_t>(), s));
  return hipStreamSynchronize(s);  // the tile buffer is released on return
}

// Stable passes over the destination's digits, low to high: in CSR order
// the sources ascend, so each transposed row keeps them ascending. The
// passes alternate between the scratch arrays and t_colidx / t_w, the last
// one ending in those; its keys give the row offsets.
hipError_t build_transpose(int32_t n, int64_t m, const int32_t* rowptr, const int32_t* colidx,
                           const int32_t* w, int32_t* t_rowptr, int32_t* t_colidx, int32_t* t_w,
                           hipStream_t s) {
  if (m == 0) {
    GC_HIP_TRY(hipMemsetAsync(t_rowptr, 0, sizeof(int32_t) * (static_cast<size_t>(n) + 1), s));
    return hipStreamSynchronize(s);
  }
  GC_HIP_TRY(radix_setup());
  const Digits dg(key_bits(n), kTransposeBits);
  const size_t mb = sizeof(int32_t) * static_cast<size_t>(m);
  const bool many = dg.passes > 1;
  Slab slab;
  const size_t k0 = slab.reserve(mb), k1 = slab.reserve(many ? mb : 0), r1 = slab.reserve(many ? mb : 0),
               w1 = slab.reserve(many && w ? mb : 0);
  RadixScratch scratch(m, dg.width, slab);
  Buf mem(slab.total, s);
  if (!mem.p) return hipErrorOutOfMemory;
  scratch.take(slab, mem.p);
  int32_t* const keys[2] = {slab.take<int32_t>(mem.p, k0), slab.take<int32_t>(mem.p, k1)};
  int32_t* const rows[2] = {t_colidx, slab.take<int32_t>(mem.p, r1)};
  int32_t* const ws[2] = {t_w, slab.take<int32_t>(mem.p, w1)};
  RadixArgs a{};
  a.key = colidx;
  a.rowptr = rowptr;
  a.n_rows = n;
  a.w = w;
  a.m = m;
  a.bits = dg.width;
  for (int p = 0; p < dg.passes; ++p) {
    const int o = (dg.passes - 1 - p) & 1;
    a.shift = p * dg.width;
    a.key_out = keys[o];
    a.row_out = rows[o];
    a.w_out = ws[o];
    GC_HIP_TRY(radix_pass(a, scratch, s));
    a.key = keys[o];
    a.row = rows[o];
    if (w) a.w = ws[o];
  }
  const int32_t tiles = grid_for(m, kOffsetTile);
  k_row_offsets<<<tiles + grid_for(static_cast<int64_t>(n) + 1, kOffsetTile), 256, 0, s>>>(keys[0], m, n, tiles, t_rowptr);
  GC_HIP_TRY(hipGetLastError());
  return hipStreamSynchronize(s);  // the Buf is released on return
}

// Stream layout of an LDS-resident pull partition: padded 16-bit columns,
// head bits, wave-tile rows, the range-major position table, range-major
// id16, and chunks (one work-group each) cut at merge-range boundaries so
// a chunk's slice of the position table fits in LDS beside the block's slice.
hipError_t build_lds_stream(gc_tocab t, hipStream_t s) {
  const int32_t B = t->B, R = t->mR;
  const int64_t P = t->P, m = t->m;
  const int64_t entries = static_cast<int64_t>(B) * (R + 1);
  t->seg = static_cast<int2*>(dev_alloc(sizeof(int2) * entries, s));
  t->rstart = static_cast<int32_t*>(dev_alloc(sizeof(int32_t) * (R + 1), s));
  t->id16s = static_cast<uint16_t*>(dev_alloc(sizeof(uint16_t) * (std::max<int64_t>(P, 1) + 8), s));
  if (!t->seg || !t->rstart || !t->id16s) return hipErrorOutOfMemory;
  t->bytes += static_cast<int64_t>(sizeof(uint16_t)) * (t->m_pad + P) + 16 * (t->m_pad / 64 + 1) + 8 * entries +
              4 * (R + 1);

  // range-major start of every (range j, block b) slice: exclusive scan of
  // the slice sizes in j-major order
  const int64_t BR = static_cast<int64_t>(B) * R;
  // Sizes from four chunks per CU (but kLdsChunkArcs) up.
  // A round costs 8 us more than its arcs at 2^14 vertices per block
  // (32 M arcs in one round 79 us an iteration, in two 87): about 24 K arcs.
  const int32_t base = static_cast<int32_t>(std::max<int64_t>(m / 1024, kLdsChunkArcs));
  const int32_t fill = 16384 + t->W / 2;
  const int32_t cap = lds_seg_cap(t->W);
  // no block has more chunks than its share of base-sized pieces (or the
  // least that cap allows), one cut short by `cap` per cap ranges, and two more
  const int64_t most = m / base + static_cast<int64_t>(B) * (2 * ((R + cap - 1) / cap) + 2);
  Slab slab;
  const size_t i_cnt = slab.reserve(sizeof(int32_t) * BR), i_rm = slab.reserve(sizeof(int32_t) * (BR + 1)),
               i_tile = slab.reserve(sizeof(int32_t) * scan_tiles(BR)),
               i_chunks = slab.reserve(sizeof(int32_t) * kChunkInts * (most + 1));
  Buf mem(slab.total, s);
  if (!mem.p) return hipErrorOutOfMemory;
  int32_t* const cnt = slab.take<int32_t>(mem.p, i_cnt);
  int32_t* const rm = slab.take<int32_t>(mem.p, i_rm);
  int32_t* const dch = slab.take<int32_t>(mem.p, i_chunks);
  const int32_t* const range_ptr = t->mrange;
  GC_HIP_TRY(hipMemsetAsync(dch, 0, sizeof(int32_t) * kChunkInts, s));
  k_chunk_size<<<1, 1024, 0, s>>>(range_ptr, t->row_ptr, B, R, cap, base, fill, dch);
  k_cut_chunks<<<grid_for(B, 256 / kWave), 256, 0, s>>>(range_ptr, t->row_ptr, B, R, cap,
                                                        static_cast<int32_t>(most), dch);
  k_seg_counts<<<grid_for(BR, 256, INT_MAX), 256, 0, s>>>(range_ptr, B, R, cnt);
  GC_HIP_TRY(hipGetLastError());
  // (the pageable copies wait for the kernels before them)
  std::vector<int32_t> hch(kChunkInts);
  GC_HIP_TRY(hipMemcpyAsync(hch.data(), dch, sizeof(int32_t) * kChunkInts, hipMemcpyDeviceToHost, s));
  GC_HIP_TRY(hipStreamSynchronize(s));
  const int32_t found = hch[0];
  if (found > most) return hipErrorUnknown;
  hch.resize(static_cast<size_t>(kChunkInts) * found);
  GC_HIP_TRY(scan_queue(cnt, rm, BR, slab.take<int32_t>(mem.p, i_tile), s));
  k_seg_table<<<grid_for(entries, 256, INT_MAX), 256, 0, s>>>(range_ptr, rm, B, R, P, t->seg, t->rstart);
  if (P > 0)
    k_id16_stream<<<grid_for(P, 256, 65536), 256, 0, s>>>(t->id_map, P, t->blk_rowoff, B, R, __builtin_ctz(t->mk), t->seg,
                                                          t->id16s);
  GC_HIP_TRY(hipGetLastError());
  if (found > 0)
    GC_HIP_TRY(hipMemcpyAsync(hch.data(), dch + kChunkInts, sizeof(int32_t) * hch.size(), hipMemcpyDeviceToHost, s));
  GC_HIP_TRY(hipStreamSynchronize(s));
  struct Chunk {
    int32_t beg, end, blk, j0, ns;
    int64_t arcs;
  };
  std::vector<Chunk> ch(static_cast<size_t>(found));
  int32_t seg_max = 1;
  int64_t top = 1;
  for (int32_t i = 0; i < found; ++i) {
    const int32_t* c = hch.data() + static_cast<size_t>(kChunkInts) * i;
    ch[i] = {c[0], c[1], c[2], c[3], c[4], c[5]};
    seg_max = std::max(seg_max, c[4]);
    top = std::max<int64_t>(top, c[5] + 1);
  }
  // the blocks' waves append in any order
  std::sort(ch.begin(), ch.end(), [](const Chunk& x, const Chunk& y) {
    return x.blk != y.blk ? x.blk < y.blk : x.j0 < y.j0;
  });
  // Dispatch order, XCD aware: the GPU hands consecutive work-groups to its
  // kXcds XCDs in turn (work-group i to XCD i mod kXcds), and each XCD has
  // its own L2. The chunks in block order are cut into one run of about
  // equal arcs per XCD, so a block's slice of c comes from memory once (twice
  // where the cut falls inside it) and from that L2 for its other chunks;
  // whole blocks dealt to the XCDs left 20 to 30 % of the CUs without a chunk
  // where blocks are few. Longer chunks run first, in eighths of the longest
  // (equal ones keep their order: neighbours share a slice and write
  // neighbouring partials); shorter lists are padded with empty chunks.
  std::vector<std::vector<int32_t>> xcd(kXcds);
  // no XCD takes more chunks than its CUs run in the least number of rounds,
  // or leaves the XCDs after it more than that
  const size_t full = (ch.size() + 255) / 256 * (256 / kXcds);
  int64_t before = 0;
  int x = 0;
  for (size_t i = 0; i < ch.size(); ++i) {
    // past its share of the arcs (the chunk's middle decides): the next XCD
    while (x + 1 < kXcds && (xcd[x].size() >= full || (2 * before + ch[i].arcs > 2 * m / kXcds * (x + 1) &&
                                                       ch.size() - i <= full * static_cast<size_t>(kXcds - 1 - x))))
      ++x;
    xcd[x].push_back(static_cast<int32_t>(i));
    before += ch[i].arcs;
  }
  for (auto& l : xcd)
    std::stable_sort(l.begin(), l.end(),
                     [&](int32_t a, int32_t b) { return ch[a].arcs * 8 / top > ch[b].arcs * 8 / top; });
  size_t longest = 0;
  for (const auto& l : xcd) longest = std::max(longest, l.size());
  std::vector<int32_t> beg, end, blk, j0v, nsv;
  for (size_t pos = 0; pos < longest; ++pos)
    for (int x = 0; x < kXcds; ++x) {
      if (pos < xcd[x].size()) {
        const Chunk& c = ch[xcd[x][pos]];
        beg.push_back(c.beg);
        end.push_back(c.end);
        blk.push_back(c.blk);
        j0v.push_back(c.j0);
        nsv.push_back(c.ns);
      } else {  // padding: no rows (the kernel returns at once)
        beg.push_back(0);
        end.push_back(0);
        blk.push_back(0);
        j0v.push_back(0);
        nsv.push_back(1);
      }
    }
  if (ch.empty()) beg.clear(), end.clear(), blk.clear(), j0v.clear(), nsv.clear();
  const int32_t nch = static_cast<int32_t>(beg.size());
  t->n_chunks = nch;
  t->seg_max = seg_max;
  const size_t room = static_cast<size_t>(std::max(nch, 1));
  t->chunk_beg = static_cast<int32_t*>(dev_alloc(sizeof(int32_t) * 5 * room, s));
  if (!t->chunk_beg) return hipErrorOutOfMemory;
  t->chunk_end = t->chunk_beg + room;
  t->chunk_blk = t->chunk_end + room;
  t->chunk_j0 = t->chunk_blk + room;
  t->chunk_ns = t->chunk_j0 + room;
  t->bytes += 5 * static_cast<int64_t>(sizeof(int32_t) * room);
  std::vector<int32_t> all;
  if (nch > 0) {
    all.reserve(5 * room);
    for (const auto* v : {&beg, &end, &blk, &j0v, &nsv}) all.insert(all.end(), v->begin(), v->end());
    GC_HIP_TRY(hipMemcpyAsync(t->chunk_beg, all.data(), sizeof(int32_t) * all.size(), hipMemcpyHostToDevice, s));
  }
  return hipStreamSynchronize(s);  // host vectors and Bufs are released on return
}

// ---- expanded contributions of the TOCAB push ----
// A push block's local rows (source u, block b) are ordered by source, so
// the rows of block b whose source lies in source block s (the W sources
// [sW, (s+1)W)) are one run, bounded by the range table at the merge
// ranges s W/k and (s+1) W/k. The work-group that has just updated the
// vertices of source block s holds their new contributions and writes them
// to each of those B runs. Long runs (128 rows or more on average) are
// walked in place, with xid16[l] = the source of row l as an offset inside
// its source block. Short ones are listed block after block per source
// block (the source-major order): xperm[q] is the row at position q,
// xid16[q] its source offset, xstart[s] the first position of source
// block s.

// cnt[s*B + b] = local rows of block b whose source lies in source block s.
__global__ void k_push_run_counts(const int32_t* __restrict__ range_ptr, int32_t B, int32_t R, int32_t S,
                                  int32_t shift, int32_t* __restrict__ cnt) {
  const int64_t total = static_cast<int64_t>(S) * B;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < total; i += stride) {
    const int64_t s = i / B, b = i - s * B;
    const int64_t j0 = s << shift, j1 = min<int64_t>(R, (s + 1) << shift);
    cnt[i] = range_ptr[j1 * B + b] - range_ptr[j0 * B + b];
  }
}

// Source-major position of every local row (base: exclusive scan of cnt).
__global__ void k_push_perm(const int32_t* __restrict__ range_ptr, const int32_t* __restrict__ base,
                            const int32_t* __restrict__ id_map, int32_t B, int32_t S, int32_t shift,
                            int32_t wmask, int32_t* __restrict__ xperm, uint16_t* __restrict__ xid16,
                            int32_t* __restrict__ xstart) {
  const int64_t total = static_cast<int64_t>(S) * B;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < total; i += stride) {
    const int64_t s = i / B, b = i - s * B;
    const int32_t st = range_ptr[(s << shift) * B + b];
    const int32_t q0 = base[i], len = base[i + 1] - q0;
    for (int32_t k = 0; k < len; ++k) {
      xperm[q0 + k] = st + k;
      xid16[q0 + k] = static_cast<uint16_t>(id_map[st + k] & wmask);
    }
    if (b == 0) xstart[s] = q0;
    if (i == 0) xstart[S] = base[total];
  }
}

// Builds t's expanded-contribution form (GC_PUSH partitions whose block
// sums fit in LDS).
hipError_t build_push_expand(gc_tocab t, hipStream_t s) {
  const int32_t B = t->B, R = t->R;
  const int32_t S = static_cast<int32_t>((static_cast<int64_t>(t->n_rows) + t->W - 1) >> t->log2W);
  const int64_t SB = static_cast<int64_t>(S) * B;
  const size_t Pn = static_cast<size_t>(std::max<int64_t>(t->P, 1));
  t->n_sblk = S;
  // padded so that the 8-byte read of the last group of four rows stays inside
  t->xid16 = static_cast<uint16_t*>(dev_alloc(sizeof(uint16_t) * (Pn + 8), s));
  t->xc = static_cast<float*>(dev_alloc(sizeof(float) * 2 * push_xc_stride(t->P), s));
  if (!t->xid16 || !t->xc) return hipErrorOutOfMemory;
  t->bytes += static_cast<int64_t>(Pn) * 2 + 16 + 8 * push_xc_stride(t->P);
  GC_HIP_TRY(hipMemsetAsync(t->xid16, 0, sizeof(uint16_t) * (Pn + 8), s));
  if (t->P >= kPushLongRun * SB) {
    k_col16<<<grid_for(t->P, 256, 65536), 256, 0, s>>>(t->id_map, t->P, t->W - 1, t->xid16);
    GC_HIP_TRY(hipGetLastError());
  } else {
    const int32_t shift = t->log2W - t->log2k;
    Buf cnt(sizeof(int32_t) * SB, s), base(sizeof(int32_t) * (SB + 1), s);
    if (!cnt.p || !base.p) return hipErrorOutOfMemory;
    k_push_run_counts<<<grid_for(SB, 256, 65536), 256, 0, s>>>(t->range_ptr, B, R, S, shift, cnt.as<int32_t>());
    GC_HIP_TRY(hipGetLastError());
    GC_HIP_TRY(scan_exclusive(cnt.as<int32_t>(), base.as<int32_t>(), SB, s));
    t->xperm = static_cast<int32_t*>(dev_alloc(sizeof(int32_t) * Pn, s));
    t->xstart = static_cast<int32_t*>(dev_alloc(sizeof(int32_t) * (S + 1), s));
    if (!t->xperm || !t->xstart) return hipErrorOutOfMemory;
    t->bytes += static_cast<int64_t>(Pn) * 4 + 4 * (S + 1);
    k_push_perm<<<grid_for(SB, 256, 65536), 256, 0, s>>>(t->range_ptr, base.as<int32_t>(), t->id_map, B, S, shift,
                                                         t->W - 1, t->xperm, t->xid16, t->xstart);
    GC_HIP_TRY(hipGetLastError());
    GC_HIP_TRY(hipStreamSynchronize(s));  // before the Bufs are released
  }
  t->bytes += static_cast<int64_t>(sizeof(uint16_t)) * t->pm_pad + 16 * (t->pm_pad / 64 + 1);
  return hipSuccess;
}

hipError_t build_partition(gc_tocab t, const int32_t* a_rowptr, const int32_t* a_col, const int32_t* a_w,
                           hipStream_t s) {
  const int32_t B = t->B, R = t->R;
  const int64_t m = t->m;
  const size_t mn = static_cast<size_t>(std::max<int64_t>(m, 1));
  const int64_t words = (m + 63) / 64;  // of head bits
  const bool pull_stream = t->dir == GC_PULL && pull_streams(t->n_rows, m, t->W, t->k);
  const bool push_stream = t->dir == GC_PUSH && !t->inner && push_expands(t->n_rows, m, t->W, t->k);
  t->mk = t->dir == GC_PULL ? merge_width(t->n_rows, m, t->W, t->k) : t->k;
  t->mR = (t->n_rows + t->mk - 1) / t->mk;
  const int64_t tile = wave_tile_arcs();
  const int64_t m_pad = (m / tile + 2) * tile, head_words = m_pad / 64 + 1;
  t->col = static_cast<int32_t*>(dev_alloc(sizeof(int32_t) * mn, s));
  if (t->weighted) t->w = static_cast<int32_t*>(dev_alloc(sizeof(int32_t) * mn, s));
  t->range_ptr = static_cast<int32_t*>(dev_alloc(sizeof(int32_t) * (R + 1) * static_cast<size_t>(B), s));
  t->blk_rowoff = static_cast<int32_t*>(dev_alloc(sizeof(int32_t) * (B + 1), s));
  if (!t->col || (t->weighted && !t->w) || !t->range_ptr || !t->blk_rowoff) return hipErrorOutOfMemory;
  t->mrange = t->range_ptr;
  if (t->mk != t->k)
    t->mrange = static_cast<int32_t*>(dev_alloc(sizeof(int32_t) * (t->mR + 1) * static_cast<size_t>(B), s));
  if (!t->mrange) return hipErrorOutOfMemory;
  uint16_t* col16 = nullptr;
  gc_head_word* heads = nullptr;
  if (pull_stream || push_stream) {
    col16 = static_cast<uint16_t*>(dev_alloc(sizeof(uint16_t) * m_pad, s));
    heads = static_cast<gc_head_word*>(dev_alloc(sizeof(gc_head_word) * head_words, s));
    // owned by the partition from here on
    (pull_stream ? t->col16 : t->pcol16) = col16;
    (pull_stream ? t->heads : t->pheads) = heads;
    (pull_stream ? t->m_pad : t->pm_pad) = m_pad;
    if (!col16 || !heads) return hipErrorOutOfMemory;
    GC_HIP_TRY(hipMemsetAsync(col16 + m, 0, sizeof(uint16_t) * (m_pad - m), s));
  }

  // the arcs block by block: passes over the digits of the block, the
  // others than the last (more than 2^kRadixBits blocks) through scratch
  GC_HIP_TRY(radix_setup());
  const Digits dg(key_bits(B), kRadixBits);
  const size_t mb = sizeof(int32_t) * mn;
  const bool two = dg.passes > 1;  // at most 32768 blocks: two passes
  Slab slab;
  const size_t i_row = slab.reserve(mb), i_k1 = slab.reserve(two ? mb : 0), i_r1 = slab.reserve(two ? mb : 0),
               i_w1 = slab.reserve(two && t->weighted ? mb : 0), i_bits = slab.reserve(sizeof(uint64_t) * words),
               i_wcnt = slab.reserve(sizeof(int32_t) * words), i_wrow = slab.reserve(sizeof(int32_t) * (words + 1)),
               i_wtile = slab.reserve(sizeof(int32_t) * scan_tiles(words));
  RadixScratch scratch(m, dg.width, slab);
  Buf mem(slab.total, s);
  if (!mem.p) return hipErrorOutOfMemory;
  scratch.take(slab, mem.p);
  int32_t* const row = slab.take<int32_t>(mem.p, i_row);
  uint64_t* const bits = slab.take<uint64_t>(mem.p, i_bits);
  int32_t* const wcnt = slab.take<int32_t>(mem.p, i_wcnt);
  int32_t* const wrow = slab.take<int32_t>(mem.p, i_wrow);
  if (m > 0) {
    RadixArgs a{};
    a.key = a_col;
    a.rowptr = a_rowptr;
    a.n_rows = t->n_rows;
    a.w = t->weighted ? a_w : nullptr;
    a.m = m;
    a.bits = dg.width;
    a.shift = t->log2W;
    if (two) {
      a.key_out = slab.take<int32_t>(mem.p, i_k1);
      a.row_out = slab.take<int32_t>(mem.p, i_r1);
      a.w_out = slab.take<int32_t>(mem.p, i_w1);
      GC_HIP_TRY(radix_pass(a, scratch, s));
      a.key = a.key_out;
      a.row = a.row_out;
      if (a.w) a.w = a.w_out;
      a.shift += dg.width;
    }
    a.key_out = t->col;
    a.row_out = row;
    a.w_out = t->w;
    a.low_out = col16;
    a.low_mask = t->W - 1;
    GC_HIP_TRY(radix_pass(a, scratch, s));
    k_head_bits<<<grid_for(words, 4, 16384), 256, 0, s>>>(row, t->col, m, t->log2W, words,
                                                          bits, wcnt);
    GC_HIP_TRY(hipGetLastError());
  }
  GC_HIP_TRY(scan_queue(wcnt, wrow, words, slab.take<int32_t>(mem.p, i_wtile), s));
  k_block_rows<<<grid_for(B + 1, 256), 256, 0, s>>>(t->col, m, t->log2W, B, bits, wrow,
                                                    words, t->blk_rowoff);
  GC_HIP_TRY(hipGetLastError());
  int32_t P32 = 0;
  GC_HIP_TRY(hipMemcpyAsync(&P32, wrow + words, sizeof(int32_t), hipMemcpyDeviceToHost, s));
  GC_HIP_TRY(hipStreamSynchronize(s));
  const int64_t P = P32;
  t->P = P;
  const size_t Pn = static_cast<size_t>(std::max<int64_t>(P, 1));
  t->id_map = static_cast<int32_t*>(dev_alloc(sizeof(int32_t) * Pn, s));
  t->row_ptr = static_cast<int32_t*>(dev_alloc(sizeof(int32_t) * (Pn + 1), s));
  // padded for 4-wide reads, and past the pull's buffer resource (its range
  // check leaves out a store's scalar offset, at most 512 floats)
  if (!t->ranks_only) {
    t->partial = static_cast<float*>(dev_alloc(sizeof(float) * (Pn + 8 + 512), s));
    t->pmin = static_cast<int32_t*>(dev_alloc(sizeof(int32_t) * (Pn + 8), s));  // padded for 16-byte reads
    t->id16 = static_cast<uint16_t*>(dev_alloc(sizeof(uint16_t) * Pn, s));
    if (!t->partial || !t->pmin || !t->id16) return hipErrorOutOfMemory;
  }
  if (!t->id_map || !t->row_ptr) return hipErrorOutOfMemory;
  t->bytes = sizeof(int32_t) * ((R + 1 + (t->mk != t->k ? t->mR + 1 : 0)) * static_cast<int64_t>(B) + B + 1 + 4 * static_cast<int64_t>(Pn) + 1 +
                                mn * (t->weighted ? 2 : 1)) +
             static_cast<int64_t>(sizeof(uint16_t)) * P;
  k_local_rows<<<grid_for(heads ? head_words : words, 4, 16384), 256, 0, s>>>(
      row, m, words, bits, wrow, t->mk - 1, t->id_map, t->row_ptr, t->id16,
      heads, head_words);
  k_range_rows<<<grid_for(static_cast<int64_t>(R + 1) * B, 256, 65536), 256, 0, s>>>(t->id_map, t->blk_rowoff, B, R,
                                                                                     t->log2k, t->range_ptr);
  if (t->mk != t->k)
    k_range_rows<<<grid_for(static_cast<int64_t>(t->mR + 1) * B, 256, 65536), 256, 0, s>>>(
        t->id_map, t->blk_rowoff, B, t->mR, __builtin_ctz(t->mk), t->mrange);
  GC_HIP_TRY(hipGetLastError());
  if (!t->ranks_only) GC_HIP_TRY(build_tiles(t->row_ptr, P, m, pull_tile_arcs(), &t->tile_row, &t->n_tiles, s));
  if (pull_stream && 4 * (P + 8) < (int64_t(1) << 31)) {
    GC_HIP_TRY(build_lds_stream(t, s));
  } else if (pull_stream) {  // too many local rows for the pull's 32-bit byte offsets
    GC_HIP_TRY(hipStreamSynchronize(s));
    dev_free(t->col16, s);
    dev_free(t->heads, s);
    t->col16 = nullptr;
    t->heads = nullptr;
    t->m_pad = 0;
  }
  if (push_stream) GC_HIP_TRY(build_push_expand(t, s));
  GC_HIP_TRY(hipStreamSynchronize(s));  // the Buf is released on return
  if (t->ranks_only) {  // what only the building has read
    dev_free(t->col, s);
    dev_free(t->id_map, s);
    t->col = nullptr;
    t->id_map = nullptr;
    t->bytes -= static_cast<int64_t>(sizeof(int32_t)) * (static_cast<int64_t>(mn) + 3 * static_cast<int64_t>(Pn)) +
                static_cast<int64_t>(sizeof(uint16_t)) * P;
  }
  return hipSuccess;
}

}  // namespace gcx
