// Internal declarations shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <string>
#include <vector>

#include "graphcage.h"

// ---------------------------------------------------------------------------
// Handles

struct gc_graph_s {
  int32_t n = 0;
  int64_t m = 0;
  bool weighted = false;
  // out-arc CSR (row = source), as loaded
  int32_t* rowptr = nullptr;
  int32_t* colidx = nullptr;
  int32_t* w = nullptr;
  // transposed CSR (row = destination, columns ascending)
  int32_t* t_rowptr = nullptr;
  int32_t* t_colidx = nullptr;
  int32_t* t_w = nullptr;
  void* scratch = nullptr;  // holds the arrays from contrib to arc_pre (but not those allocated later)
  // PageRank scratch: contributions (two buffers for the fused plain pull),
  // push accumulators, FP64 dangling partials and totals
  float* contrib[2] = {nullptr, nullptr};
  double* sums = nullptr;     // push accumulators (FP64 atomics)
  int32_t* tile_row_in = nullptr;  // pull tiles over the transposed graph
  int32_t n_tiles_in = 0;
  int32_t longest_in = 0;  // largest in-degree (only for graphs that fit one work-group's LDS)
  // one slot per update work-group; [1]: kDangSlots slots, used in turn with
  // [0] by updates of at most that many work-groups
  double* dpart[2] = {nullptr, nullptr};
  double* dtotal = nullptr;   // [2] ping-pong dangling totals
  int32_t dpart_slots = 0;
  bool values_f32 = false;  // the weight arrays hold FP32 values (GC_VALUES_F32)
  // convergence mode (allocated by the first pagerank_converge call): FP64
  // partials of the L1 change per update work-group, results, and a second
  // FP32 iterate
  double* lpart = nullptr;
  double* ltotal = nullptr;     // the one-work-group form's change and count; [2]: number (int32) of the last call that ended
  uint32_t conv_calls = 0;      // calls so far, which number them
  float* rank_tmp = nullptr;
  // traversal scratch
  uint32_t* front = nullptr;  // status arrays (Section 3.3), one bit per vertex
  uint32_t* next = nullptr;
  int32_t* queue[2] = {nullptr, nullptr};
  uint32_t* visited = nullptr;  // BFS: bitmap of vertices with a final depth
  int32_t* mark = nullptr;      // SSSP push: round in which a vertex was queued
  // arc prefixes of the two queues ([n], [n+1]); BC: in-degrees of the level
  // order, and the prefixes of all its levels
  int32_t* arc_deg = nullptr;
  int32_t* arc_pre = nullptr;
  bool bits_clean = false;      // front and next are all zero
  uint32_t level_seq = 0;       // number of the last level (or convergence step) published to stats_host
  // betweenness centrality (allocated by the first bc_accumulate call):
  // path counts, two alternating arrays of (1 + delta) / sigma, BFS depths
  // and the vertices in level order of the current source
  double* bc_sigma = nullptr;
  double* bc_coef = nullptr;  // [2n]
  int32_t* bc_depth = nullptr;
  int32_t* bc_order = nullptr;
  int32_t* stats = nullptr;     // device counters read back once per level (kStatSlots)
  int32_t* stats_host = nullptr;  // pinned mirror
  int32_t clock_khz = 100000;   // rate of the device wall clock stamped into stats
  int64_t bytes = 0;
  // learned level scheduler attached to this graph (sched_attach)
  gc_sched sched = nullptr;
  gc_sched sched_kind[3] = {nullptr, nullptr, nullptr};  // per kind (BFS, SSSP, PageRank); null: sched
  std::vector<gc_tocab> sched_parts;
  int32_t pr_learned_action = -1;  // pagerank_learned's form for the attached network (-1: not chosen yet)
  // per-level record of the last traversal: action and wall time (ms)
  std::vector<int32_t> trace_action;
  std::vector<float> trace_ms;
};

// Row structure of 64 consecutive arcs of a stream-layout partition: bit i
// set when arc 64w + i is the first arc of its local row, the number of
// local rows that start before arc 64w (the index of the first row whose
// head lies at or after the word), and bit 0 of the next word.
struct alignas(16) gc_head_word {
  uint64_t bits;
  int32_t row;
  int32_t next;
};

struct gc_tocab_s {
  gc_graph g = nullptr;
  int32_t dir = GC_PULL;
  int32_t W = 0, log2W = 0, k = 0, log2k = 0, B = 0, R = 0;
  int32_t n_rows = 0, n_cols = 0;
  int64_t P = 0;
  int64_t m = 0;
  bool weighted = false;
  int32_t* blk_rowoff = nullptr;  // [B+1]
  int32_t* row_ptr = nullptr;     // [P+1]
  int32_t* id_map = nullptr;      // [P]
  int32_t* col = nullptr;         // [m]
  int32_t* w = nullptr;           // [m] or null
  int32_t* range_ptr = nullptr;   // [(R+1)*B], j-major
  // Ranges the merges of a GC_PULL partition work in: k, R and range_ptr, or
  // narrower ones where those are few (merge_width).
  int32_t mk = 0, mR = 0;
  int32_t* mrange = nullptr;      // [(mR+1)*B], j-major; range_ptr itself when mk = k
  float* partial = nullptr;       // [P] pull partial sums (Algorithm 4)
  uint16_t* id16 = nullptr;       // [P] id_map mod mk: position inside the merge range
  int32_t* tile_row = nullptr;    // [n_tiles+1] first local row of each pull tile
  int32_t n_tiles = 0;
  // Stream layout of an LDS-resident pull partition (W <= kLdsMaxWidth):
  // 16-bit columns inside the block, one head bit per arc marking the first
  // arc of every local row, and partial sums stored range-major (all blocks'
  // partials of merge range j contiguous) so the merge reads one stream.
  uint16_t* col16 = nullptr;      // [m_pad], zero past m
  gc_head_word* heads = nullptr;  // [m_pad/64 + 1], bits at and past m set
  int64_t m_pad = 0;              // multiple of wave_tile_arcs(), >= m + wave_tile_arcs()
  int2* seg = nullptr;            // [B][mR+1]: first local row of block b in range j, shift to range-major index
  int32_t* rstart = nullptr;      // [mR+1] range-major start of merge range j
  uint16_t* id16s = nullptr;      // [P] id16 in range-major order
  int32_t* chunk_beg = nullptr;   // [n_chunks] first local row (one buffer holds the five chunk arrays)
  int32_t* chunk_end = nullptr;   // [n_chunks] one past the last local row
  int32_t* chunk_blk = nullptr;   // [n_chunks] block
  int32_t* chunk_j0 = nullptr;    // [n_chunks] first merge range the chunk's rows fall in
  int32_t* chunk_ns = nullptr;    // [n_chunks] number of merge ranges the chunk's rows span
  int32_t n_chunks = 0;
  int32_t seg_max = 0;            // largest chunk_ns (sizes the work-group's LDS table)
  int32_t* pmin = nullptr;        // [P + 8] traversal partials (next flags / min; range-major for SSSP over the stream layout)
  double* bc_part = nullptr;      // [P] BC path-count partials (allocated on first use)
  float* val32 = nullptr;         // [m_pad] FP32 arc values in stream order (first valued SpMV)
  int32_t* w_pad = nullptr;       // [m_pad] integer weights in stream order, 0 past m (first SSSP over the stream layout)
  uint8_t* w8 = nullptr;          // [m_pad] the same as bytes, instead of w_pad when every weight lies in [0, 255]
  // GC_PUSH: the same arcs in blocks of the width that PageRank is fastest
  // over (push_width), which it takes instead; null: W itself.
  gc_tocab inner = nullptr;
  bool ranks_only = false;  // such a second layout: it keeps the expanded form alone
  // Expanded contributions of a GC_PUSH partition with block sums in LDS
  // (W <= kPushLdsMaxWidth, B <= kPushExpandMaxBlocks): the work-group that
  // updates source block s writes the new contribution of each local row
  // whose source lies in it (block b's rows [range_ptr[j0 B + b],
  // range_ptr[j1 B + b]) for the merge ranges j0 .. j1 of the block) to xc.
  uint16_t* xid16 = nullptr;      // [P + 8] source of each local row (source-major when xperm is set), offset inside its source block
  int32_t* xperm = nullptr;       // [P] short runs only: the local row at each source-major position
  int32_t* xstart = nullptr;      // [n_sblk + 1] short runs only: first source-major position of each source block
  float* xc = nullptr;            // [2P] contribution of each local row's source, two iterates in turn
  int32_t n_sblk = 0;             // source blocks (ceil(rows / W)); 0 without the expanded form
  // ... and its arcs as streams: destination offsets inside the block (16
  // bits) and one head bit per arc marking the first arc of each local row
  // (the head word layout of the pull's stream layout), padded to whole
  // 512-arc tiles.
  uint16_t* pcol16 = nullptr;     // [pm_pad], zero past m
  gc_head_word* pheads = nullptr; // [pm_pad/64 + 1], bits at and past m set
  int64_t pm_pad = 0;
  int64_t bytes = 0;
};

// ---------------------------------------------------------------------------
// Runtime helpers (gc_runtime.hip)

namespace gcx {

void set_error(const char* fmt, ...);
void* dev_alloc(size_t bytes, hipStream_t s);
void dev_free(void* p, hipStream_t s);

// RAII buffer from the library allocator
struct Buf {
  void* p = nullptr;
  hipStream_t s = nullptr;
  Buf() = default;
  Buf(size_t bytes, hipStream_t st) : p(dev_alloc(bytes, st)), s(st) {}
  ~Buf() { if (p) dev_free(p, s); }
  Buf(const Buf&) = delete;
  Buf& operator=(const Buf&) = delete;
  template <class T> T* as() const { return static_cast<T*>(p); }
  void* release() { void* q = p; p = nullptr; return q; }
};

// Several arrays in one buffer of the library allocator (an allocation goes
// through the caller's hook): reserve() every array, allocate once, take().
struct Slab {
  std::vector<size_t> at;
  size_t total = 0;
  size_t reserve(size_t bytes) {
    at.push_back(total);
    total += (std::max<size_t>(bytes, 1) + 255) & ~size_t(255);
    return at.size() - 1;
  }
  template <class T> T* take(void* base, size_t i) const {
    return reinterpret_cast<T*>(static_cast<char*>(base) + at[i]);
  }
};

// ---- construction kernels (gc_build.hip) ----
// Device-side structural check of an out-arc CSR; *bad_out != 0 if broken.
hipError_t check_csr(int32_t n, int64_t m, const int32_t* rowptr, const int32_t* colidx, int32_t* bad_out,
                     hipStream_t s);
// Exclusive scan of int32 `in[0..n)` into `out[0..n]` (out[n] = total).
hipError_t scan_exclusive(const int32_t* in, int32_t* out, int64_t n, hipStream_t s);
// Transposed CSR with rows sorted by column; weights carried (w may be null).
hipError_t build_transpose(int32_t n, int64_t m, const int32_t* rowptr, const int32_t* colidx,
                           const int32_t* w, int32_t* t_rowptr, int32_t* t_colidx, int32_t* t_w,
                           hipStream_t s);
// Pull tile table: tile i owns the rows whose first arc lies in
// [i*tile_arcs, (i+1)*tile_arcs); out[i] = first such row, out[n_tiles] = rows.
// The pinned word `longest`, where given, gets the longest row's arcs (found
// by one work-group).
hipError_t build_tiles(const int32_t* row_ptr, int64_t rows, int64_t arcs, int32_t tile_arcs,
                       int32_t** out, int32_t* n_tiles, hipStream_t s, int32_t* longest = nullptr);
// TOCAB partition of CSR A (see tocab_partition); fills t's arrays.
hipError_t build_partition(gc_tocab t, const int32_t* a_rowptr, const int32_t* a_col,
                           const int32_t* a_w, hipStream_t s);

// ---- PageRank (gc_pagerank.hip) ----
int32_t pull_tile_arcs();
int32_t wave_tile_arcs();
// Largest block width whose FP32 contribution slice is staged in LDS.
constexpr int32_t kLdsMaxWidth = 1 << 15;
// Largest block width of a TOCAB push whose block sums (FP64) sit in LDS.
constexpr int32_t kPushLdsMaxWidth = 1 << 14;
// Width of the blocks that the push with block sums in LDS runs over:
// kPushLdsMaxWidth, halved until there are kPushBlocks of them (or they are
// 1024 wide), one work-group each; wider blocks hold a source's arcs in fewer
// rows. PageRank, 20 iterations at 2^14, 13, 12, 11, 10: R-MAT of 16 arcs and
// 20,000 vertices 1420, 954, 592, 477, 370 us; 300,007: 1690, 1073, 812, 698,
// 725; 10^6: 2398, 1884, 1652, 2043, 2654; 3 M: 3182, 3799, 4334, 5062, 7938.
// W itself where the width would be twice that: 15 % of a run, and a second
// layout to build (a grid of 2 M vertices at 2^12 with its transpose 1457 us,
// 2144 with one).
constexpr int32_t kPushBlocks = 128;
inline int32_t push_width(int32_t n, int32_t W) {
  int32_t w = kPushLdsMaxWidth;
  while (w > 1024 && (static_cast<int64_t>(n) + w - 1) / w < kPushBlocks) w /= 2;
  return W > kPushLdsMaxWidth || w == 2 * W ? W : w;
}
// Most blocks of a push partition with expanded contributions (a work-group
// keeps two run bounds per block in LDS).
constexpr int32_t kPushExpandMaxBlocks = 4096;
// Whether a push partition of k-wide ranges has the expanded form: block sums
// in LDS, 16-bit offsets, and arc indices that fit 32 bits past the padded end.
inline bool push_expands(int32_t n, int64_t m, int32_t W, int32_t k) {
  return W <= kPushLdsMaxWidth && k <= W && m > 0 && m + 1024 < INT32_MAX &&
         (static_cast<int64_t>(n) + W - 1) / W <= kPushExpandMaxBlocks;
}
// Average run length (local rows per (source block, block) pair) from which
// the expanded push walks its runs in place rather than through a
// source-major list.
constexpr int64_t kPushLongRun = 128;
// Offset of the second buffer of expanded contributions (16-byte aligned).
inline int64_t push_xc_stride(int64_t P) { return (std::max<int64_t>(P, 1) + 3) & ~int64_t(3); }
// Least arcs per chunk of an LDS-resident block (one work-group each): a
// 512-arc tile for every other wave (half of that, and twice, measured the
// same or up to 5 % slower from 10^5 to 10^6 arcs).
constexpr int32_t kLdsChunkArcs = 16 * 256;
// LDS bytes one work-group of the LDS-resident pull may use: half a CU's
// 160 KB (two resident work-groups) for slices up to 2^13 floats, all of it
// for wider ones.
inline int32_t lds_budget(int32_t W) { return W >= (1 << 14) ? 160 * 1024 - 512 : 80 * 1024 - 512; }
// LDS bytes of the pull's per-wave output staging (16 waves x (384 rows +
// 16 spare slots) floats).
constexpr int32_t kLdsStageBytes = 16 * (384 + 16) * 4;
// Largest range table (entries) that fits beside a W-float slice and the
// staging (with 8 entries of padding).
inline int32_t lds_seg_cap(int32_t W) { return ((lds_budget(W) - 4 * W - kLdsStageBytes) / 4 - 8) / 2; }
// ---- SpMV (gc_spmv.hip; the stream-layout form in gc_pagerank.hip) ----
hipError_t spmv_run(gc_graph g, gc_tocab t, const float* x, float* y, hipStream_t s);
hipError_t spmv_stream(gc_graph g, gc_tocab t, const float* x, const float* vals, float* y, hipStream_t s);
hipError_t stream_values(gc_graph g, gc_tocab t, hipStream_t s);

// Convergence mode of pagerank_run: iterate until the L1 change between
// consecutive iterates is at most tol (or max_iters); iters / delta report
// the iterations run and the last change.
struct Converge {
  double tol = 0.0;
  int32_t max_iters = 0;
  int32_t iters = 0;
  double delta = 0.0;
};
// Device buffers an iteration writes besides rank_out: contributions (two,
// used in turn by the forms that read one while writing the next), FP64
// push sums (n), FP64 dangling partials (one per update work-group, at most
// the graph's dpart_slots; a second buffer of kDangSlots, or null: every
// iteration's partials are then reduced by a kernel of their own) and their
// two totals, and the pull partition's partial sums (P + 8). By default the graph's and the partition's own.
constexpr int32_t kDangSlots = 1024;
struct PrBuffers {
  float* contrib[2];
  double* sums;
  double* dpart[2];
  double* dtotal;
  float* partial;
};
hipError_t pagerank_run(gc_graph g, gc_tocab t, int32_t dir, float damping, int32_t dangling,
                        const float* rank_in, float* rank_out, int32_t iters, hipStream_t s,
                        Converge* cv = nullptr, int32_t ladder = -1, const PrBuffers* bufs = nullptr);

// Whether a pull partition has the stream layout: a slice that fits the LDS, a
// range table of at most 2^25 entries (of a block, the whole of it goes
// through the host once), and arc indices that fit 32 bits past the padded end.
inline bool pull_streams(int32_t n, int64_t m, int32_t W, int32_t k) {
  auto parts = [&](int32_t w) { return (static_cast<int64_t>(n) + w - 1) / w; };
  return W <= kLdsMaxWidth && parts(W) * (parts(k) + 1) <= (int64_t(1) << 25) && m + 1024 < INT32_MAX;
}

// Width of the ranges that the merges of a pull partition work in, since a
// merge gives each range one work-group: k, halved as follows while the range
// table stays below an eighth of the arcs.
// Stream layout: until there are 128 (or they are 256 wide). PageRank, 20
// iterations, with ranges of k, with 64, 128 and 256: 10^6 vertices of 16
// arcs, k = 2^14: 1461, 1081, 887, 894 us; 300,007 of 16, 2^14: 657, 386, 361,
// 385; of 4, 2^12: 312, 312, 296, 331 (a tile of the pull that meets more
// ranges takes longer).
// Wider blocks: until they are 2048 wide, and on to 1024 while there are
// fewer than 512. The merge of 256 threads holds a range's FP64 sums in LDS,
// so 2048 of them let a CU run its work-groups: 2.5 M vertices of 16 arcs with
// k = 2^13 5552 us, 4815 with 4096, 4501 with 2048, 4557 with 1024; 10^6 of 16,
// k = 2^14: 3381, 2119, 1940, 1861.
// (The batched form, whose ranges are 1024 wide, takes blocks of at most 2^15
// without the stream layout as well: they are left at k.)
inline int32_t merge_width(int32_t n, int64_t m, int32_t W, int32_t k) {
  auto parts = [&](int32_t w) { return (static_cast<int64_t>(n) + w - 1) / w; };
  const bool stream = pull_streams(n, m, W, k);
  auto wanted = [&] { return stream ? k > 256 && parts(k) < 128 : k > 2048 || (k > 1024 && parts(k) < 512); };
  while (wanted() && parts(W) * (parts(k / 2) + 1) <= m / 8 + 65536) k /= 2;
  return k;
}

// Small graphs (gc_pr_small.hip): whether a graph fits the one-work-group
// form's LDS, whether a call in `form` is faster there, and that form of
// pagerank_run. (Push over a partition as asked for, or over its second
// layout.)
enum class PrForm { kPull, kPush, kTocabPull, kTocabPush, kTocabPushInner };
bool pr_small_fits(int64_t n, int64_t m, bool conv);
bool pr_small_pays(gc_graph g, PrForm form, bool conv, int32_t iters);
hipError_t pr_small_run(gc_graph g, float damping, int32_t dangling, const float* rank_in, float* rank_out,
                        int32_t iters, hipStream_t s, Converge* cv);

// PageRank's working-set action among 0 push, 1 pull, 2 + i TOCAB over parts[i].
int32_t pagerank_fallback_action(const gc_tocab* parts, int32_t n_parts);
// Scheduler training rows for PageRank (see sched_collect, kind 2).
hipError_t collect_pagerank(gc_graph g, gc_tocab* parts, int32_t n_parts, int32_t n_rows, float* features,
                            float* times, int32_t max_rows, int32_t* rows, hipStream_t s);

// ---- autotuner (gc_autotune.hip) ----
// Candidate widths start at max(2^12, min_W).
hipError_t autotune(gc_graph g, int32_t dir, int32_t min_W, int32_t* W_out, int32_t* k_out, float* ms_out,
                    hipStream_t s);

// ---- traversal (gc_traverse.hip) ----
hipError_t bfs_run(gc_graph g, gc_tocab t, int32_t source, int32_t* depth, int32_t* levels,
                   uint32_t policy, hipStream_t s);
hipError_t sssp_run(gc_graph g, gc_tocab t, int32_t source, int32_t* dist, int32_t* rounds,
                    uint32_t policy, hipStream_t s, bool* overflow);
hipError_t bc_run(gc_graph g, gc_tocab t, const int32_t* sources, int32_t n_src, double* bc, uint32_t policy,
                  hipStream_t s);
hipError_t collect(gc_graph g, gc_tocab* parts, int32_t n_parts, bool bfs, const int32_t* sources, int32_t n_src,
                   float* features, float* times, int32_t max_rows, int32_t* rows, hipStream_t s);
void sched_features(int64_t n, int64_t m, int64_t n_f, int64_t m_f, int32_t level, double prior_ms,
                    int64_t prior_arcs, float* f);

// Waits until the pinned word holds `seq`, which a kernel queued on s writes:
// it spins for as long as short work takes (a stream synchronisation costs
// more than such kernels), then leaves the waiting to the runtime.
hipError_t wait_mirror(const int32_t* word, int32_t seq, hipStream_t s);

// Waits until everything queued on s has run: a kernel behind it writes the
// next number to g's mirror. At the end of a BFS of 738 us (a grid of 4 M vertices)
// this took 4 us, a stream synchronisation 36.
hipError_t wait_queued(gc_graph g, hipStream_t s);

// The scheduler's 6 inputs for a level (the same arithmetic on the host and
// in the device-side decision): log1p(frontier vertices), log1p(frontier
// out-arcs), log1p(m / n), log2(ceil(n / 2^18) + 1), level / 16, and
// log1p(the previous level's time per out-arc of its frontier, in ns), 0
// before the first level.
__host__ __device__ inline void level_features(int64_t n, int64_t m, int64_t n_f, int64_t m_f, int32_t level,
                                               double prior_ms, int64_t prior_arcs, float* f) {
  f[0] = static_cast<float>(log1p(static_cast<double>(n_f)));
  f[1] = static_cast<float>(log1p(static_cast<double>(m_f)));
  f[2] = static_cast<float>(log1p(static_cast<double>(m) / static_cast<double>(n > 1 ? n : 1)));
  f[3] = static_cast<float>(log2(static_cast<double>((n + (1 << 18) - 1) >> 18) + 1.0));
  f[4] = static_cast<float>(level) / 16.0f;
  f[5] = static_cast<float>(log1p(prior_ms * 1e6 / static_cast<double>(prior_arcs > 1 ? prior_arcs : 1)));
}

// Device counters of one traversal level (int32 slots), written once per
// level to a pinned host mirror by the level's last kernel.
constexpr int kStatArcs = 0;      // out-arcs of the next frontier, with
constexpr int kStatQLen = 1;      // its vertices: one 64-bit word (below 2^31 each)
constexpr int kStatOverflow = 2;  // SSSP: a path length reached INT32_MAX
constexpr int kStatSeq = 3;       // host mirror: the level whose counters it holds
constexpr int kStatT0 = 4;        // device wall clock at the level's start (64-bit)
constexpr int kStatT1 = 6;        // device wall clock when its relaxation kernels have finished (64-bit)
constexpr int kStatChoice = 8;    // learned scheduler: action for the next level (-1: no finite output)
constexpr int kStatInDegLo = 10;  // in-arcs of the next frontier (64-bit: lo, hi)
constexpr int kStatBuild = 12;    // the packed count of a queue built from status bits (64-bit)
constexpr int kStatOut = 16;      // learned scheduler: its K outputs (FP32 bit patterns)
constexpr int kStatSlots = kStatOut + GC_SCHED_HIDDEN;

// Learned policy: the working-set rule's choice is kept unless the network
// predicts its own pick faster by more than this margin (its outputs are
// log times relative to the fastest action, so 0.3 is about 35 %: the
// network overrides the rule only where it expects a clear win).
constexpr float kLearnedGate = 0.3f;

// ---- scheduler network (gc_sched.hip) ----
int32_t sched_actions(gc_sched m);
// The network deciding for one kind of work on g (0 BFS, 1 SSSP, 2
// PageRank): the one attached for that kind, else the shared one (or null).
inline gc_sched sched_for(gc_graph g, int kind) { return g->sched_kind[kind] ? g->sched_kind[kind] : g->sched; }
// Device pointer to the network's parameters (layout in gc_mlp.h).
const float* sched_params(gc_sched m);
// Device pointer to the training range of its inputs (null before training).
const float* sched_range(gc_sched m);
// Decision from host features: action (-1 when an output is not finite)
// and, when out is given, the K outputs. Synchronises s.
hipError_t sched_decide(gc_sched m, const float* features, hipStream_t s, int32_t* action, float* out = nullptr);

// Records HIP events around the launches made in its scope while
// profiling is on (gc_profile); a no-op otherwise.
class ProfScope {
 public:
  ProfScope(const char* name, hipStream_t s);
  ~ProfScope();
  ProfScope(const ProfScope&) = delete;
  ProfScope& operator=(const ProfScope&) = delete;

 private:
  const char* name_;
  hipStream_t s_;
  hipEvent_t start_ = nullptr, stop_ = nullptr;
};

}  // namespace gcx

#define GC_HIP_TRY(expr)                    \
  do {                                      \
    hipError_t e_ = (expr);                 \
    if (e_ != hipSuccess) return e_;        \
  } while (0)
