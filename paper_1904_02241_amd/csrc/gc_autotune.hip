// Block-width autotuner: successive halving over candidate (W, k) pairs,
// each timed on PageRank iterations of the graph itself with HIP events.
// The paper picks its subgraph size by a sweep (Section 4.3); here the sweep
// runs per graph and its result is cached for the process.

#include <algorithm>
#include <cstring>
#include <map>
#include <mutex>
#include <tuple>
#include <vector>

#include "gc_internal.h"

namespace {

struct Candidate {
  int32_t W, k;
  double ms = 0.0;  // best time per iteration seen
};

using Key = std::tuple<int32_t, int64_t, int32_t, uint64_t, int32_t>;
std::mutex g_mu;
std::map<Key, Candidate> g_cache;

bool allowed(int64_t n, int32_t W, int32_t k) {
  const int64_t B = (n + W - 1) / W, R = (n + k - 1) / k;
  return B <= 32768 && B * (R + 1) <= (int64_t(1) << 28);
}

// The block width that PageRank runs over with a partition of width W: a
// push partition's own, or its second layout's.
int32_t run_width(gc_graph g, int32_t dir, int32_t W) {
  if (dir == GC_PULL) return W;
  const int32_t w = gcx::push_width(g->n, W);
  return gcx::push_expands(g->n, g->m, w, w) ? w : W;
}

// Whether every partition of g runs as one work-group, which reads none.
bool one_group(gc_graph g, int32_t dir) {
  return gcx::pr_small_pays(g, dir == GC_PULL ? gcx::PrForm::kTocabPull : gcx::PrForm::kTocabPushInner, false, 20);
}

// Whether the partitions of width W with merge ranges k and j run alike.
bool same_ranges(gc_graph g, int32_t dir, int32_t W, int32_t k, int32_t j) {
  if (one_group(g, dir)) return true;
  if (dir == GC_PUSH) return run_width(g, dir, W) != W;
  return gcx::merge_width(g->n, g->m, W, k) == gcx::merge_width(g->n, g->m, W, j);
}

// Leaves one candidate of those that run alike (timing them against each
// other would pick by noise): the one whose own blocks are those run over,
// which needs no second layout, else the first.
void leave_one_of_each(gc_graph g, int32_t dir, std::vector<Candidate>& cand) {
  std::vector<Candidate> left;
  for (const Candidate& c : cand) {
    auto alike = std::find_if(left.begin(), left.end(), [&](const Candidate& o) {
      return one_group(g, dir) || run_width(g, dir, o.W) == run_width(g, dir, c.W);
    });
    if (alike == left.end()) left.push_back(c);
    else if (!one_group(g, dir) && run_width(g, dir, c.W) == c.W) *alike = c;
  }
  cand.swap(left);
}

// Times `iters` PageRank iterations on partition t (after one warm-up).
hipError_t time_iters(gc_graph g, gc_tocab t, int32_t iters, float* ra, float* rb, hipStream_t s, double* ms) {
  GC_HIP_TRY(gcx::pagerank_run(g, t, t->dir, 0.85f, GC_DANGLING_UNIFORM, ra, rb, 1, s));
  hipEvent_t e0, e1;
  GC_HIP_TRY(hipEventCreate(&e0));
  GC_HIP_TRY(hipEventCreate(&e1));
  hipError_t e = hipEventRecord(e0, s);
  if (e == hipSuccess) e = gcx::pagerank_run(g, t, t->dir, 0.85f, GC_DANGLING_UNIFORM, rb, ra, iters, s);
  if (e == hipSuccess) e = hipEventRecord(e1, s);
  if (e == hipSuccess) e = hipEventSynchronize(e1);
  float f = 0.0f;
  if (e == hipSuccess) e = hipEventElapsedTime(&f, e0, e1);
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  *ms = static_cast<double>(f) / iters;
  return e;
}

}  // namespace

namespace gcx {

hipError_t autotune(gc_graph g, int32_t dir, int32_t min_W, int32_t* W_out, int32_t* k_out, float* ms_out,
                    hipStream_t s) {
  // graph signature: sizes plus a hash of sampled offsets
  std::vector<int32_t> sample(65);
  const int64_t n = g->n;
  for (int i = 0; i <= 64; ++i) {
    const int64_t v = n * i / 64;
    GC_HIP_TRY(hipMemcpyAsync(&sample[i], g->rowptr + v, sizeof(int32_t), hipMemcpyDeviceToHost, s));
  }
  GC_HIP_TRY(hipStreamSynchronize(s));
  uint64_t h = 1469598103934665603ull;  // FNV-1a over the sample
  for (int32_t x : sample) {
    for (int b = 0; b < 4; ++b) {
      h ^= static_cast<uint8_t>(x >> (8 * b));
      h *= 1099511628211ull;
    }
  }
  const Key key{g->n, g->m, dir, h, min_W};
  {
    std::lock_guard<std::mutex> lk(g_mu);
    auto it = g_cache.find(key);
    if (it != g_cache.end()) {
      *W_out = it->second.W;
      *k_out = it->second.k;
      *ms_out = static_cast<float>(it->second.ms);
      return hipSuccess;
    }
  }
  int32_t top = 1 << 10;
  while (top < n && top < (1 << 22)) top <<= 1;
  std::vector<Candidate> cand;
  const int32_t lo = std::max(1 << 12, min_W);
  for (int32_t W = lo; W <= std::max(top, lo); W <<= 1)
    if (allowed(n, W, 4096)) cand.push_back({W, 4096});
  if (cand.empty()) cand.push_back({std::max(1 << 22, lo), 4096});
  leave_one_of_each(g, dir, cand);
  Buf ra(sizeof(float) * n, s), rb(sizeof(float) * n, s);
  if (!ra.p || !rb.p) return hipErrorOutOfMemory;
  // uniform start vector: any vector gives the same amount of work
  {
    std::vector<float> init(static_cast<size_t>(n), 1.0f / static_cast<float>(n));
    GC_HIP_TRY(hipMemcpyAsync(ra.p, init.data(), sizeof(float) * n, hipMemcpyHostToDevice, s));
    GC_HIP_TRY(hipStreamSynchronize(s));
  }
  auto evaluate = [&](Candidate& c, int32_t iters) -> hipError_t {
    gc_tocab t = nullptr;
    if (tocab_partition(g, dir, c.W, c.k, s, &t) != GC_OK) return hipErrorInvalidValue;
    double ms = 0.0;
    const hipError_t e = time_iters(g, t, iters, ra.as<float>(), rb.as<float>(), s, &ms);
    (void)hipStreamSynchronize(s);
    tocab_free(t);
    if (e == hipSuccess) c.ms = ms;
    return e;
  };
  // successive halving on W, then the merge range for the winner
  int32_t iters = 2;
  while (cand.size() > 1) {
    for (auto& c : cand) GC_HIP_TRY(evaluate(c, iters));
    std::sort(cand.begin(), cand.end(), [](const Candidate& a, const Candidate& b) { return a.ms < b.ms; });
    cand.resize((cand.size() + 1) / 2);
    iters *= 2;
  }
  Candidate best = cand[0];
  if (best.ms == 0.0) GC_HIP_TRY(evaluate(best, iters));
  for (int32_t k : {2048, 8192, 16384}) {
    if (!allowed(n, best.W, k) || same_ranges(g, dir, best.W, k, best.k)) continue;
    Candidate c{best.W, k};
    GC_HIP_TRY(evaluate(c, iters));
    Candidate b2 = best;
    GC_HIP_TRY(evaluate(b2, iters));  // re-time the incumbent under the same conditions
    best = (c.ms < b2.ms) ? c : b2;
  }
  {
    std::lock_guard<std::mutex> lk(g_mu);
    g_cache[key] = best;
  }
  *W_out = best.W;
  *k_out = best.k;
  *ms_out = static_cast<float>(best.ms);
  return hipSuccess;
}

}  // namespace gcx
