// The tile reduction of the stream layout, shared by the LDS-resident pulls:
// a wave takes 512 consecutive arcs of a block (8 per lane, already gathered
// from the block's slice in LDS), joins the arcs of each row, and stores the
// finished rows at their range-major index.
#pragma once

#include <hip/hip_runtime.h>

#include <climits>
#include <cstdint>
#include <type_traits>

#include "gc_device.h"

namespace gcs {

using gcd::kWave;
using gcd::wave_lds_fence;

constexpr int kLdsThreads = 1024;
constexpr int kLdsWaves = kLdsThreads / kWave;
constexpr int kArcsPerLane = 8;
constexpr int kWaveTile = kArcsPerLane * kWave;  // 512 arcs, 8 head words
constexpr int kStageRows = 384;                  // staged row sums per wave in the first pass
constexpr int kTileRowsMax = 512;                // rows one tile can complete
constexpr int kStageSpare = 16;                  // spare slots per wave for elements that end no staged row
static_assert(kStageRows % kWave == 0 && (kTileRowsMax - kStageRows) % kWave == 0 &&
              kTileRowsMax - kStageRows <= kStageRows, "staging passes of whole store instructions");

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint64_t word_bits(const u32x4& w) {
  return static_cast<uint64_t>(w[0]) | (static_cast<uint64_t>(w[1]) << 32);
}

// Merge-range index of local row r, searching forward from j: sb[j] is the
// first row of the chunk's j-th merge range (ascending; sb[ns] lies past
// the chunk and sb[ns+1..ns+3] hold INT32_MAX), four entries per step.
__device__ __forceinline__ int32_t seek_range(const int32_t* sb, int32_t j, int32_t r) {
  for (;;) {
    const int32_t adv = (sb[j + 1] <= r) + (sb[j + 2] <= r) + (sb[j + 3] <= r) + (sb[j + 4] <= r);
    j += adv;
    if (adv < 4) return j;
  }
}
constexpr int kSegPad = 4;  // LDS entries past the position table read by seek_range and the cursor

// Buffer resource over the partial sums: a store whose offset lies past the
// resource's size is dropped by the hardware, which lets every lane issue
// the same number of stores per tile (no branch around a store, so the
// compiler can count outstanding memory operations and keep the prefetched
// tiles in flight while the stores drain).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t partial_rsrc(void* partial, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(partial, 0, static_cast<int>(bytes), 0x00020000);
}

constexpr int kStoresPerTile = 6;  // stores of the first staging pass, issued by every tile

// kStoresPerTile stores the hardware drops (offsets past any resource size
// below 2^31, distinct so that none is a dead store of another).
__device__ __forceinline__ void drop_stores(__amdgpu_buffer_rsrc_t out) {
#pragma unroll
  for (int i = 0; i < kStoresPerTile; ++i) __builtin_amdgcn_raw_buffer_store_b32(0u, out, 0x80000000u + 4u * i, 0, 0);
}

// Lanes of the wave selected by a mask held in scalar registers.
__device__ __forceinline__ bool lane_in(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }


// What a tile's rows are reduced with: FP32 sums carried from tile to tile in
// FP64 (PageRank, SpMV), or maxima of unsigned 32-bit values (the traversals,
// whose candidates are kept as INT32_MAX - distance so that 0 is "none").
// Both have all-zero bits as their identity, so a value is left out by
// masking it.
struct SumOp {
  using T = float;
  using Carry = double;
  static __device__ __forceinline__ uint32_t bits(T x) { return __float_as_uint(x); }
  static __device__ __forceinline__ T from(uint32_t b) { return __uint_as_float(b); }
  static __device__ __forceinline__ T join(T a, T b) { return a + b; }
  // the value flowing into a lane, with what the earlier tiles carry
  static __device__ __forceinline__ T open(T c, Carry o) { return static_cast<T>(static_cast<Carry>(c) + o); }
  static __device__ __forceinline__ Carry tail(T t, Carry o) { return static_cast<Carry>(t) + o; }
};
struct MaxOp {
  using T = uint32_t;
  using Carry = uint32_t;
  static __device__ __forceinline__ uint32_t bits(T x) { return x; }
  static __device__ __forceinline__ T from(uint32_t b) { return b; }
  static __device__ __forceinline__ T join(T a, T b) { return max(a, b); }
  static __device__ __forceinline__ T open(T c, Carry o) { return max(c, o); }
  static __device__ __forceinline__ Carry tail(T t, Carry o) { return max(t, o); }
};

// Value a DPP control moves into each lane (lanes with no source get 0).
template <class Op, int kCtrl, int kRowMask>
__device__ __forceinline__ typename Op::T dpp_moved(typename Op::T a) {
  return Op::from(static_cast<uint32_t>(
      __builtin_amdgcn_update_dpp(0, static_cast<int>(Op::bits(a)), kCtrl, kRowMask, 0xF, false)));
}

// One step of a wave-wide segmented inclusive scan: a lane that has met no
// head yet within the reach of the steps so far (not in F) joins the value
// the DPP control moves in. F itself is kept as a lane mask in scalar
// registers and widened by the caller after each step.
template <class Op, int kCtrl, int kRowMask>
__device__ __forceinline__ void seg_scan_step(typename Op::T& A, uint64_t F) {
  const typename Op::T s = Op::join(A, dpp_moved<Op, kCtrl, kRowMask>(A));
  A = lane_in(F) ? A : s;
}

// DPP controls (gfx9): shift right by n lanes inside each row of 16, copy
// lane 15 / 31 into the following row(s), shift right by one lane across
// the whole wave.
constexpr int kDppRowShr1 = 0x111, kDppRowShr2 = 0x112, kDppRowShr4 = 0x114, kDppRowShr8 = 0x118;
constexpr int kDppRowBcast15 = 0x142, kDppRowBcast31 = 0x143, kDppWaveShr1 = 0x138;

// What a wave carries from one tile of its range to the next: the running
// sum of the row still open at the tile's end (when that row is one the wave
// must write), a window of 64 entries of the chunk's position table held one
// per lane, and a cursor into it with the next boundaries and shifts in
// scalar registers.
template <class Op>
struct PullCarry {
  typename Op::Carry open = 0;
  int32_t open_row = -1;           // >= 0 when the wave owes that row's sum
  int32_t jw = 0;                  // first table entry of the window
  int32_t sbw, sdw;                // lane l: sb[jw + l], sd[jw + l] (past the table: its last spare)
  int32_t jc = 0;                  // sb[jc] <= every row the wave still writes; jc - jw <= 60
  int32_t b1, b2, b3, d0, d1, d2;  // sb[jc+1..jc+3], sd[jc..jc+2]
};

template <class Op>
__device__ __forceinline__ void load_window(const int32_t* sb, const int32_t* sd, int32_t ns, int lane,
                                            PullCarry<Op>& c) {
  const int32_t i = min(c.jw + lane, ns + kSegPad - 1);
  c.sbw = sb[i];
  c.sdw = sd[i];
}

template <class Op>
__device__ __forceinline__ void cursor_from_window(PullCarry<Op>& c) {
  const int32_t o = c.jc - c.jw;
  c.b1 = __builtin_amdgcn_readlane(c.sbw, o + 1);
  c.b2 = __builtin_amdgcn_readlane(c.sbw, o + 2);
  c.b3 = __builtin_amdgcn_readlane(c.sbw, o + 3);
  c.d0 = __builtin_amdgcn_readlane(c.sdw, o);
  c.d1 = __builtin_amdgcn_readlane(c.sdw, o + 1);
  c.d2 = __builtin_amdgcn_readlane(c.sdw, o + 2);
}

// Moves the cursor to the range holding row r (r >= sb[jc]): the count of
// window entries at or below r, restarting the window when the cursor and
// the three boundaries after it would not fit in it.
template <class Op>
__device__ __forceinline__ void seek_cursor(const int32_t* sb, const int32_t* sd, int32_t ns, int lane, int32_t r,
                                            PullCarry<Op>& c) {
  for (;;) {
    const int32_t cnt = __popcll(__ballot(c.sbw <= r));  // >= 1: sb[jw] <= r
    if (cnt <= kWave - 3) {
      c.jc = c.jw + cnt - 1;
      break;
    }
    c.jw += cnt - 1;  // advances by at least 61; entries past the table are INT32_MAX, so this ends
    load_window(sb, sd, ns, lane, c);
  }
  cursor_from_window(c);
}

constexpr uint32_t kPushOut = 1u << 23;  // moves the staging slot of an arc that ends no row past every pass

// Byte offsets (past the store's base) of the stores k < nk of a staging
// pass: store k holds rows rs + i, i = lo + 64k + lane, written to index
// i + D0 / D1 / D2 below / from / past the range boundaries i1 and i2
// (kTwo: i2 lies among the rows written), dropped from iz on. The lane is
// compared with scalar thresholds; the store's base offset 4(lo + 64k)
// travels in the scalar offset operand, which the hardware leaves out of
// its range check, so a dropped lane's offset alone is past the resource.
template <bool kTwo>
__device__ __forceinline__ void row_offsets(uint32_t (&off)[kStageRows / kWave], int nk, int lane, int32_t lo,
                                            int32_t i1, int32_t i2, int32_t iz, int32_t D0, int32_t D1, int32_t D2) {
  constexpr int32_t kDropIndex = 1 << 29;  // (lane + kDropIndex) * 4 >= 2^31
#pragma unroll
  for (int k = 0; k < kStageRows / kWave; ++k) {
    if (k < nk) {
      const int32_t base = lo + k * kWave;
      const bool p1 = lane >= i1 - base, pz = lane >= iz - base;
      int32_t d = p1 ? D1 : D0;
      if (kTwo) d = lane >= i2 - base ? D2 : d;
      d = pz ? kDropIndex : d;
      off[k] = static_cast<uint32_t>(lane + d) << 2;
    }
  }
}

// The same for a tile whose rows lie in more than three merge ranges (blocks
// whose arcs concentrate near the diagonal leave a few rows in each of the
// other ranges: dozens of ranges per tile): every row's range is searched
// in the position table between entry jc and hi, the last one at or below
// row re - 1, all of a lane's rows together. Rows from re on are dropped.
__device__ __forceinline__ void row_offsets_search(uint32_t (&off)[kStageRows / kWave], int nk, int lane, int32_t lo,
                                                   int32_t rs, int32_t re, const int32_t* sb, const int32_t* sd,
                                                   int32_t jc, int32_t hi) {
  constexpr int kN = kStageRows / kWave;
  constexpr int32_t kDropIndex = 1 << 29;
  int32_t j[kN];
#pragma unroll
  for (int k = 0; k < kN; ++k) j[k] = jc;
  const int32_t span = hi - jc;  // >= 1
  for (int32_t step = 1 << (31 - __builtin_clz(span)); step > 0; step >>= 1) {  // uniform
#pragma unroll
    for (int k = 0; k < kN; ++k) {
      if (k < nk) {
        const int32_t jj = min(j[k] + step, hi);
        j[k] = sb[jj] <= rs + lo + k * kWave + lane ? jj : j[k];
      }
    }
  }
#pragma unroll
  for (int k = 0; k < kN; ++k) {
    if (k < nk) {
      const int32_t row = rs + lo + k * kWave + lane;
      const int32_t d = row < re ? rs + sd[j[k]] : kDropIndex;
      off[k] = static_cast<uint32_t>(lane + d) << 2;
    }
  }
}

// Reduces one tile: hw is the head word of the lane's arcs, x their values.
template <class Op>
__device__ __forceinline__ void reduce_wave_tile(const u32x4& hw, const typename Op::T (&x)[kArcsPerLane], int lane,
                                                 const int32_t* sb, const int32_t* sd, int32_t ns, int32_t r0,
                                                 int32_t r1, PullCarry<Op>& cr, __amdgpu_buffer_rsrc_t out,
                                                 typename Op::T* stage) {
  using T = typename Op::T;
  const uint32_t wlo = hw[0], whi = hw[1];
  const int32_t wrow = static_cast<int32_t>(hw[2]);
  const int32_t ta = __builtin_amdgcn_readfirstlane(wrow);
  const int32_t tz = __builtin_amdgcn_readlane(wrow + __popc(wlo) + __popc(whi), kWave - 1);
  const uint32_t next_head = __builtin_amdgcn_readlane(static_cast<int32_t>(hw[3]), kWave - 1) & 1u;
  // rows the wave writes from this tile: those whose head is here and that
  // belong to the chunk, and the row left open by the previous tile
  const int32_t rz = min(tz, r1);
  const int32_t rmin = cr.open_row >= 0 ? cr.open_row : max(ta, r0);
  if (rmin < rz && rmin >= cr.b1) seek_cursor(sb, sd, ns, lane, rmin, cr);
  // this lane's 8 head bits and the head bit of the arc after them (bit 8)
  const int sub = lane & 7;
  const uint32_t wa = sub < 4 ? wlo : whi, wb = sub < 4 ? whi : hw[3];
  const uint32_t my9 = __builtin_amdgcn_alignbit(wb, wa, 8 * (sub & 3)) & 0x1FFu;
  const uint32_t my8 = my9 & 0xFFu;
  const int32_t first = wrow + (sub < 4 ? 0 : __popc(wlo)) + __popc(wa & ((1u << (8 * (sub & 3))) - 1u));
  // none[e]: all ones when arc e ends no row (the arc after it is no head)
  uint32_t none[kArcsPerLane];
#pragma unroll
  for (int e = 0; e < kArcsPerLane; ++e)
    none[e] = static_cast<uint32_t>(__builtin_amdgcn_sbfe(static_cast<int32_t>(~my9), e + 1, 1));
  // The lane's open result: a run over its 8 arcs from the row's start
  // (or the lane's first arc) that carries over arc e - 1 (its bits masked
  // to the identity otherwise) when that arc ends no row.
  T run = x[0];
#pragma unroll
  for (int e = 1; e < kArcsPerLane; ++e) run = Op::join(x[e], Op::from(Op::bits(run) & none[e - 1]));
  // Segmented inclusive scan of the lanes' open results across the wave (the
  // flag of a lane is whether it holds a head). The flags live in a
  // scalar lane mask, widened after each step the way the DPP moves data.
  const uint64_t H = __ballot(my8 != 0u);
  T A = run;
  uint64_t F = H;
  seg_scan_step<Op, kDppRowShr1, 0xF>(A, F);
  F |= (F << 1) & 0xFFFEFFFEFFFEFFFEull;
  seg_scan_step<Op, kDppRowShr2, 0xF>(A, F);
  F |= (F << 2) & 0xFFFCFFFCFFFCFFFCull;
  seg_scan_step<Op, kDppRowShr4, 0xF>(A, F);
  F |= (F << 4) & 0xFFF0FFF0FFF0FFF0ull;
  seg_scan_step<Op, kDppRowShr8, 0xF>(A, F);
  F |= (F << 8) & 0xFF00FF00FF00FF00ull;
  seg_scan_step<Op, kDppRowBcast15, 0xA>(A, F);
  F |= ((F & (1ull << 15)) ? 0x00000000FFFF0000ull : 0ull) | ((F & (1ull << 47)) ? 0xFFFF000000000000ull : 0ull);
  seg_scan_step<Op, kDppRowBcast31, 0xC>(A, F);
  // lane l: the open result at the end of lane l - 1, joined with what earlier
  // tiles carry when no lane before l holds a head
  const T c = dpp_moved<Op, kDppWaveShr1, 0xF>(A);
  const uint64_t past_head = H ? ((~0ull << __builtin_ctzll(H)) << 1) : 0ull;
  const T with_open = Op::open(c, cr.open);
  const T carry = lane_in(past_head) ? c : with_open;
  // The rows this tile completes form one run [rs, re): the open row (if
  // the wave owes it) and every row of the chunk with its head here, except
  // the last one when it continues into the next tile. Their sums are
  // staged in LDS by row and written back so that store k of the wave holds
  // rows rs + 64k .. rs + 64k + 63 (coalesced); the position table turns a
  // row into its range-major index. Every lane issues the same stores
  // (unused ones get a dropped offset), so the compiler's count of
  // outstanding memory operations stays exact.
  const int32_t rs = rmin;
  const int32_t re = min(rz, next_head ? tz : tz - 1);
  // Staging slot of each arc: its row's offset from rs (as unsigned: rows
  // before rs wrap to huge values) when the arc ends its row, pushed out by
  // kPushOut otherwise. Every arc writes its run to the staging; those with
  // no row of the pass go to one of the wave's spare slots.
  uint32_t slot[kArcsPerLane];
  {
    uint32_t r = static_cast<uint32_t>(first - 1 - rs) + (my9 & 1u);  // offset of arc 0's row
#pragma unroll
    for (int e = 0; e < kArcsPerLane; ++e) {
      slot[e] = (none[e] & kPushOut) | r;  // r < 512, or wrapped past 2^31: the OR acts as an add
      r += 1u + none[e];
    }
  }
  // The staged runs: the same masked run again, now starting from the
  // carried sum unless arc 0 is a head (it reaches exactly the arcs before
  // the lane's first head, i.e. the end of the row carried into the lane;
  // an LDS atomic add of the carry to that row's slot costs more than these
  // instructions).
  T st[kArcsPerLane];
  {
    const uint32_t cont0 = static_cast<uint32_t>(__builtin_amdgcn_sbfe(static_cast<int32_t>(~my9), 0, 1));
    T r = Op::join(x[0], Op::from(Op::bits(carry) & cont0));
    st[0] = r;
#pragma unroll
    for (int e = 1; e < kArcsPerLane; ++e) {
      r = Op::join(x[e], Op::from(Op::bits(r) & none[e - 1]));
      st[e] = r;
    }
  }
  // rows within the cursor's three ranges index with it; a tile that reaches
  // past the cached boundary b3 searches its rows' ranges
  const bool many = re > cr.b3;  // uniform
  const int32_t i1 = cr.b1 - rs, i2 = cr.b2 - rs, iz = min(re, cr.b3) - rs;
  const int32_t D0 = rs + cr.d0, D1 = rs + cr.d1, D2 = rs + cr.d2;  // row rs + i goes to index i + D
  const uint32_t spare = kStageRows + (lane & (kStageSpare - 1));
  // Staging passes: rows [0, 384) of the run in every tile (6 stores),
  // rows [384, 512) only in tiles that complete more rows (a tile completes
  // at most 512). Every tile thus issues at least kStoresPerTile stores, the
  // count the compiler's memory waits assume.
  auto stage_pass = [&](auto pass_tag) {
    constexpr int pass = decltype(pass_tag)::value;
    constexpr uint32_t lo = pass == 0 ? 0u : static_cast<uint32_t>(kStageRows);
    constexpr int n = pass == 0 ? kStageRows : kTileRowsMax - kStageRows;  // rows of this pass
    // slots of the pass run [0, n); anything at or past n lands in
    // [n, n + 16), which this pass does not read back
    const uint32_t cap = spare - static_cast<uint32_t>(kStageRows - n);
#pragma unroll
    for (int e = 0; e < kArcsPerLane; ++e) stage[min(slot[e] - lo, cap)] = st[e];
    wave_lds_fence();
    T v[n / kWave];
#pragma unroll
    for (int k = 0; k < n / kWave; ++k) v[k] = stage[k * kWave + lane];
    // the offsets take one of three branches; the stores follow unconditionally
    // (stores inside the branches would leave the compiler unable to count
    // them on every path)
    uint32_t off[kStageRows / kWave];
    if (__builtin_expect(many, 0)) {
      const int32_t cnt = __popcll(__ballot(cr.sbw < re));  // entries of the window at or below the last row
      const int32_t hi = cnt < kWave ? cr.jw + cnt - 1 : ns;
      row_offsets_search(off, n / kWave, lane, static_cast<int32_t>(lo), rs, re, sb, sd, cr.jc, hi);
    } else if (i2 < iz) row_offsets<true>(off, n / kWave, lane, static_cast<int32_t>(lo), i1, i2, iz, D0, D1, D2);
    else row_offsets<false>(off, n / kWave, lane, static_cast<int32_t>(lo), i1, i2, iz, D0, D1, D2);
#pragma unroll
    for (int k = 0; k < n / kWave; ++k)
      __builtin_amdgcn_raw_buffer_store_b32(Op::bits(v[k]), out, off[k], 4 * (static_cast<int32_t>(lo) + k * kWave), 0);
    wave_lds_fence();  // the staging is rewritten next
  };
  stage_pass(std::integral_constant<int, 0>());
  if (re - rs > kStageRows) stage_pass(std::integral_constant<int, 1>());  // uniform
  // the row open at the tile's end, if the wave writes it (lane 63 holds its
  // open result)
  using Carry = typename Op::Carry;
  const T run63 = Op::from(__builtin_amdgcn_readlane(static_cast<int>(Op::bits(run)), kWave - 1));
  const T c63 = Op::from(__builtin_amdgcn_readlane(static_cast<int>(Op::bits(c)), kWave - 1));
  const Carry tail = Op::tail((H >> 63) ? run63 : Op::join(run63, c63), H ? Carry(0) : cr.open);
  const int32_t ro = tz - 1;  // the row of the tile's last arc
  const bool owe = !next_head && (tz > ta ? (ro >= r0 && ro < r1) : cr.open_row >= 0);
  cr.open_row = owe ? ro : -1;
  cr.open = owe ? tail : Carry(0);
}

}  // namespace gcs
