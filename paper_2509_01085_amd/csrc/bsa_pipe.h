// Shared by the bf16 MFMA attention kernels: work items of a launch, the walk over block lists and
// the backward's query-block records.
#pragma once

#include <math.h>

#include <algorithm>

#include "bsa_mfma.h"

namespace bsa {

constexpr int PG = 4;     // query blocks per workgroup
constexpr int PBK = 64;   // tokens per block on this path

// ---- work items -------------------------------------------------------------------------
// A launch covers `units` units of work (four query blocks of a head each).  Workgroups are
// dispatched round-robin over the 8 XCDs, so XCD x is given the contiguous unit range
// [x*q + min(x, r), ...) with q = units / 8, r = units % 8: neighbouring query blocks, whose
// lists overlap, share that XCD's L2.  When the launch is only a few rounds long (units per
// workgroup slot), its tail leaves most of the chip idle; then the last split_n units of every
// XCD's range (all of them in the shortest launches, and there in fewer segments where lists are short) are walked
// in split_S segments by separate, shorter workgroups dispatched last, and a combine launch merges their partial results.
constexpr int kCUs = 256;  // compute units of the MI355X


struct SplitPlan {
  int S, n;   // segments per split unit; split units per XCD (0: no splitting)
  int grid;   // workgroups of the main launch
  int units;  // number of split units = workgroups of the combine launch
  int by_lists;  // 1: a unit has a segment per kSegPairs listed pairs, at least two and at most S
};

constexpr int kSegPairs = 4;

// tiles: blocks of a head, the longest union a unit can walk
static SplitPlan plan_split(int units, int slots, int tiles, bool allow) {
  SplitPlan p{1, 0, 0, 0, 0};
  const int q = units / 8, r = units % 8, cmax = q + (r ? 1 : 0);
  if (!allow || q < 5) {
    // Below 40 units a launch stands alone: how long the lists are is known only on the device, and a second launch
    // costs more than it saves where a row lists one block or two (16 units, 64 tiles, one block a list: 13 us whole,
    // 21 split in eight; half of the blocks listed: 84 and 31).
  } else if (2 * units <= slots && tiles >= 32) {
    // Less than half a round: a launch lasts as long as one walk (about 10 us and 1.5 per tile) with most slots
    // empty, so every unit is split, in as many segments as there are slots.  Below 32 tiles the combine launch
    // costs what the shorter walks save.
    // 144 units, 48 tiles, a fifth split in four against all in three: walk 74 and 43 us, combine 12 and 15.
    // A segment is worth kSegPairs listed pairs of the unit or more, two segments at least: with one block a list the eight
    // segments of 64 units, 256 tiles, cost 33 us for the forward and 34 for dQ, mostly for empty partial results, two
    // cost 21 and 21 (a fifth of the units in four: 25 and 22).
    p.S = std::min(slots / units, std::min(8, tiles / 8));
    p.n = cmax;
    p.by_lists = 1;
  } else if (units < 12 * slots) {  // short launch: split the last fifth in four
    p.S = 4;
    p.n = (q + 4) / 5;
  }
  p.grid = 8 * (cmax - p.n + p.S * p.n);
  p.units = 8 * p.n;
  return p;
}

struct Item {
  int unit, seg, nseg;
  int sidx;  // ordinal of a split unit (addresses its partial results), -1 for a whole unit
};

// One XCD's range of units, walked as items: the whole units, then the segments of the split ones.
struct Share {
  int start, cnt, split, S, sbase;
  __device__ inline Share(int x, int units, int S_, int n) : S(S_), sbase(x * n) {
    const int q = units >> 3, r = units & 7;
    start = x * q + min(x, r);
    cnt = q + (x < r ? 1 : 0);
    split = min(n, cnt);
  }
  __device__ inline bool item(int k, Item& it) const {
    const int whole = cnt - split;
    if (k < whole) {
      it.unit = start + k; it.seg = 0; it.nseg = 1; it.sidx = -1;
      return true;
    }
    const int kk = k - whole, si = kk / S;
    if (si >= split) return false;
    it.unit = start + whole + si; it.seg = kk - si * S; it.nseg = S; it.sidx = sbase + si;
    return true;
  }
};

__device__ inline bool item_of(int b, int units, int S, int n, Item& it) {
  return Share(b & 7, units, S, n).item(b >> 3, it);
}

// the split unit a workgroup of the combine launch finishes (none: an XCD with fewer units than n)
__device__ inline bool split_item_of(int b, int units, int S, int n, Item& it) {
  const int q = units >> 3, r = units & 7, x = b & 7, si = b >> 3;
  const int cnt = q + (x < r ? 1 : 0), split = min(n, cnt);
  if (si >= split) return false;
  it.unit = x * q + min(x, r) + cnt - split + si; it.seg = 0; it.nseg = S; it.sidx = x * n + si;
  return true;
}

// Listed pairs of a unit, whose rows' lists stand one behind the other: the same value in every segment and in the
// combine launch, and cheaper than the union that it bounds.
__device__ inline int pairs_of(const Geom& g, const int32_t* q2k_ptr, int unit, int ngroups, int pg) {
  const int first = (unit % ngroups) * pg;
  const int32_t* ptr = q2k_ptr + (int64_t)(unit / ngroups) * g.N;
  return ptr[min(first + pg, g.N)] - ptr[first];
}

// Where the forward's two kernels are both launched: are there so many listed blocks a row that the one of bsa_attn_fwd.hip is
// the faster one?
__device__ inline bool lists_are_long(const Geom& g, const AttnArgs& a) {
  return a.fwd_long && a.q2k_ptr[g.rows] >= (int64_t)a.fwd_long * g.rows;
}

// Ascending walk over the union of NL block lists kept as bit masks in LDS.  Every value
// is wave-uniform; readfirstlane moves the words to scalar registers so the bit scanning
// costs scalar, not vector, instructions.
template <int NL, int NOWN>
struct WalkN {
  const uint32_t* masks;  // [NL][W]
  int W, own_list, word, left;
  uint32_t u, own, own2;  // own, own2: the wavefront's own list(s), NOWN of them, own_list and own_list + 1
  __device__ inline WalkN(const uint32_t* m, int W_, int own_)
      : masks(m), W(W_), own_list(own_), word(-1), left(0x7fffffff), u(0), own(0), own2(0) {}
  __device__ inline uint32_t any(int w) const {
    uint32_t all = masks[w];
#pragma unroll
    for (int k = 1; k < NL; ++k) all |= masks[k * W + w];
    return all;
  }
  __device__ inline void load() {
    u = __builtin_amdgcn_readfirstlane(any(word));
    own = __builtin_amdgcn_readfirstlane(masks[own_list * W + word]);
    if (NOWN == 2) own2 = __builtin_amdgcn_readfirstlane(masks[(own_list + 1) * W + word]);
  }
  // next tile of the union; mine: bit 0 = on the first own list, bit 1 = on the second
  __device__ inline int next(uint32_t& mine) {
    if (left <= 0) return -1;
    while (u == 0) {
      if (++word >= W) return -1;
      load();
    }
    const int b = __builtin_ctz(u);
    u &= u - 1;
    mine = ((own >> b) & 1u) | (NOWN == 2 ? ((own2 >> b) & 1u) << 1 : 0u);
    --left;
    return word * 32 + b;
  }
  // restrict a fresh walk to segment `seg` of `nseg` equal parts of the union
  __device__ inline void restrict_to(int seg, int nseg) {
    int total = 0;
    for (int w = 0; w < W; ++w) total += __builtin_popcount(__builtin_amdgcn_readfirstlane(any(w)));
    int skip = (int)((int64_t)seg * total / nseg);
    left = (int)((int64_t)(seg + 1) * total / nseg) - skip;
    while (++word < W) {
      load();
      const int c = __builtin_popcount(u);
      if (skip < c) break;
      skip -= c;
      u = 0;
    }
    for (; skip > 0; --skip) u &= u - 1;
  }
};

#define BSA_FENCE() __builtin_amdgcn_sched_barrier(0)
#define BSA_WAIT_VM(n) asm volatile("s_waitcnt vmcnt(" #n ")" ::: "memory")

// Record of 32 retained query rows in the backward workspace (the image in memory is the image in
// LDS).  A query block has one, or two when it retains more than 32 queries.
template <int D>
struct BwdRec {
  static constexpr int RB = D * 2;
  static constexpr int QC = 0;               // [32][D] bf16, swizzled rows
  static constexpr int GC = 32 * RB;         // [32][D] bf16, swizzled rows
  static constexpr int LS = 64 * RB;         // float lse2[32]
  static constexpr int DL = LS + 128;        // float -delta[32]
  static constexpr int BYTES = DL + 128;     // multiple of 256
};

int fwd_walk_units(const Geom& g, int n_keep);  // its units; within one round of the CUs the smallest that are
int grant_fwd_walk(const Geom& g, const AttnArgs& a);  // before any launch of the call
struct FwdSplit {
  int S, n, by_lists;  // segments of a split unit, split units of an XCD, as in SplitPlan
  int blocks;          // query blocks of a unit
};
int launch_fwd_walk(const Geom& g, const AttnArgs& a, int cap, FwdSplit& split, hipStream_t st);
// finishes the split units of the forward kernels that were launched; n of the others is 0
int launch_fwd_combine(const Geom& g, const AttnArgs& a, const FwdSplit& walk, const FwdSplit& pipe, hipStream_t st);
int grant_bwd_dkv_pipe(const Geom& g, const AttnArgs& a);  // before any launch of the call
int launch_bwd_dkv_pipe(const Geom& g, const AttnArgs& a, hipStream_t st);

}  // namespace bsa
