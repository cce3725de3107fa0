// Forward of the sparse attention on bf16 matrix cores (Bk = 64, d = 128 or 64).
//
//   S^T = K Q^T,  O^T += V^T P^T  over the tiles that a query block lists (Eq. 5), online softmax in the exp2 domain, the query
//   index on the MFMA column.
//
// A unit is four 32-column tiles of queries of neighbouring query blocks: a tile a block (17 to 32 retained queries: four
// blocks), two a block (more: two blocks; also the dense baseline), one for two blocks (at most 16: eight blocks).  One workgroup
// of four wavefronts, one a SIMD, walks the union of the unit's lists; the wavefronts take its entries in turn, each for all four
// tiles, and their partial results are merged at the end.  There is no barrier in the walk, a wavefront never waits for
// a tile that is not its own, and an entry costs a product only for the tiles that list it.  Q^T of the four tiles stands in 128
// registers, O^T in all 256 accumulation registers.  A wavefront has a private ring of 32-key halves in LDS (two of K, two of V):
// a half goes from memory to LDS, from there once to registers (64), and serves every tile that lists it, so an LDS fragment
// feeds 2.3 MFMAs on the benchmark layer, where the other kernel reads one for each.
//
// With one wavefront a SIMD nothing else fills a gap, so the order of instructions is fixed here.  A job is a half for
// a tile.  Behind every MFMA of the next job's S stands a share of the current job's exponentials, sums and conversions, behind every
// MFMA of the current job's O a share of the next one's maxima and exponents, and the requests and LDS reads of the
// halves to come stand one behind an MFMA each.  What does not depend on the lists is compiled for every set of tiles: a jump
// costs about 40 cycles here (the same loop with a jump for every choice took 2.38 ms on the benchmark layer).  A row maximum lags
// behind (kRise below): the accumulators are seldom scaled after the first tiles.
//
// One workgroup stays on a CU and takes unit after unit: the dispatcher hands out workgroups round the shader engines, and a CU
// that was free waited 14 us for its next one.  Units are handed out by the length of their lists, reckoned by every workgroup
// alike, and a unit begins its round of the union where the others of its XCD are by that reckoning, so that they read the same
// tiles at a time (70,400 tokens, 40 heads: 27.4 ms from the first entry on, 24.2 so).
//
// What bounds it: a wavefront's issue (33,280 tokens: something in 60 % of its cycles, a vector instruction in 41 %) next to the
// matrix cores (busy 38 %), at 2.0 GHz.  At 161,280 tokens the fabric (287 GB in 39 ms).
// Measured (MI355X, in turn with the walk of four lists with a barrier a tile, bsa_attn_pipe.hip, which stays the faster one
// where lists are short): 33,280 tokens, 12 heads, d = 128, half of the queries, p = 0.9: 1.97 -> 1.71 ms; 70,400 tokens, 40
// heads: 27.8 -> 23.7; dense, 23,296 tokens: 3.40 -> 3.09; 23,296 tokens, d = 64, every query: 1.42 -> 1.18; a quarter of the
// queries: 0.57 -> 0.54.
#include <type_traits>

#include "bsa_pipe.h"

namespace bsa {

enum FwdMode { kOne, kTwo, kPack };  // 32-column tiles: one a query block, two a block, one for two blocks

constexpr int kFwdList = 2048;     // union entries in LDS at a time
// A row maximum lags: it is moved when a logit exceeds it by more than kRise (exp2 domain).  The probability of the key at
// the maximum is 1, which bf16 holds exactly, and it is the keys that weigh most in a row whose rounding shows.  So where a
// logit exceeds the maximum by more than kLag and its probability 1 + kShare l, l the lane's sum so far, the residual of the job's
// probabilities is multiplied, too.  Error of O against that of P relative to the row's maximum (4 heads of 64 blocks, noise of 1.0 on
// the fields): a maximum that lags by up to 2^16 with no residual 1.10, this 0.98; at a noise of 0.3 1.006 and 0.999.
// A move scales 64 registers, about one and a half jobs' time, a residual costs half of that.  Time with the lag of 2^16, a move instead
// of the residual, and this: dense, 23,296 tokens, 2.96, 3.07 and 3.05 ms; 33,280 tokens 1.61, 1.66 and 1.66 ms; 3,072 tokens
// 49, 58 and 55 us.  With the limits of each tile in registers the loop spills (dense 3.28 ms).
constexpr float kLag = 3.f, kShare = 1.f, kRise = 6.f;
constexpr float kLowest = -3.4e38f;
constexpr int kFwdPlan = 512;       // items of a workgroup at most that are handed out by their length
constexpr uint32_t kFwdFixed = 256;  // what a unit costs besides its pairs, in pairs (64 to 800: no difference of more than 2 %)

// The accumulators stand in accumulation registers that are named here, not by the compiler: at the joins of the paths
// below it would move them about (64 to 176 register moves a path).  BSA_ACC_HERE: nothing of the compiler's is in an
// accumulation register here; between two of them it has no value to put there.
#define BSA_A10(t) "a" t "0", "a" t "1", "a" t "2", "a" t "3", "a" t "4", "a" t "5", "a" t "6", "a" t "7", "a" t "8", "a" t "9"
#define BSA_ACC                                                                                                              \
  BSA_A10(""), BSA_A10("1"), BSA_A10("2"), BSA_A10("3"), BSA_A10("4"), BSA_A10("5"), BSA_A10("6"), BSA_A10("7"), BSA_A10("8"), \
      BSA_A10("9"), BSA_A10("10"), BSA_A10("11"), BSA_A10("12"), BSA_A10("13"), BSA_A10("14"), BSA_A10("15"), BSA_A10("16"),   \
      BSA_A10("17"), BSA_A10("18"), BSA_A10("19"), BSA_A10("20"), BSA_A10("21"), BSA_A10("22"), BSA_A10("23"), BSA_A10("24"),  \
      "a250", "a251", "a252", "a253", "a254", "a255"

#define BSA_ACC_HERE() asm volatile("" : : : BSA_ACC)
template <int R>
__device__ inline void acc_zero() { asm volatile("v_accvgpr_write_b32 a[%0], 0" : : "n"(R)); }
template <int R>
__device__ inline float acc_get() {
  float v;
  asm volatile("v_accvgpr_read_b32 %0, a[%1]" : "=v"(v) : "n"(R));
  return v;
}
#define BSA_ACC_MUL1(k) "v_accvgpr_read_b32 %0, a[%2+" k "]\n\tv_mul_f32 %0, %1, %0\n\tv_accvgpr_write_b32 a[%2+" k "], %0\n\t"
#define BSA_ACC_MUL4(a, b, c, d) BSA_ACC_MUL1(a) BSA_ACC_MUL1(b) BSA_ACC_MUL1(c) BSA_ACC_MUL1(d)
template <int R>
__device__ inline void acc_mul16(float by) {
  float t;
  asm volatile(BSA_ACC_MUL4("0", "1", "2", "3") BSA_ACC_MUL4("4", "5", "6", "7") BSA_ACC_MUL4("8", "9", "10", "11")
               BSA_ACC_MUL4("12", "13", "14", "15") : "=&v"(t) : "v"(by), "n"(R));
}
// registers R .. R + 15 += A B; FRESH: B was written by vector instructions not long ago
template <int R, bool FRESH>
__device__ inline void acc_mfma(bf16x8 a, bf16x8 b) {
  if (FRESH) asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 a[%2:%3], %0, %1, a[%2:%3]" : : "v"(a), "v"(b), "n"(R), "n"(R + 15));
  else asm volatile("v_mfma_f32_32x32x16_bf16 a[%2:%3], %0, %1, a[%2:%3]" : : "v"(a), "v"(b), "n"(R), "n"(R + 15));
}
// the products issued so far have reached the registers
__device__ inline void acc_settled() { asm volatile("s_nop 15\n\ts_nop 15"); }

// Keeps what was computed here in this path: the compiler moves what paths have in common behind their join.
template <int S, typename T>
__device__ inline void stay1(T& x) { asm volatile("; tile %1" : "+v"(x) : "n"(S)); }
template <int S, typename... T>
__device__ inline void stay(T&... x) { (stay1<S>(x), ...); }
__device__ inline float max2(float a, float b) {
  float m;
  asm volatile("v_max_f32 %0, %1, %2" : "=v"(m) : "v"(a), "v"(b));
  return m;
}
__device__ inline void max3(float& m, float a, float b) { asm volatile("v_max3_f32 %0, %0, %1, %2" : "+v"(m) : "v"(a), "v"(b)); }
__device__ inline bf16x8 pack8(const float* v) {
  u32x4 p;
#pragma unroll
  for (int k = 0; k < 4; ++k) p[k] = pack_bf16(v[2 * k], v[2 * k + 1]);
  return as_frag(p);
}

constexpr int nth_bit(int set, int n) { return n == 0 ? __builtin_ctz(set) : nth_bit(set & (set - 1), n - 1); }

template <int D, int MODE>
struct Fwd {
  static constexpr int PGB = MODE == kPack ? 8 : MODE == kTwo ? 2 : 4;  // query blocks of a unit = lists
  static constexpr int RB = D * 2, CPR = D / 8, HB = 32 * RB;           // bytes of a row, 16-byte chunks, bytes of 32 rows
  static constexpr int DT = D / 32, DS = D / 16, NREG = DT * 16 + 2;
  static constexpr int ROWB = RB + 16;                                  // output rows in LDS, padded
  static constexpr int RING = 4 * 4 * HB;                               // four wavefronts: two halves each of K and V
  static constexpr int FIXED = RING + kFwdList * 4 + 2 * 4096 + PBK * 4 + PGB * PBK * 6 + (kFwdPlan + 1) * 4;  // LDS but for the lists' bits
  static size_t lds(const Geom& g) { return FIXED + (size_t)((PGB + 1) * ((g.N + 31) / 32) + 1) * 4; }
};

// ---- the unit's rows: which query block, retained position and token a lane's column of tile s stands for
template <int MODE>
__device__ inline int tile_block(int s, int col) { return MODE == kPack ? 2 * s + (col >> 4) : MODE == kTwo ? s >> 1 : s; }
template <int MODE>
__device__ inline int tile_pos(int s, int col) { return MODE == kPack ? (col & 15) : MODE == kTwo ? 32 * (s & 1) + col : col; }

// Retained rows and their copies (Sec. 3.2.2, token filling): where the rows of a unit go.  Token t of the unit's blocks takes
// its own row, src[t], or that of its window's critical token; dest[t] = its place in the tensor | its row << 20, or ~0.
template <int PGB>
__device__ inline void find_rows(const Geom& g, const int16_t* src, const int* koff, int i0, int end, uint32_t* dest) {
  for (int t = threadIdx.x; t < PGB * PBK; t += 256) {
    const int blk = t / PBK, c = t % PBK;
    int r = src[t];
    if (r < 0 && !g.dense) r = src[blk * PBK + window_center(g, window_of(g, c))];
    dest[t] = i0 + blk < end && r >= 0 ? (uint32_t)(block_origin(g, i0 + blk) + koff[c]) | (uint32_t)r << 20 : ~0u;
  }
}
// rows [tile][32] of the finished output to their tokens
template <int D, int MODE>
__device__ inline void store_tokens(const uint8_t* rows, const float* lse, const uint32_t* dest, uint16_t* Oh, float* Lh) {
  using F = Fwd<D, MODE>;
  const int chunk = threadIdx.x % F::CPR;
#pragma unroll 8
  for (int t = threadIdx.x / F::CPR; t < F::PGB * PBK; t += 256 / F::CPR) {
    const uint32_t e = dest[t];
    if (e == ~0u) continue;
    const int64_t tok = e & 0xfffffu;
    const int r = e >> 20;
    *reinterpret_cast<u32x4*>(Oh + tok * D + 8 * chunk) = *reinterpret_cast<const u32x4*>(rows + r * F::ROWB + 16 * chunk);
    if (chunk == 0) Lh[tok] = lse[r];
  }
}

// normalisation of a row with sum l at maximum m.  No mass: an empty list gives zeros, a list of nothing but -inf logits
// NaN (packed, where a tile of the other block's list counts as one of them, zeros for both).
template <int MODE>
__device__ inline float row_scale(float l) {
  return l > 0.f ? 1.f / l : MODE == kPack || __builtin_signbit(l) ? 0.f : NAN;
}
__device__ inline float row_lse(float m, float l) { return l > 0.f ? (m + __builtin_amdgcn_logf(l)) * kLn2 : -INFINITY; }

struct FwdArgs {
  Geom g;
  AttnArgs a;
};
// The kernel's arguments, read anew: what one part of an item needs does not stay in scalar registers through the others.
__device__ inline FwdArgs arguments() {
  auto p = (__attribute__((address_space(4))) const FwdArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  FwdArgs v;
  __builtin_memcpy(&v, (const void*)p, sizeof v);
  return v;
}

template <int D, int MODE>
__global__ __launch_bounds__(256, 1) void fwd_walk_kernel(FwdArgs) {
  using F = Fwd<D, MODE>;
  constexpr int PGB = F::PGB, RB = F::RB, CPR = F::CPR, HB = F::HB, DT = F::DT, DS = F::DS, NREG = F::NREG;
  constexpr int ND = HB / 4096;  // groups of four requests for 32 rows
  extern __shared__ __align__(16) uint8_t smem[];  // (from LDS address 0: the fragments' addresses rely on the ring's alignment)
  uint32_t* list = reinterpret_cast<uint32_t*>(smem + F::RING);
  float(*ms)[4][64] = reinterpret_cast<float(*)[4][64]>(list + kFwdList);  // maxima and sums of the wavefronts' parts
  float(*ls)[4][64] = ms + 4;
  int* koff = reinterpret_cast<int*>(ls + 4);
  int16_t* src = reinterpret_cast<int16_t*>(koff + PBK);              // a token's row among the unit's retained ones
  uint32_t* dest = reinterpret_cast<uint32_t*>(src + PGB * PBK);      // where the rows go
  uint32_t* plan = dest + PGB * PBK;                                  // [kFwdPlan + 1] items of this workgroup (below)
  int* base = reinterpret_cast<int*>(plan + kFwdPlan + 1);                   // [W + 1] entries ahead of a word's
  // behind it [PGB][W] masks

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // (read anew, too: addresses that follow from it are not kept from one item to the next)
  auto thread = [] {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
  };
  const int slot = blockIdx.x >> 3;
  const uint32_t lds0 = uniform_lds(smem) + wave * 4 * HB;  // K half, K half, V half, V half
  uint32_t off16, off32, voff[4];  // the lane's offsets in the rows of four requests, less what the instruction adds
  float c2;
  // Items of this XCD go round its workgroups as a queue would hand them out if an item lasted as long as its lists say: every
  // workgroup follows the same reckoning, so there is no counter to share, and it knows when an item begins.
  {
  const int tid = thread(), lane = tid & 63;
  const FwdArgs args = arguments();
  const Geom& g = args.g;
  const AttnArgs& a = args.a;
  if (a.fwd_long && !lists_are_long(g, a)) return;
  const int ngroups = (g.N + a.fwd_blocks - 1) / a.fwd_blocks;
  const Share share(blockIdx.x & 7, ngroups * g.B * g.H, a.split_S, a.split_n);
  const int slots = a.fwd_slots, whole = share.cnt - share.split;
  auto cost_of = [&](int k) -> uint32_t {
    return k < whole ? pairs_of(g, a.q2k_ptr, share.start + k, ngroups, a.fwd_blocks) + kFwdFixed : 0;
  };
  if (tid < PBK) koff[tid] = intra_offset(g, tid);
  c2 = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(a.sm_scale * kLog2e)));
  off16 = __builtin_amdgcn_readfirstlane(intra_offset(g, 16)) * RB;
  off32 = __builtin_amdgcn_readfirstlane(intra_offset(g, 32)) * RB;
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    const int r = n * (1024 / RB) + lane / CPR;
    voff[n] = (uint32_t)(intra_offset(g, r) * RB + (((lane % CPR) ^ swz<D>(r)) << 4) - 1024 * n);
  }

  // dense items are alike, and where there are very many a fixed share is as good
  if (slot >= slots) {
    if (tid == 0) plan[0] = (uint32_t)(whole + slot - slots) << 16, plan[1] = ~0u;  // a segment
  } else if (!g.dense && whole > slots && whole <= slots * (kFwdPlan / 2)) {
    if (wave == 0) {
      auto first_row = [&](int u) { return (int64_t)(u / ngroups) * g.N + min(u % ngroups * a.fwd_blocks, g.N); };
      const uint32_t all = a.q2k_ptr[first_row(share.start + share.cnt)] - a.q2k_ptr[first_row(share.start)];
      const uint32_t period = all / share.cnt + kFwdFixed;  // the mean of a unit
      uint32_t load = lane < slots ? cost_of(lane) : 0xffffffffu, given = 1, costs = cost_of((slots & ~63) + lane);
      if (lane == slot) plan[0] = slot << 16;
      for (int n = slots; n < whole; ++n) {
        if (!(n & 63)) costs = cost_of(n + lane);
        uint32_t low = load;
        low = min(low, (uint32_t)__builtin_amdgcn_mov_dpp(low, 0x128, 0xf, 0xf, false));
        low = min(low, (uint32_t)__builtin_amdgcn_mov_dpp(low, 0x124, 0xf, 0xf, false));
        low = min(low, (uint32_t)__builtin_amdgcn_mov_dpp(low, 0x122, 0xf, 0xf, false));
        low = min(low, (uint32_t)__builtin_amdgcn_mov_dpp(low, 0x121, 0xf, 0xf, false));
        const uint32_t at = min((uint32_t)__builtin_amdgcn_readlane(low, 0), (uint32_t)__builtin_amdgcn_readlane(low, 16));
        const int to = __builtin_ctzll(__builtin_amdgcn_ballot_w64(load == at));
        if (lane == to) {
          if (to == slot) plan[given] = n << 16 | (uint32_t)(((uint64_t)(at % period) << 16) / period);
          load += __builtin_amdgcn_readlane(costs, n & 63);
          if (++given == kFwdPlan) load = 0xfffffffeu;
        }
      }
      if (lane == slot) plan[given] = 0xffffffffu;
    }
  } else if (tid == 0) {
    plan[0] = slot < whole ? 0xfffffffeu : ~0u;  // every slots-th unit
  }
  __syncthreads();
  }
  for (int nth = 0, k = slot;; ++nth) {
  uint32_t begin = 0;  // where the item begins its round of the union, in parts of 65,536
  {
    uint32_t e = __builtin_amdgcn_readfirstlane(plan[0]);
    if (e != 0xfffffffeu) e = __builtin_amdgcn_readfirstlane(plan[nth]);
    if (e == 0xffffffffu) return;
    if (e != 0xfffffffeu) {
      k = e >> 16;
      begin = e & 0xffffu;
    } else if (nth) {
      k += arguments().a.fwd_slots;
    }
  }
  uint64_t kbase, vbase;
  int lo, hi, total;
  bf16x8 qf[4][DS];
  {
  const int tid = thread(), lane = tid & 63, grp = lane >> 5, col = lane & 31;
  const FwdArgs args = arguments();
  const Geom& g = args.g;
  const AttnArgs& a = args.a;
  const int ngroups = (g.N + a.fwd_blocks - 1) / a.fwd_blocks, W = (g.N + 31) / 32;
  const Share share(blockIdx.x & 7, ngroups * g.B * g.H, a.split_S, a.split_n);
  uint32_t* masks = reinterpret_cast<uint32_t*>(base + W + 1);
  Item it;
  if (!share.item(k, it) || (nth && it.nseg > 1)) return;  // (past the whole units)
  const int64_t bh = it.unit / ngroups;
  const int i0 = (it.unit % ngroups) * a.fwd_blocks, end = min(i0 + a.fwd_blocks, g.N);
  const uint16_t* Qh = static_cast<const uint16_t*>(a.Q) + bh * g.L * D;
  kbase = uniform64(static_cast<const uint16_t*>(a.K) + bh * g.L * D);
  vbase = uniform64(static_cast<const uint16_t*>(a.V) + bh * g.L * D);

  // requested first, used last: the retained positions; then the lists, a wavefront each (two lists: two wavefronts each)
  int kid[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int i = i0 + tile_block<MODE>(s, col), pos = tile_pos<MODE>(s, col);
    kid[s] = i < end && pos < a.n_keep ? g.dense ? pos : a.keep_idx[(bh * g.N + i) * a.n_keep + pos] : -1;
  }
  constexpr int LPW = PGB > 4 ? PGB / 4 : 1, NJ = 4;  // lists of a wavefront; entries of a list a lane has in flight
  const int step = PGB == 2 ? 128 : 64;
  int beg[LPW], cnt[LPW], ent[LPW][NJ];
#pragma unroll
  for (int q = 0; q < LPW; ++q) {
    const int ql = PGB == 2 ? wave >> 1 : wave + 4 * q, i = i0 + ql;
    const bool has = !g.dense && i < end;
    beg[q] = has ? a.q2k_ptr[bh * g.N + i] : 0;
    cnt[q] = has ? a.q2k_ptr[bh * g.N + i + 1] - beg[q] : 0;
    beg[q] += PGB == 2 ? lane + 64 * (wave & 1) : lane;
    cnt[q] -= PGB == 2 ? lane + 64 * (wave & 1) : lane;
#pragma unroll
    for (int n = 0; n < NJ; ++n) ent[q][n] = n * step < cnt[q] ? a.q2k_idx[beg[q] + n * step] : -1;
  }
  for (int n = tid; n < PGB * PBK; n += 256) src[n] = -1;
  for (int n = tid; n < PGB * W; n += 256) {
    const int w = n % W, first = w * 32;
    const bool all = g.dense && i0 + n / W < end;
    masks[n] = !all ? 0u : first + 32 <= g.N ? 0xffffffffu : (1u << (g.N - first)) - 1u;
  }
  __syncthreads();
  // Q^T fragments (B operands) of the four tiles: lane (col, grp) holds channels 16 s + 8 grp .. +7 of its column's query
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int qid = min(kid[s], PBK - 1), blk = tile_block<MODE>(s, col);
    const bool has = i0 + blk < end && tile_pos<MODE>(s, col) < a.n_keep;
    const int id = max(qid, 0);
    const int qtok = has ? block_origin(g, i0 + blk) + koff[id] : 0;
    if (has && wave == s) src[blk * PBK + id] = (int16_t)(32 * s + col);
#pragma unroll
    for (int n = 0; n < DS; ++n) {
      u32x4 v = {0u, 0u, 0u, 0u};
      if (has) v = *reinterpret_cast<const u32x4*>(Qh + (int64_t)qtok * D + 16 * n + 8 * grp);
      qf[s][n] = as_frag(v);
    }
  }
  // the unit's lists as sets (an entry out of range does not count)
#pragma unroll
  for (int q = 0; q < LPW; ++q) {
    uint32_t* set = masks + (PGB == 2 ? wave >> 1 : wave + 4 * q) * W;
    auto add = [&](int j) {
      if ((unsigned)j < (unsigned)g.N) atomicOr(&set[j >> 5], 1u << (j & 31));
    };
#pragma unroll
    for (int n = 0; n < NJ; ++n) add(ent[q][n]);
    for (int t = NJ * step; t < cnt[q]; t += step) add(a.q2k_idx[beg[q] + t]);
  }
  __syncthreads();
  find_rows<PGB>(g, src, koff, i0, end, dest);
  auto any = [&](int w) {
    uint32_t u = masks[w];
#pragma unroll
    for (int k = 1; k < PGB; ++k) u |= masks[k * W + w];
    return u;
  };
  if (wave == 0) {  // entries ahead of every word of the union
    int sum = 0;
    const int per = (W + 63) / 64;
    for (int k = 0; k < per; ++k) sum += per * lane + k < W ? __popc(any(per * lane + k)) : 0;
    int upto = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int v = __shfl_up(upto, off);
      if (lane >= off) upto += v;
    }
    int n = upto - sum;
    for (int k = 0; k < per; ++k) {
      const int w = per * lane + k;
      if (w < W) {
        base[w] = n;
        n += __popc(any(w));
      }
    }
    if (lane == 63) base[W] = upto;
  }
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int k = 0; k < DS; ++k) settle(qf[s][k]);

  __syncthreads();
  total = __builtin_amdgcn_readfirstlane(base[W]);
  lo = it.nseg > 1 ? (int)((int64_t)it.seg * total / it.nseg) : 0;
  hi = it.nseg > 1 ? (int)((int64_t)(it.seg + 1) * total / it.nseg) : total;
  }
  BSA_ACC_HERE();
  static_for<0, 4 * DT * 16>([](auto R) { acc_zero<decltype(R)::value>(); });  // O^T of tile s, channels 32 t ..: 16 (DT s + t) ..
  float m[4], l[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    m[s] = kLowest;
    l[s] = -0.f;  // the first tile makes it +0 or more
  }
  for (int p0 = lo; p0 < hi; p0 += kFwdList) {
    const int cnt = min(kFwdList, hi - p0);
    if (p0 != lo) __syncthreads();
    {
    const int tid = thread();
    const Geom g = arguments().g;
    const int W = (g.N + 31) / 32;
    const uint32_t* masks = reinterpret_cast<uint32_t*>(base + W + 1);
    for (int t = tid; t < g.N; t += 256) {
      const int w = t >> 5, bit = t & 31;
      uint32_t u = masks[w];
#pragma unroll
      for (int q = 1; q < PGB; ++q) u |= masks[q * W + w];
      const int at = base[w] + __popc(u & ((1u << bit) - 1u)) - p0;
      if (((u >> bit) & 1u) && (unsigned)at < (unsigned)cnt) {
        uint32_t lists = 0, tiles = 0;
#pragma unroll
        for (int k = 0; k < PGB; ++k) lists |= ((masks[k * W + w] >> bit) & 1u) << k;
        if (MODE == kOne) tiles = lists;
        if (MODE == kTwo) tiles = (lists & 1u) * 3u | (lists >> 1) * 12u;
        if (MODE == kPack) {
          const uint32_t e = (lists | lists >> 1) & 0x55u;
          tiles = (e | e >> 1) & 0x33u;
          tiles = (tiles | tiles >> 2) & 0xfu;
        }
        list[at] = (uint32_t)block_origin_fast(g, t) | tiles << 20 | lists << 24;
      }
    }
    }
    __syncthreads();
    const int mine = (cnt - wave + 3) >> 2;
    if (mine <= 0) continue;
    const int lane = thread() & 63, grp = lane >> 5, col = lane & 31;

    // ---- this wavefront's walk: every fourth entry, in halves of 32 keys.  A whole unit begins where the others of this XCD
    // are at the time, and goes round: they read the same few tiles at a time, which one L2 holds.
    const int nh = 2 * mine;
    const int from = begin ? (int)((uint64_t)begin * cnt >> 16) : 0;
    auto entry = [&](int i) {
      const int p = 4 * min(i, mine - 1) + wave + from;
      return list[p < cnt ? p : p - cnt];
    };
    auto source = [&](uint64_t tensor, uint32_t e, int part) { return tensor + (uint64_t)(e & 0xfffffu) * RB + (part ? off32 : 0u); };
    auto request = [&](uint64_t src, uint32_t dst, auto N) {  // 1 KB of 32 rows
      constexpr int n = decltype(N)::value;
      dma_kb<1024 * (n & 3)>(src + (n >> 2 ? off16 : 0u), voff[n & 3], dst + 4096 * (n >> 2));
    };
    // LDS addresses of the fragments: constants and swizzles are flipped bits of one address each
    const int L16 = lane & 15, q16 = lane >> 4, rsub = L16 >> 2, jj = L16 & 3;
    const uint32_t kat = col * RB + ((grp ^ swz<D>(col)) << 4);
    const uint32_t vat = 2 * HB + (4 * grp + rsub) * RB + (((D == 128 ? rsub : rsub >> 1) << 2 | ((2 * (q16 & 1) + (jj >> 1)) ^ grp)) << 4) + 8 * (jj & 1);
    uint32_t ats = kat | vat << 16;  // (in one register)
    stay1<0>(ats);
    bf16x8 kf[DS], vf[2 * DT];
    auto read_k = [&](uint32_t at, auto KK) { kf[KK] = frag_at(at ^ (32 * KK)); };
    auto read_v = [&](uint32_t at, auto VV) {
      constexpr int v = decltype(VV)::value;
      const uint32_t q = at ^ ((v % DT) << 6);
      vf[v] = frag_tr_at(q + (v / DT) * 16 * RB, (q ^ (8 * RB | 32)) + (v / DT) * 16 * RB);
    };
    auto k_at = [&](int h) {
      stay1<0>(ats);
      return (ats & 0xffffu) + (lds0 + (h & 1) * HB);
    };
    auto v_at = [&](int h) {
      stay1<0>(ats);
      return (ats >> 16) + (lds0 + (h & 1) * HB);
    };
    // Halves go from memory to LDS one half ahead of the reads into registers, and those one job ahead of their use; past
    // the end the last tile is requested again.  e0, e1: entries of the tile at hand and of the next one.
    uint32_t e0 = __builtin_amdgcn_readfirstlane(entry(0)), e1 = __builtin_amdgcn_readfirstlane(entry(1));
    {
      const uint64_t k0 = source(kbase, e0, 0), k1 = source(kbase, e0, 1), v0 = source(vbase, e0, 0);
      static_for<0, 4 * ND>([&](auto N) { request(k0, lds0, N); });
      static_for<0, 4 * ND>([&](auto N) { request(k1, lds0 + HB, N); });
      static_for<0, 4 * ND>([&](auto N) { request(v0, lds0 + 2 * HB, N); });
    }
#pragma unroll
    for (int v = 0; v < 2 * DT; ++v) vf[v] = as_frag(u32x4{0u, 0u, 0u, 0u});
    wait_vm<8 * ND>();
    {
      const uint32_t at = k_at(0);
      static_for<0, DS>([&](auto KK) { read_k(at, KK); });
    }

    // Runs f for one tile.
    auto for_tile = [&](int s, auto f) {
      if (s & 2) {
        if (s & 1) f(std::integral_constant<int, 3>{});
        else f(std::integral_constant<int, 2>{});
      } else {
        if (s & 1) f(std::integral_constant<int, 1>{});
        else f(std::integral_constant<int, 0>{});
      }
    };
    constexpr int E = 4;  // exponentials taken ahead of the phase boundary
    f32x16 x;     // logits of the next job
    float y[16];  // exponents, then probabilities of the current one
#pragma unroll
    for (int r = 0; r < 16; ++r) y[r] = r < E ? 0.f : -INFINITY;
    // A job is (half, tile).  The loop is compiled for every set of tiles that list an entry: what depends on the place of
    // a job in its half costs nothing, and jumps (about 40 cycles each for a wavefront alone on its SIMD) are few.
    // Requests and LDS reads are issued one behind every product: a wavefront waits for the port at a second one.
    int bc = __builtin_ctz(e0 >> 20);  // tile of the current job: at first none, with probabilities of 0 for a tile that will have one
    bool vfree = false;  // the previous half had one job: its V is yet to be read
    int hn = 0;
    float sum = 0.f, mx = 0.f;
    bf16x8 pf[2];
    // softmax of the current job, an eighth (or quarter) of it behind an MFMA; sums follow the exponentials at a step's distance
    auto softmax = [&](auto S, auto KK) {
      constexpr int s = decltype(S)::value, k = decltype(KK)::value;
      constexpr int ea = E + (16 - E) * k / DS, ez = E + (16 - E) * (k + 1) / DS, pa = 12 * k / DS, pz = 12 * (k + 1) / DS;
#pragma unroll
      for (int r = ea; r < ez; ++r) {
        stay1<s>(y[r]);
        y[r] = __builtin_amdgcn_exp2f(y[r]);
      }
      static_assert(pz <= ea, "summed at a distance from the exponentials");
#pragma unroll
      for (int r = pa; r < pz; ++r) {
        if (r == 0) sum = y[r];
        else sum += y[r];
      }
      if (pa < 8 && pz >= 8) pf[0] = pack8(y);
      stay<s>(sum);
      if (k == DS - 1) stay<s>(pf[0]);
    };
    // S^T = K Q^T of the next job under the softmax of the current one.  V: half hv of V goes to registers, the one behind it
    // is requested.
    auto logits = [&](auto S, auto V, int hv) {
      constexpr int s = decltype(S)::value;
      uint64_t src = 0;
      uint32_t at = 0, dst = 0;
      if (V) {
        wait_vm<4 * ND>();
        src = source(vbase, (hn ^ (hv + 1)) & ~1 ? e1 : e0, (hv + 1) & 1);
        dst = lds0 + (2 + ((hv + 1) & 1)) * HB;
        at = v_at(hv);
      }
      BSA_ACC_HERE();
      static_for<0, DS>([&](auto KK) {
        constexpr int k = decltype(KK)::value;
        if constexpr (k == 0) mfma_first(x, kf[k], qf[s][k]);
        else mfma_next(x, kf[k], qf[s][k]);
        if constexpr (decltype(V)::value) {
          static_for<k * 2 * DT / DS, (k + 1) * 2 * DT / DS>([&](auto VV) { read_v(at, VV); });
          static_for<k * 4 * ND / DS, (k + 1) * 4 * ND / DS>([&](auto N) { request(src, dst, N); });
        }
        softmax(S, KK);
        BSA_FENCE();
      });
    };
    // O^T += V^T P^T of the current job under the maxima and exponents of the next one, tile sn (none: -1), of the half hn.  First: the job
    // before had all of the half's K in registers, and the half behind the next one is requested.  Last: K of the next half goes to registers.
    auto values = [&](auto S, auto SN, auto First, auto Last) {
      constexpr int s = decltype(S)::value, sn = decltype(SN)::value;
      uint64_t src = 0;
      uint32_t at = 0, dst = 0;
      if (Last) {
        if (First) wait_vm<4 * ND>();
        else wait_vm<12 * ND>();
        at = k_at(hn + 1);
      }
      if (First) {
        src = source(kbase, e1, hn & 1);
        dst = lds0 + (hn & 1) * HB;
      }
      BSA_ACC_HERE();
      static_for<0, 2 * DT>([&](auto VV) {
        constexpr int v = decltype(VV)::value, n = 2 * DT - 2, ra = v < 2 ? 0 : 16 * (v - 2) / n, rz = v < 2 ? 0 : 16 * (v - 1) / n;
        acc_mfma<16 * (DT * s + v % DT), v % DT == 0>(vf[v], pf[v / DT]);
        if constexpr (v < 2) {  // what is left of the softmax, while the logits are on their way
          sum += y[12 + 2 * v];
          sum += y[13 + 2 * v];
          if (v == 1) {
            l[s] += sum;
            pf[1] = pack8(y + 8);
            stay<s>(pf[1]);
          }
          stay<s>(sum);
        }
        if constexpr (decltype(Last)::value) static_for<v * DS / (2 * DT), (v + 1) * DS / (2 * DT)>([&](auto KK) { read_k(at, KK); });
        if constexpr (decltype(First)::value) static_for<v * 4 * ND / (2 * DT), (v + 1) * 4 * ND / (2 * DT)>([&](auto N) { request(src, dst, N); });
        if constexpr (sn >= 0) {
          if constexpr (v == 1) {  // (the logits are whole now)
            stay<s>(m[sn]);
            if (MODE == kPack) {
              const uint32_t both = (e0 >> (24 + 2 * sn)) & 3u;
              if (both != 3u) {
                const bool own_block = (both >> (col >> 4)) & 1u;
#pragma unroll
                for (int r = 0; r < 16; ++r) x[r] = own_block ? x[r] : -INFINITY;
              }
            }
          }
#pragma unroll
          for (int r = ra; r < rz; ++r) {
            if (r == 1) mx = max2(x[0], x[1]);
            else if (r & 1) max3(mx, x[r - 1], x[r]);
            y[r] = __builtin_fmaf(x[r], c2, -m[sn < 0 ? 0 : sn]);
            if (r < E) y[r] = __builtin_amdgcn_exp2f(y[r]);
            stay1<s>(y[r]);
          }
        }
        BSA_FENCE();
      });
    };
    // a row maximum of the next job rises: its tile's sums and accumulators follow (at the tile's first job they are zeros)
    auto raise = [&](auto S) {
      constexpr int s = decltype(S)::value;
      const float up = fmaxf(m[s], pair_max(mx) * c2), alpha = __builtin_amdgcn_exp2f(m[s] - up);
      if (__builtin_amdgcn_ballot_w64(m[s] != kLowest) != 0) {
        l[s] *= alpha;
        acc_settled();
        static_for<0, DT>([&](auto T) { acc_mul16<16 * (DT * s + decltype(T)::value)>(alpha); });
      }
      m[s] = up;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        y[r] = __builtin_fmaf(x[r], c2, -up);
        if (r < E) y[r] = __builtin_amdgcn_exp2f(y[r]);
      }
    };
    // O^T of tile s += V^T R^T, R what the rounding to bf16 will leave of the next job's probabilities.  First job of its half: V
    // is not in registers yet, and what is there has served.
    auto residual = [&](auto S, auto First) {
      constexpr int s = decltype(S)::value;
      if constexpr (decltype(First)::value) {
        wait_vm<0>();
        const uint32_t at = v_at(hn);
        static_for<0, 2 * DT>([&](auto VV) { read_v(at, VV); });
      }
      BSA_ACC_HERE();
      static_for<0, 2>([&](auto Q) {
        constexpr int q = decltype(Q)::value;
        u32x4 left;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int r = 8 * q + 2 * k;
          const float a = r < E ? y[r] : __builtin_amdgcn_exp2f(y[r]), b = r < E ? y[r + 1] : __builtin_amdgcn_exp2f(y[r + 1]);
          const uint32_t p = pack_bf16(a, b);
          left[k] = pack_bf16(a - __uint_as_float(p << 16), b - __uint_as_float(p & 0xffff0000u));
        }
        static_for<q * DT, (q + 1) * DT>([&](auto VV) {
          constexpr int v = decltype(VV)::value;
          acc_mfma<16 * (DT * s + v % DT), v % DT == 0>(vf[v], as_frag(left));
        });
      });
    };
    using std::bool_constant;
    auto entry_halves = [&](auto A) {
      constexpr int set = decltype(A)::value, jobs = __builtin_popcount(set);
      for (int part = 0; part < 2; ++part, ++hn) {
        static_for<0, jobs>([&](auto J) {
          constexpr int j = decltype(J)::value, bn = nth_bit(set, j);
          const std::integral_constant<int, bn> S{};
          constexpr bool last = j == jobs - 1;
          if constexpr (j == 0) {
            if (vfree) logits(S, bool_constant<true>{}, hn - 1);
            else logits(S, bool_constant<false>{}, 0);
            for_tile(bc, [&](auto C) { values(C, S, bool_constant<true>{}, bool_constant<last>{}); });
          } else {
            logits(S, bool_constant<j == 1>{}, hn);
            values(std::integral_constant<int, nth_bit(set, j - 1)>{}, S, bool_constant<false>{}, bool_constant<last>{});
          }
          if (__builtin_expect(__builtin_amdgcn_ballot_w64(mx * c2 > m[bn] + kLag) != 0, 0)) {
            const float top = __builtin_fmaf(mx, c2, -m[bn]);
            if (__builtin_amdgcn_ballot_w64(top > kRise) != 0) raise(S);
            else if (__builtin_amdgcn_ballot_w64(__builtin_amdgcn_exp2f(top) > __builtin_fmaf(l[bn], kShare, 1.f)) != 0) residual(S, bool_constant<j == 0>{});
          }
        });
        bc = nth_bit(set, jobs - 1);
        vfree = jobs == 1;
      }
    };
    for (;;) {
      const uint32_t set = (e0 >> 20) & 15u;
      if constexpr (MODE == kTwo) {
        if (set == 3) entry_halves(std::integral_constant<int, 3>{});
        else if (set == 12) entry_halves(std::integral_constant<int, 12>{});
        else entry_halves(std::integral_constant<int, 15>{});
      } else {
        switch (set) {
          case 1: entry_halves(std::integral_constant<int, 1>{}); break;
          case 2: entry_halves(std::integral_constant<int, 2>{}); break;
          case 3: entry_halves(std::integral_constant<int, 3>{}); break;
          case 4: entry_halves(std::integral_constant<int, 4>{}); break;
          case 5: entry_halves(std::integral_constant<int, 5>{}); break;
          case 6: entry_halves(std::integral_constant<int, 6>{}); break;
          case 7: entry_halves(std::integral_constant<int, 7>{}); break;
          case 8: entry_halves(std::integral_constant<int, 8>{}); break;
          case 9: entry_halves(std::integral_constant<int, 9>{}); break;
          case 10: entry_halves(std::integral_constant<int, 10>{}); break;
          case 11: entry_halves(std::integral_constant<int, 11>{}); break;
          case 12: entry_halves(std::integral_constant<int, 12>{}); break;
          case 13: entry_halves(std::integral_constant<int, 13>{}); break;
          case 14: entry_halves(std::integral_constant<int, 14>{}); break;
          default: entry_halves(std::integral_constant<int, 15>{}); break;
        }
      }
      if (hn >= nh) break;
      e0 = e1;
      e1 = __builtin_amdgcn_readfirstlane(entry((hn >> 1) + 1));
    }
    // the last job
    if (vfree) {
      wait_vm<0>();
      const uint32_t at = v_at(nh - 1);
      static_for<0, 2 * DT>([&](auto VV) { read_v(at, VV); });
    }
    static_for<0, DS>([&](auto KK) { softmax(std::integral_constant<int, 0>{}, KK); });
    for_tile(bc, [&](auto C) { values(C, std::integral_constant<int, -1>{}, bool_constant<false>{}, bool_constant<false>{}); });
    BSA_WAIT_VM(0);
  }

  // ---- sum of the four wavefronts, in order, a tile at a time through the idle ring (two tiles fit): wavefront w sums DT of
  // the 4 DT groups of four channels
  BSA_ACC_HERE();
  acc_settled();
  const int lane = thread() & 63, grp = lane >> 5, col = lane & 31;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    ms[wave][s][lane] = m[s];
    ls[wave][s][lane] = l[s];
  }
  {
  const FwdArgs args = arguments();
  const Geom& g = args.g;
  const AttnArgs& a = args.a;
  const int ngroups = (g.N + a.fwd_blocks - 1) / a.fwd_blocks;
  const Share share(blockIdx.x & 7, ngroups * g.B * g.H, a.split_S, a.split_n);
  Item it;
  share.item(k, it);
  const int64_t bh = it.unit / ngroups;
  constexpr int RW = 4 * DT * 64;
  f32x4* red = reinterpret_cast<f32x4*>(smem);  // [parity][wavefront][channel group][64 lanes]
  float* part = it.sidx >= 0 ? a.part + ((int64_t)it.sidx * a.split_S + it.seg) * (4 * NREG * 64) + lane : nullptr;
  float* lse = reinterpret_cast<float*>(list);
  u32x2 out[4][DT];
  __syncthreads();
  static_for<0, 4>([&](auto S) {
    constexpr int s = decltype(S)::value;
    float mt = ms[0][s][lane], lt = -0.f;
#pragma unroll
    for (int w = 1; w < 4; ++w) mt = fmaxf(mt, ms[w][s][lane]);
#pragma unroll
    for (int w = 0; w < 4; ++w) lt += ls[w][s][lane] * __builtin_amdgcn_exp2f(ms[w][s][lane] - mt);
    const float f = __builtin_amdgcn_exp2f(m[s] - mt);
    f32x4* half = red + (s & 1) * 4 * RW;
    BSA_ACC_HERE();
    static_for<0, 4 * DT>([&](auto Q) {
      constexpr int q = decltype(Q)::value, r = 16 * DT * s + 4 * q;
      half[wave * RW + q * 64 + lane] = f32x4{acc_get<r>() * f, acc_get<r + 1>() * f, acc_get<r + 2>() * f, acc_get<r + 3>() * f};
    });
    __syncthreads();
    const float lsum = pair_sum(lt), inv = row_scale<MODE>(lsum);
#pragma unroll
    for (int n = 0; n < DT; ++n) {
      const int q = wave * DT + n;  // channels 8 q + 4 grp .. +3
      f32x4 v = half[q * 64 + lane];
#pragma unroll
      for (int w = 1; w < 4; ++w) v += half[w * RW + q * 64 + lane];
      if (it.nseg > 1) {
#pragma unroll
        for (int e = 0; e < 4; ++e) part[((int64_t)s * NREG + 4 * q + e) * 64] = v[e];
      }
      out[s][n].x = pack_bf16(v[0] * inv, v[1] * inv);
      out[s][n].y = pack_bf16(v[2] * inv, v[3] * inv);
    }
    if (wave == s) {
      if (it.nseg > 1) {
        part[((int64_t)s * NREG + NREG - 2) * 64] = mt;
        part[((int64_t)s * NREG + NREG - 1) * 64] = lt;
      }
      if (grp == 0) lse[32 * s + col] = row_lse(mt, lsum);
    }
  });
  if (it.nseg == 1) {
    uint8_t* rows = smem;  // (the even half: read for the last time ahead of the last barrier)
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int n = 0; n < DT; ++n) *reinterpret_cast<u32x2*>(rows + (32 * s + col) * F::ROWB + 16 * (wave * DT + n) + 8 * grp) = out[s][n];
    __syncthreads();
    store_tokens<D, MODE>(rows, lse, dest, static_cast<uint16_t*>(a.O_out) + bh * g.L * D, a.LSE_out + bh * g.L);
  }

  }
  __syncthreads();
  }
}

// Merges the segments of a split unit, in order; wavefront s has tile s.  Both forward kernels leave their partial results alike
// (of the other one, two tiles a block, a unit has eight tiles and two workgroups here), so where both are launched one
// combine launch serves the one that worked: lists of one block, 259 blocks, 3 heads, d = 128, every query, 43 us with a launch
// each and 34 so; of 16 blocks, 364 blocks, 12 heads, half of the queries 196 and 193.
template <int D, int MODE>
__global__ __launch_bounds__(256) void fwd_combine_kernel(Geom g, AttnArgs a, FwdSplit walk, FwdSplit pipe) {
  using F = Fwd<D, MODE>;
  constexpr int PGB = F::PGB, DT = F::DT, NREG = F::NREG;
  __shared__ __align__(16) uint8_t rows[128 * F::ROWB];
  __shared__ float lse[128];
  __shared__ int koff[PBK];
  __shared__ int16_t src[PGB * PBK];
  __shared__ uint32_t dest[PGB * PBK];
  const int tid = threadIdx.x, lane = tid & 63, s = tid >> 6, grp = lane >> 5, col = lane & 31;
  const FwdSplit p = (a.fwd_long ? lists_are_long(g, a) : walk.n > 0) ? walk : pipe;
  const int parts = p.blocks > PGB ? p.blocks / PGB : 1, nth = blockIdx.x >> 3, sub = nth % parts;  // workgroups of a unit
  const int ngroups = (g.N + p.blocks - 1) / p.blocks;
  Item it;
  if (!split_item_of((nth / parts) << 3 | (blockIdx.x & 7), ngroups * g.B * g.H, p.S, p.n, it)) return;
  const int64_t bh = it.unit / ngroups;
  const int i0 = (it.unit % ngroups) * p.blocks + sub * PGB, end = min(i0 + min(p.blocks, PGB), g.N);
  if (p.by_lists) it.nseg = min(it.nseg, max(2, pairs_of(g, a.q2k_ptr, it.unit, ngroups, p.blocks) / kSegPairs));
  if (tid < PBK) koff[tid] = intra_offset(g, tid);
  for (int k = tid; k < PGB * PBK; k += 256) src[k] = -1;
  __syncthreads();
  const int blk = tile_block<MODE>(s, col), pos = tile_pos<MODE>(s, col);
  if (i0 + blk < end && pos < a.n_keep)
    src[blk * PBK + min(max(a.keep_idx[(bh * g.N + i0 + blk) * a.n_keep + pos], 0), PBK - 1)] = (int16_t)(32 * s + col);
  __syncthreads();
  find_rows<PGB>(g, src, koff, i0, end, dest);
  const int64_t seg = 4 * NREG * 64 * parts;
  const float* part = a.part + (int64_t)it.sidx * p.S * seg + (4 * sub + s) * (NREG * 64) + lane;
  // m = max m_s, (l, O~) = sum of (l_s, O~_s) 2^(m_s - m)
  float m = kLowest, l = -0.f;
  for (int sg = 0; sg < it.nseg; ++sg) m = fmaxf(m, part[sg * seg + (NREG - 2) * 64]);
  float o[DT * 16];
#pragma unroll
  for (int k = 0; k < DT * 16; ++k) o[k] = 0.f;
  for (int sg = 0; sg < it.nseg; ++sg) {
    float v[NREG];  // all loads of the segment in flight together
#pragma unroll
    for (int k = 0; k < NREG; ++k) v[k] = __builtin_nontemporal_load(part + sg * seg + k * 64);
    const float w = __builtin_amdgcn_exp2f(v[NREG - 2] - m);
    l += w * v[NREG - 1];
#pragma unroll
    for (int k = 0; k < DT * 16; ++k) o[k] += w * v[k];
  }
  l = pair_sum(l);
  const float inv = row_scale<MODE>(l);
#pragma unroll
  for (int q = 0; q < DT * 4; ++q) {
    u32x2 v;
    v.x = pack_bf16(o[4 * q] * inv, o[4 * q + 1] * inv);
    v.y = pack_bf16(o[4 * q + 2] * inv, o[4 * q + 3] * inv);
    *reinterpret_cast<u32x2*>(rows + (32 * s + col) * F::ROWB + 16 * q + 8 * grp) = v;
  }
  if (grp == 0) lse[32 * s + col] = row_lse(m, l);
  __syncthreads();
  store_tokens<D, MODE>(rows, lse, dest, static_cast<uint16_t*>(a.O_out) + bh * g.L * D, a.LSE_out + bh * g.L);
}

struct FwdPlan {
  int blocks;        // query blocks of a unit
  int units;
  int slots;         // workgroups of an XCD that walk whole units
  int S, n;          // segments of a split unit, split units of an XCD
};

static int mode_of(const Geom& g, int n_keep) { return g.dense || n_keep > 32 ? kTwo : n_keep > 16 ? kOne : kPack; }

// One workgroup a CU.  cap: partial results (of a unit's segment) that the workspace holds.
static FwdPlan plan_fwd(const Geom& g, int mode, int cap) {
  const int most = mode == kPack ? 8 : mode == kTwo ? 2 : 4, least = mode == kPack ? 2 : 1;
  FwdPlan p{most, 0, 0, 1, 0};
  auto units_of = [&](int n) { return (g.N + n - 1) / n * g.B * g.H; };
  // Within one round, the smallest units that still are one: 4 heads of 128 blocks, 32 of 64 queries kept, 72 listed, units of
  // four blocks 97 us, of two 71.
  while (p.blocks > least && units_of(p.blocks - least) <= kCUs) p.blocks -= least;
  p.units = units_of(p.blocks);
  const int q = p.units / 8, cmax = q + (p.units % 8 ? 1 : 0);
  if (p.units > kCUs) {
    // The last units of an XCD in halves, handed out at the end: enough to even out what the reckoning of lengths misses, no
    // more, because a segment costs what a unit costs besides its walk and the combine launch its partial results.  Only while the
    // workspace has room, which is sized by the other kernel's plan: below twelve rounds of its workgroups.
    // Every twelfth unit in two, against every fifth in four and none: 33,280 tokens 1.77, 1.87 and 1.83 ms, 23,296 tokens
    // with short lists 0.485, 0.548 and 0.486, with a quarter of the queries 0.58, 0.61 and 0.63.
    p.S = 2;
    p.n = (q + 11) / 12;
    const int over = cmax - kCUs / 8;  // fewer than two rounds: what is more than one, in quarters
    if (over < kCUs / 8 && 8 * over * 4 <= cap) {
      p.S = 4;
      p.n = over;
    }
  }
  if (8 * p.n * p.S > cap) p.n = 0, p.S = 1;
  p.slots = std::min(cmax - p.n, kCUs / 8);
  return p;
}

int fwd_walk_units(const Geom& g, int n_keep) { return plan_fwd(g, mode_of(g, n_keep), 0).units; }

// calls f with the channels and the mode as constants
template <typename F>
static int for_instance(const Geom& g, int n_keep, F f) {
  auto go = [&](auto D) {
    const int mode = mode_of(g, n_keep);
    return mode == kPack ? f(D, std::integral_constant<int, kPack>{}) : mode == kTwo ? f(D, std::integral_constant<int, kTwo>{}) : f(D, std::integral_constant<int, kOne>{});
  };
  return g.d == 128 ? go(std::integral_constant<int, 128>{}) : go(std::integral_constant<int, 64>{});
}

int grant_fwd_walk(const Geom& g, const AttnArgs& a) {
  return for_instance(g, a.n_keep, [&](auto D, auto M) { return allow_dynamic_lds<fwd_walk_kernel<D, M>>(Fwd<D, M>::lds(g)); });
}

int launch_fwd_walk(const Geom& g, const AttnArgs& args, int cap, FwdSplit& split, hipStream_t st) {
  AttnArgs a = args;
  const FwdPlan p = plan_fwd(g, mode_of(g, a.n_keep), a.fwd_ws ? cap : 0);
  split = FwdSplit{p.S, p.n, 0, p.blocks};
  a.split_S = p.S;
  a.split_n = p.n;
  a.fwd_slots = p.slots;
  a.fwd_blocks = p.blocks;
  return for_instance(g, a.n_keep, [&](auto D, auto M) {
    hipLaunchKernelGGL((fwd_walk_kernel<D, M>), dim3(8 * (p.slots + p.S * p.n)), dim3(256), (Fwd<D, M>::lds(g)), st, FwdArgs{g, a});
    return check_launch();
  });
}

int launch_fwd_combine(const Geom& g, const AttnArgs& a, const FwdSplit& walk, const FwdSplit& pipe, hipStream_t st) {
  return for_instance(g, a.n_keep, [&](auto D, auto M) {
    const int grid = 8 * std::max(walk.n, pipe.n * std::max(1, pipe.blocks / Fwd<D, M>::PGB));
    if (grid) hipLaunchKernelGGL((fwd_combine_kernel<D, M>), dim3(grid), dim3(256), 0, st, g, a, walk, pipe);
    return check_launch();
  });
}

}  // namespace bsa
