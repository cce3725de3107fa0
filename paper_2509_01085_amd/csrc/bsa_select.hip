// Sparse-KV selection (Sec. 3.2.3, Eq. 4): block logits -> per-row order (score descending) ->
// cumulative softmax mass -> minimal prefix reaching the threshold -> CSR block lists
// (the paper's q2k_num / q2k_index of Sec. 3.3) plus the transposed lists that give every
// KV block a single owner in the backward pass.
//
// Pipeline (all on one stream, no host round trip; nnz stays on the device):
//   1. scores_kernel       s[r][j] = score_scale * <Qbar_r, Kbar_j>, fp64, channel-ascending,
//      scores_tile_kernel  multiply and add rounded separately (the order another
//                          implementation must follow to reproduce every comparison)
//   2. row_select_kernel   one workgroup per row: e = exp(s - s_max), Z, then a bisection for
//                          the key of the last block of the minimal prefix (no sort); marks
//                          the k* selected blocks in a bit mask, writes k*
//   3. scan_kernel         exclusive scan of the counts -> q2k_ptr, nnz
//   4. expand_kernel       bit mask -> ascending block ids at q2k_ptr[r]
//   5-7. transpose         per (head, 8 columns): ballot-count, scan, ballot-fill -> k2q
//   lists_kernel           3 to 7 in one launch where rows are few
#include <math.h>

#include "bsa_common.h"

namespace bsa {

static inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct SelectWs {
  double* scores;   // [rows][N]
  uint32_t* mask;   // [rows][W]
  int32_t* cnt;     // [rows]  q2k counts
  int32_t* kcnt;    // [rows]  k2q counts
  size_t bytes;
};

static SelectWs carve(const Geom& g, void* base) {
  SelectWs w;
  const size_t W = (g.N + 31) / 32;
  size_t off = 0;
  uint8_t* p = static_cast<uint8_t*>(base);
  w.scores = reinterpret_cast<double*>(p + off); off += align256((size_t)g.rows * g.N * sizeof(double));
  w.mask = reinterpret_cast<uint32_t*>(p + off); off += align256((size_t)g.rows * W * 4);
  w.cnt = reinterpret_cast<int32_t*>(p + off); off += align256((size_t)g.rows * 4);
  w.kcnt = reinterpret_cast<int32_t*>(p + off); off += align256((size_t)g.rows * 4);
  w.bytes = off;
  return w;
}

size_t select_workspace_bytes(const Geom& g) { return carve(g, nullptr).bytes; }

// ---- library-owned scratch for callers that cannot allocate (bsa_select_kv_static) ----------
// One copy per GPU, resident from module load until the process ends.  `scratch` names the
// array only towards hipGetSymbolAddress: in host code the identifier is a host-side stand-in,
// not a device address, so everything below that needs the memory uses the looked-up pointer.
constexpr size_t kStaticScratchBytes = BSA_STATIC_SELECT_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

int static_select_scratch(void** ptr, size_t* bytes) {
  constexpr int kMaxDev = 64;
  static void* dev_ptr[kMaxDev] = {};  // each device holds its own copy at its own address
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDev) return BSA_ERR_LAUNCH;
  if (!dev_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return BSA_ERR_LAUNCH;
    dev_ptr[dev] = p;
  }
  *ptr = dev_ptr[dev];
  *bytes = kStaticScratchBytes;
  return BSA_OK;
}

// ---------------------------------------------------------------- 1. block logits
// A wavefront computes R rows x 64 columns, one column a lane: the K operand of a channel is one LDS read
// (the tile is staged transposed, the next 32 channels are requested while these are multiplied), the R
// Q operands are the same for all lanes and come through scalar loads, so for R = 8 sixteen fp64 instructions
// stand against one LDS read.  A workgroup is 4 R rows.  The latency of a stage bounds it where workgroups are few;
// where they are many it reaches 43 % of the fp64 rate (40 heads of 1,100 blocks, d = 128), which is not its bound,
// and the tile below 51 %.
// Every output is accumulated over the channels in ascending order, multiply and add rounded
// separately, whatever the tiling.
// Microseconds, d = 128, the 64 x 64 tile below and this: 12 heads of 48 blocks 32 and 10, 4 of 546 47 and 32, 12 of
// 364 44 and 32.
constexpr int TJ = 64, KC = 32;
typedef double double2_a8 __attribute__((ext_vector_type(2), aligned(8)));  // (rows are only 8-byte aligned)

template <int R>
__global__ __launch_bounds__(256) void scores_kernel(Geom g, const double* __restrict__ Qbar,
                                                     const double* __restrict__ Kbar, double scale,
                                                     double* __restrict__ S) {
  __shared__ double ks[2][KC][TJ + 1];
  constexpr int NP = KC * TJ / 2 / 256;  // 16-byte pieces of a stage per thread
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int bh = blockIdx.z;
  const int i0 = (blockIdx.y * 4 + wave) * R, j0 = blockIdx.x * TJ;
  const double* Qh = Qbar + (int64_t)bh * g.N * g.d;
  const double* Kh = Kbar + (int64_t)bh * g.N * g.d;
  const double* q[R];  // rows past the last one repeat it and are not stored
#pragma unroll
  for (int u = 0; u < R; ++u) q[u] = Qh + (int64_t)min(i0 + u, g.N - 1) * g.d;

  // piece n of a thread: channels 2 sp, 2 sp + 1 of column sc + 16 n
  const int sp = tid % (KC / 2), sc = tid / (KC / 2);
  double2_a8 v[NP];
  auto request = [&](int c0) {  // (d is a multiple of 8; channels past it are not multiplied)
    const int c = c0 + 2 * sp < g.d ? c0 + 2 * sp : 0;
#pragma unroll
    for (int n = 0; n < NP; ++n)
      v[n] = *reinterpret_cast<const double2_a8*>(Kh + (int64_t)min(j0 + sc + 16 * n, g.N - 1) * g.d + c);
  };
  auto stage = [&](int buf) {
#pragma unroll
    for (int n = 0; n < NP; ++n) {
      ks[buf][2 * sp][sc + 16 * n] = v[n].x;
      ks[buf][2 * sp + 1][sc + 16 * n] = v[n].y;
    }
  };
  double acc[R] = {};
  request(0);
  stage(0);
  __syncthreads();
  for (int c0 = 0, buf = 0; c0 < g.d; c0 += KC, buf ^= 1) {
    const bool more = c0 + KC < g.d;
    if (more) request(c0 + KC);
    const int kc = min(KC, g.d - c0);
#pragma unroll 2
    for (int c = 0; c < kc; c += 4) {
      double qc[R][4];
#pragma unroll
      for (int u = 0; u < R; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) qc[u][e] = q[u][c0 + c + e];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double k = ks[buf][c + e][lane];
#pragma unroll
        for (int u = 0; u < R; ++u) acc[u] = __dadd_rn(acc[u], __dmul_rn(qc[u][e], k));
      }
    }
    if (more) stage(buf ^ 1);  // (its readers passed the barrier of the iteration before)
    __syncthreads();
  }
  const int j = j0 + lane;
#pragma unroll
  for (int u = 0; u < R; ++u)
    if (i0 + u < g.N && j < g.N) S[((int64_t)bh * g.N + i0 + u) * g.N + j] = __dmul_rn(acc[u], scale);
}

// Many tiles: 64 x 64 scores a workgroup, 4 x 4 a thread (rows i0 + 4 ti .., columns j0 + 4 tj ..), both operands in
// LDS: 4 + 4 reads for 16 multiply-adds a channel.  Nothing is requested ahead, so it takes enough workgroups on a
// CU to cover a stage, and channels enough to make stages long.
constexpr int kTile = 64, kTileKC = 16;
__global__ __launch_bounds__(256) void scores_tile_kernel(Geom g, const double* Qbar, const double* Kbar, double scale, double* S) {
  __shared__ __align__(16) double qs[kTileKC][kTile + 2];  // +2: conflict-free staging stores, rows stay 16-byte aligned
  __shared__ __align__(16) double ks[kTileKC][kTile + 2];
  const int bh = blockIdx.z;
  const int i0 = blockIdx.y * kTile, j0 = blockIdx.x * kTile;
  const int tid = threadIdx.x, ti = tid / 16, tj = tid % 16;
  const double* Qh = Qbar + (int64_t)bh * g.N * g.d;
  const double* Kh = Kbar + (int64_t)bh * g.N * g.d;
  double acc[4][4] = {};
  for (int c0 = 0; c0 < g.d; c0 += kTileKC) {
    __syncthreads();
    for (int e = tid; e < kTile * kTileKC; e += 256) {
      const int r = e / kTileKC, c = e % kTileKC;
      qs[c][r] = (i0 + r < g.N && c0 + c < g.d) ? Qh[(int64_t)(i0 + r) * g.d + c0 + c] : 0.0;
    }
    for (int e = tid; e < kTile * kTileKC; e += 256) {
      const int r = e / kTileKC, c = e % kTileKC;
      ks[c][r] = (j0 + r < g.N && c0 + c < g.d) ? Kh[(int64_t)(j0 + r) * g.d + c0 + c] : 0.0;
    }
    __syncthreads();
    const int kc = min(kTileKC, g.d - c0);
    for (int c = 0; c < kc; ++c) {
      double q[4], k[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        q[u] = qs[c][4 * ti + u];
        k[u] = ks[c][4 * tj + u];
      }
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[a][u] = __dadd_rn(acc[a][u], __dmul_rn(q[a], k[u]));
    }
  }
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = i0 + 4 * ti + a, j = j0 + 4 * tj + u;
      if (i < g.N && j < g.N) S[((int64_t)bh * g.N + i) * g.N + j] = __dmul_rn(acc[a][u], scale);
    }
}

template <int R>
static bool launch_scores(const Geom& g, const double* Qbar, const double* Kbar, double scale, double* S, int64_t least, hipStream_t st) {
  const dim3 grid((g.N + TJ - 1) / TJ, (g.N + 4 * R - 1) / (4 * R), g.B * g.H);
  if ((int64_t)grid.x * grid.y * grid.z < least) return false;
  hipLaunchKernelGGL(scores_kernel<R>, grid, dim3(256), 0, st, g, Qbar, Kbar, scale, S);
  return true;
}

// ---------------------------------------------------------------- 2. per-row selection
// Eq. 4 without a sort.  In the order (score descending, block id ascending) the selected set
// is a prefix, so it is fixed by the key of its last element.  Scores map to 64-bit integers
// that order the same way; with G(t) = sum of e_j over keys >= t (non-increasing in t) the
// last selected key is the largest t with G(t) >= p*Z.  It is found by bisection, keeping a
// bracket [lo, hi] with G(lo) >= p*Z > G(hi + 1) and the number of keys inside it, until one key is
// left.  The first kValueSteps pivots halve the bracket's range of scores, which are spread like the keys
// of a row are, about log2 N + 2 steps; bits would be bisected through sign and exponent first, which took
// about twice as many.  After that, and wherever the middle of two scores is no key inside the bracket
// (infinities), the pivot is the middle key, so the search ends whatever the scores are.
// More than one key left in a bracket of one value means equal scores: those are
// taken in ascending block id while the mass is short.  Sums run in a fixed order (per lane
// ascending, butterfly across lanes, wavefronts in order), so the result is reproducible (the number of wavefronts,
// and with it the order, depends on the number of blocks alone);
// it equals the sequential-prefix definition whenever no comparison is within rounding of a
// tie, which the callers' margin check establishes.
__device__ inline unsigned long long order_key(double s) {
  if (s == 0.0) s = 0.0;  // -0 and +0 compare equal
  const unsigned long long u = (unsigned long long)__double_as_longlong(s);
  return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}

__device__ inline double key_score(unsigned long long key) {  // the score of a key
  return __longlong_as_double((long long)((key >> 63) ? key ^ 0x8000000000000000ull : ~key));
}

// The value of lane ^ M where all lanes that differ from this one in higher bits below 64 only hold the same
// value, that is in a butterfly from 32 down to 1 (a rotation within 16 lanes then reaches the same value as
// the exchange).  Register exchanges instead of the LDS crossbar: a bisection step is one chain of them.
template <int M>
__device__ inline uint32_t butterfly(uint32_t v) {
  if constexpr (M == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return (threadIdx.x & 32) ? r[0] : r[1];
  } else if constexpr (M == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return (threadIdx.x & 16) ? r[0] : r[1];
  } else {  // row_ror:8, row_ror:4, quad_perm [2,3,0,1], quad_perm [1,0,3,2]
    constexpr int ctrl = M == 8 ? 0x128 : M == 4 ? 0x124 : M == 2 ? 0x4e : 0xb1;
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, 0xf, 0xf, true);
  }
}
template <int M>
__device__ inline unsigned long long butterfly(unsigned long long v) {
  return ((unsigned long long)butterfly<M>((uint32_t)(v >> 32)) << 32) | butterfly<M>((uint32_t)v);
}
template <int M>
__device__ inline double butterfly(double v) {
  return __longlong_as_double((long long)butterfly<M>((unsigned long long)__double_as_longlong(v)));
}
// the reduction of op over a wavefront in every lane, pairs in the order 32, 16, .., 1
template <typename T, typename Op>
__device__ inline T wave_reduce(T v, Op op) {
  v = op(v, butterfly<32>(v));
  v = op(v, butterfly<16>(v));
  v = op(v, butterfly<8>(v));
  v = op(v, butterfly<4>(v));
  v = op(v, butterfly<2>(v));
  return op(v, butterfly<1>(v));
}
__device__ inline double wave_sum(double v) {
  return wave_reduce(v, [](double a, double b) { return __dadd_rn(a, b); });
}
__device__ inline double wave_max(double v) {
  return wave_reduce(v, [](double a, double b) { return fmax(a, b); });
}
__device__ inline unsigned long long wave_max_key(unsigned long long v) {
  return wave_reduce(v, [](unsigned long long a, unsigned long long b) { return a > b ? a : b; });
}

// A chain of bisection steps bounds it (few rows) or the compares and masked additions of a step (many).
// Microseconds with bits for pivots, the LDS crossbar, up to 16 elements skipped by branches and four
// wavefronts a row above 1,024 blocks, and now: 576 rows of 48 blocks 16 and 8, 4,368 of 364 41 and 22,
// 44,000 of 1,100 1,271 and 276.
// MAXE: elements per thread, the next of the compiled numbers (elements past the row have the key 0 and no mass).
constexpr int kValueSteps = 24;
template <int NW, int MAXE>
__global__ __launch_bounds__(64 * NW) void row_select_kernel(Geom g, const double* S, double p, double zq,
                                                            uint32_t* mask, int32_t* cnt) {
  constexpr int NT = 64 * NW;
  extern __shared__ __align__(16) uint8_t smem[];
  unsigned long long* lkey = reinterpret_cast<unsigned long long*>(smem);  // [N], for the equal-score path
  __shared__ double red[NW];
  __shared__ int redc[NW];
  __shared__ unsigned long long rk[2][NW];
  __shared__ uint32_t bits[256];
  const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const double* s = S + (int64_t)row * g.N;
  const int W = (g.N + 31) / 32;

  auto block_sum = [&](double v) -> double {  // the same value in every thread
    v = wave_sum(v);
    if (NW == 1) return v;
    __syncthreads();
    if (lane == 0) red[wave] = v;
    __syncthreads();
    double t = red[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) t = __dadd_rn(t, red[w]);
    return t;
  };
  // both at once (one pair of barriers): the sum in the same order as block_sum
  auto block_sum_count = [&](double v, int c, double& vs, int& cs) {
    v = wave_sum(v);
    if (NW == 1) {
      vs = v;
      cs = c;
      return;
    }
    __syncthreads();
    if (lane == 0) {
      red[wave] = v;
      redc[wave] = c;
    }
    __syncthreads();
    double t = red[0];
    int tc = redc[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) {
      t = __dadd_rn(t, red[w]);
      tc += redc[w];
    }
    vs = t;
    cs = tc;
  };
  auto block_max = [&](double v) -> double {
    v = wave_max(v);
    if (NW == 1) return v;
    __syncthreads();
    if (lane == 0) red[wave] = v;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NW; ++w) v = fmax(v, red[w]);
    return v;
  };
  auto block_count = [&](int c) -> int {  // c is wave-uniform
    if (NW == 1) return c;
    __syncthreads();
    if (lane == 0) redc[wave] = c;
    __syncthreads();
    int t = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) t += redc[w];
    return t;
  };

  double sv[MAXE];
  double smin = INFINITY, smax = -INFINITY;
#pragma unroll
  for (int e = 0; e < MAXE; ++e) {
    const int j = e * NT + tid;
    sv[e] = j < g.N ? s[j] : -INFINITY;  // element e of a thread: j = e * NT + tid
    smax = fmax(smax, sv[e]);
    if (j < g.N) smin = fmin(smin, sv[e]);
  }
  smax = block_max(smax);
  smin = -block_max(-smin);
  for (int k = tid; k < 256; k += NT) bits[k] = 0u;

  unsigned long long key[MAXE];
  double ev[MAXE];
  double zl = 0.0;
  unsigned long long kmin = ~0ull, kmax = 0ull;
#pragma unroll
  for (int e = 0; e < MAXE; ++e) {
    const int j = e * NT + tid;
    const bool live = j < g.N;
    key[e] = live ? order_key(sv[e]) : 0ull;  // padding: below every real key, no mass
    ev[e] = live ? exp(sv[e] - smax) : 0.0;
    zl = __dadd_rn(zl, ev[e]);
    if (live) {
      lkey[j] = key[e];
      kmin = key[e] < kmin ? key[e] : kmin;
      kmax = key[e] > kmax ? key[e] : kmax;
    }
  }
  const double Z = block_sum(zl);
  // smallest and largest key of the row
  kmin = ~wave_max_key(~kmin);
  kmax = wave_max_key(kmax);
  if (NW > 1) {
    __syncthreads();
    if (lane == 0) { rk[0][wave] = kmin; rk[1][wave] = kmax; }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      kmin = rk[0][w] < kmin ? rk[0][w] : kmin;
      kmax = rk[1][w] > kmax ? rk[1][w] : kmax;
    }
  }
  auto count_where = [&](unsigned long long lo_incl, bool equal_only) -> int {  // keys >= lo (or == lo)
    int cl = 0;
#pragma unroll
    for (int e = 0; e < MAXE; ++e)
      cl += __popcll(__ballot(equal_only ? key[e] == lo_incl : key[e] >= lo_incl));
    return block_count(cl);
  };

  // The selection is "every key above `last`, plus the first `need` blocks (ascending id)
  // whose key equals `last`"; `tie` says that several blocks share that key.
  int kstar = g.N, need = 1;
  bool all = true, tie = false;
  unsigned long long last = 0ull;
  if (p < 1.0) {
    all = false;
    const double target = __dmul_rn(p, Z);
    unsigned long long lo = kmin, hi = kmax;
    double vlo = smin, vhi = smax;  // scores between which the bracket's keys lie
    int cnt_lo = g.N, cnt_hi = 0;   // keys >= lo; keys > hi
    for (int step = 0; cnt_lo - cnt_hi > 1 && lo < hi; ++step) {
      const double mid = 0.5 * vlo + 0.5 * vhi;
      unsigned long long cand = order_key(mid);
      if (step >= kValueSteps || !(cand > lo && cand <= hi)) {
        cand = lo + ((hi - lo) >> 1) + ((hi - lo) & 1ull);
        step = kValueSteps;  // (the scores no longer say where the bracket is)
      }
      double gl = 0.0;
      int cl = 0;
#pragma unroll
      for (int e = 0; e < MAXE; ++e) {
        const bool ge = key[e] >= cand;
        gl = __dadd_rn(gl, ge ? ev[e] : 0.0);
        cl += __popcll(__ballot(ge));
      }
      double G;
      int c;
      block_sum_count(gl, cl, G, c);
      if (G >= target) {
        lo = cand;
        vlo = mid;
        cnt_lo = c;
      } else {
        hi = cand - 1;
        vhi = mid;
        cnt_hi = c;
      }
    }
    // the keys still inside the bracket [lo, hi] are all equal (one key, unless scores tie exactly)
    tie = cnt_lo - cnt_hi > 1;
    if (tie) {  // equal scores: add them one at a time, as the sorted prefix would
      double gl = 0.0, el = 0.0;
#pragma unroll
      for (int e = 0; e < MAXE; ++e) {
        gl = __dadd_rn(gl, key[e] > lo ? ev[e] : 0.0);
        if (key[e] == lo) el = ev[e];
      }
      double c = block_sum(gl);
      el = block_max(el);  // the mass of one tied element (identical in all of them)
      const int tied = cnt_lo - cnt_hi;
      need = 0;
      do {
        c = __dadd_rn(c, el);
        ++need;
      } while (c < target && need < tied);
    }
    kstar = cnt_hi + need;
    // the last selected key: the one key value inside the bracket
    unsigned long long lk = 0ull;
#pragma unroll
    for (int e = 0; e < MAXE; ++e)
      if (key[e] >= lo && key[e] <= hi && key[e] > lk) lk = key[e];
    lk = wave_max_key(lk);
    if (NW > 1) {
      __syncthreads();
      if (lane == 0) rk[0][wave] = lk;
      __syncthreads();
#pragma unroll
      for (int w = 0; w < NW; ++w) lk = rk[0][w] > lk ? rk[0][w] : lk;
    }
    last = lk;
  }

  // Eq. 3 (statistical dynamic threshold): only blocks whose score reaches
  // tau = mean + std * zq are candidates; they are a prefix of the same order, so the filter
  // can only shorten the selection.  No candidate: the best block alone.
  if (zq == zq && zq != -INFINITY) {
    double sl = 0.0;
#pragma unroll
    for (int e = 0; e < MAXE; ++e)
      if (e * NT + tid < g.N) sl = __dadd_rn(sl, key_score(key[e]));
    const double mean = __ddiv_rn(block_sum(sl), (double)g.N);
    double dl = 0.0;
#pragma unroll
    for (int e = 0; e < MAXE; ++e)
      if (e * NT + tid < g.N) {
        const double dvn = __dadd_rn(key_score(key[e]), -mean);
        dl = __dadd_rn(dl, __dmul_rn(dvn, dvn));
      }
    const double var = g.N > 1 ? __ddiv_rn(block_sum(dl), (double)(g.N - 1)) : 0.0;
    const double tau = __dadd_rn(mean, __dmul_rn(__dsqrt_rn(var), zq));
    const unsigned long long ktau = order_key(tau);
    const int ncand = tau == tau ? count_where(ktau, false) : 0;
    if (ncand < kstar) {
      all = false;
      if (ncand >= 1) {
        kstar = ncand;
        last = ktau;  // "above last, or equal to it": every key >= ktau
        tie = false;
        need = 1;
      } else {
        kstar = 1;
        last = kmax;
        need = 1;
        tie = count_where(kmax, true) > 1;
      }
    }
  }

  if (!all) {
    if (NW > 1) __syncthreads();  // bits[] cleared by everyone
#pragma unroll
    for (int e = 0; e < MAXE; ++e) {
      const int j = e * NT + tid;
      if (j < g.N && (key[e] > last || (!tie && key[e] == last))) atomicOr(&bits[j >> 5], 1u << (j & 31));
    }
    if (tie && tid == 0) {  // equal scores: ascending block id, one thread (rare)
      int left = need;
      for (int j = 0; j < g.N && left > 0; ++j)
        if (lkey[j] == last) {
          atomicOr(&bits[j >> 5], 1u << (j & 31));
          --left;
        }
    }
  }
  __syncthreads();
  for (int w = tid; w < W; w += NT) {
    uint32_t v = bits[w];
    if (all) v = (w * 32 + 32 <= g.N) ? 0xffffffffu : ((1u << (g.N - w * 32)) - 1u);
    mask[(int64_t)row * W + w] = v;
  }
  if (tid == 0) cnt[row] = kstar;
}

// ---------------------------------------------------------------- 3. exclusive scan
// One workgroup, 4,096 counts a step: four a thread, a scan of the wavefront by lane shifts, one barrier for
// the sixteen totals (two sets in turn), the next counts requested ahead.  Bound by the latency of a step.
// 44,000 counts 72 -> 13 us, 4,368 in one step 5.2 -> 5.0 (each thread summed and wrote a run of its own before).
typedef int int4_a4 __attribute__((ext_vector_type(4), aligned(4)));
__global__ __launch_bounds__(1024) void scan_kernel(const int32_t* cnt, int n, int32_t* ptr, int64_t* total) {
  __shared__ int part[2][16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  auto counts = [&](int k) {
    int4_a4 v = {0, 0, 0, 0};
    if (k + 4 <= n) return *reinterpret_cast<const int4_a4*>(cnt + k);
#pragma unroll
    for (int e = 0; e < 3; ++e)
      if (k + e < n) v[e] = cnt[k + e];
    return v;
  };
  int carry = 0;
  int4_a4 next = counts(4 * tid);
  for (int base = 0, buf = 0; base < n; base += 4096, buf ^= 1) {
    const int k = base + 4 * tid;
    const int4_a4 v = next;
    next = counts(k + 4096);
    const int own = v.x + v.y + v.z + v.w;
    int incl = own;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int u = __shfl_up(incl, o);
      if (lane >= o) incl += u;
    }
    if (lane == 63) part[buf][wave] = incl;
    __syncthreads();
    int run = carry + incl - own;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
      const int t = part[buf][w];
      if (w < wave) run += t;
      carry += t;
    }
    const int4_a4 out = {run, run + v.x, run + v.x + v.y, run + v.x + v.y + v.z};
    if (k + 4 <= n) {
      *reinterpret_cast<int4_a4*>(ptr + k) = out;
    } else {
#pragma unroll
      for (int e = 0; e < 3; ++e)
        if (k + e < n) ptr[k + e] = out[e];
    }
  }
  if (tid == 0) {
    ptr[n] = carry;
    if (total) *total = carry;
  }
}

// ---------------------------------------------------------------- 4. mask -> ascending ids
__global__ __launch_bounds__(256) void expand_kernel(Geom g, const uint32_t* mask, const int32_t* ptr,
                                                     int32_t* out) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= g.rows) return;
  const int W = (g.N + 31) / 32;
  int base = ptr[row];
  for (int w0 = 0; w0 < W; w0 += 64) {
    const int w = w0 + lane;
    uint32_t word = w < W ? mask[(int64_t)row * W + w] : 0u;
    const int pc = __popc(word);
    int incl = pc;
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(incl, o);
      if (lane >= o) incl += v;
    }
    int pos = base + incl - pc;
    while (word) {
      const int b = __ffs(word) - 1;
      out[pos++] = w * 32 + b;
      word &= word - 1;
    }
    base += __shfl(incl, 63);
  }
}

// ---------------------------------------------------------------- 5-7. transpose
// One wavefront per (head, kCols KV blocks).  FILL=false counts the listing query
// blocks of each column; FILL=true writes them, ascending, at k2q_ptr[column].  A wavefront is one chain over
// the head's rows, so a few columns each (whole words cost 32 steps a chain and left most SIMDs idle), counts
// and cursors in scalar registers.
// A word of 32 columns a wavefront and now, microseconds: 12 heads of 364 blocks count 9.2 and 5.4, fill 17 and 5.5.
constexpr int kCols = 8;
template <bool FILL>
__global__ __launch_bounds__(256) void transpose_kernel(Geom g, const uint32_t* mask, int32_t* kcnt,
                                                        const int32_t* kptr, int32_t* kidx) {
  const int lane = threadIdx.x & 63;
  const int W = (g.N + 31) / 32, G = (g.N + kCols - 1) / kCols;  // words of a row, groups of columns
  const int unit = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (unit >= g.B * g.H * G) return;
  const int bh = unit / G, c0 = (unit % G) * kCols;
  const uint32_t* word = mask + (int64_t)bh * g.N * W + c0 / 32;
  const int shift = c0 % 32;
  int acc[kCols];  // running count (or write cursor) of column c0 + b, the same in every lane
#pragma unroll
  for (int b = 0; b < kCols; ++b) acc[b] = FILL ? kptr[(int64_t)bh * g.N + min(c0 + b, g.N - 1)] : 0;
  const unsigned long long lt = (1ull << lane) - 1ull;
  auto bits = [&](int i0) -> uint32_t {
    const int i = i0 + lane;
    return i < g.N ? word[(int64_t)i * W] >> shift : 0u;
  };
  uint32_t next = bits(0);
  for (int i0 = 0; i0 < g.N; i0 += 64) {
    const uint32_t now = next;
    next = bits(i0 + 64);
#pragma unroll
    for (int b = 0; b < kCols; ++b) {
      const bool set = (now >> b) & 1u;  // (bits past the last column are zero)
      const unsigned long long m = __ballot(set);
      if (FILL && set) kidx[acc[b] + __popcll(m & lt)] = i0 + lane;
      acc[b] += __popcll(m);
    }
  }
  if (!FILL && lane == 0) {
#pragma unroll
    for (int b = 0; b < kCols; ++b)
      if (c0 + b < g.N) kcnt[(int64_t)bh * g.N + c0 + b] = acc[b];
  }
}

// ---------------------------------------------------------------- 3-7 in one launch
// Few rows: the five launches are a chain of latencies (3 to 5 us each), so one workgroup does all of it with the
// masks in LDS.  Expansion: a wavefront per row, a column a lane, ids stored side by side; transpose as above.
// One CU does the work, so the line lies low.  Microseconds, the launches (each with a gap of a few more ahead of it
// in a short program) and one: 32 rows of 16 blocks, both directions, 14 and 4.9; 576 of 48, q2k alone, 8 and 9.8;
// 756 of 126, both, 24 and 40.  Whole selections of 64 blocks, d = 64: 256 rows 25.0 and 21.7 (q2k alone 16.6 and
// 16.4), 384 rows 26 and 26, 512 rows 25 and 30.
constexpr int kFewRows = 256, kFewBlocks = 64;
__global__ __launch_bounds__(1024) void lists_kernel(Geom g, const uint32_t* mask, const int32_t* cnt, int32_t* q2k_ptr, int32_t* q2k_idx,
                                                     int32_t* k2q_ptr, int32_t* k2q_idx, int64_t* total) {
  __shared__ uint32_t bits[kFewRows * (kFewBlocks / 32)];
  __shared__ int start[kFewRows], count[kFewRows], part[2][16];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int W = (g.N + 31) / 32;
  const unsigned long long lt = (1ull << lane) - 1ull;
  // exclusive scan of one value a thread; start[], ptr[0 .. rows]; a barrier inside and one at the end
  auto scan = [&](int own, int (&tot)[16], int32_t* ptr, int64_t* sum) {
    int incl = own;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int u = __shfl_up(incl, o);
      if (lane >= o) incl += u;
    }
    if (lane == 63) tot[wave] = incl;
    __syncthreads();
    int run = incl - own, all = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
      if (w < wave) run += tot[w];
      all += tot[w];
    }
    if (tid < g.rows) start[tid] = ptr[tid] = run;
    if (tid == 0) {
      ptr[g.rows] = all;
      if (sum) *sum = all;
    }
    __syncthreads();
  };
  for (int k = tid; k < g.rows * W; k += 1024) bits[k] = mask[k];
  scan(tid < g.rows ? cnt[tid] : 0, part[0], q2k_ptr, total);
  for (int row = wave; row < g.rows; row += 16) {
    int pos = start[row];
    for (int c0 = 0; c0 < g.N; c0 += 64) {
      const int c = c0 + lane;
      const bool set = c < g.N && (bits[row * W + min(c >> 5, W - 1)] >> (c & 31) & 1u);
      const unsigned long long m = __ballot(set);
      if (set) q2k_idx[pos + __popcll(m & lt)] = c;
      pos += __popcll(m);
    }
  }
  if (!k2q_ptr) return;
  const int G = (g.N + kCols - 1) / kCols, units = g.B * g.H * G;
  for (int fill = 0; fill < 2; ++fill) {
    for (int unit = wave; unit < units; unit += 16) {
      const int bh = unit / G, c0 = (unit - bh * G) * kCols;
      const int head = bh * g.N, shift = c0 % 32;
      int acc[kCols];
#pragma unroll
      for (int b = 0; b < kCols; ++b) acc[b] = fill ? start[head + min(c0 + b, g.N - 1)] : 0;
      for (int i0 = 0; i0 < g.N; i0 += 64) {
        const int i = i0 + lane;
        const uint32_t now = i < g.N ? bits[(head + i) * W + c0 / 32] >> shift : 0u;
#pragma unroll
        for (int b = 0; b < kCols; ++b) {
          const bool set = (now >> b) & 1u;  // (bits past the last column are zero)
          const unsigned long long m = __ballot(set);
          if (fill && set) k2q_idx[acc[b] + __popcll(m & lt)] = i;
          acc[b] += __popcll(m);
        }
      }
      if (!fill && lane == 0) {
#pragma unroll
        for (int b = 0; b < kCols; ++b)
          if (c0 + b < g.N) count[head + c0 + b] = acc[b];
      }
    }
    if (fill) return;
    __syncthreads();  // counts written, start[] read by everyone
    scan(tid < g.rows ? count[tid] : 0, part[1], k2q_ptr, nullptr);
  }
}

// One wavefront per row up to 1,536 blocks (24 elements a lane), four (and two barriers a bisection step) above.  Whole
// selections, d = 64, us, one wavefront a row and four: 1,028 blocks, 1 head 68 and 69, 40 heads 681 and 963; 1,536
// blocks 95 and 100, 1,417 and 1,781.
template <int NW, int MAXE, int... MORE>
static void launch_row_select_of(const Geom& g, double p, double zq, const SelectWs& w, hipStream_t st) {
  if constexpr (sizeof...(MORE) > 0)
    if (g.N > 64 * NW * MAXE) return launch_row_select_of<NW, MORE...>(g, p, zq, w, st);
  hipLaunchKernelGGL((row_select_kernel<NW, MAXE>), dim3(g.rows), dim3(64 * NW), g.N * sizeof(unsigned long long), st, g, w.scores, p, zq, w.mask, w.cnt);
}
static void launch_row_select(const Geom& g, double p, double zq, const SelectWs& w, hipStream_t st) {
  if (g.N <= 1536) launch_row_select_of<1, 1, 2, 4, 6, 8, 12, 16, 20, 24>(g, p, zq, w, st);
  else launch_row_select_of<4, 8, 12, 16, 32>(g, p, zq, w, st);
}

// Tiles from 4,608 of them (4.5 rounds of four a CU) at 128 channels and from 5,632 at 64, never below.
// Microseconds of the whole selection, wavefront rows and tiles:
//   d = 256: 12 heads of 1,100 blocks (3,888 tiles) 492 and 507, 40 of 700 (4,840) 732 and 677, 12 of 2,520 (19,200) 2,810 and 2,573
//   d = 128: 12 of 1,100 271 and 276, 12 of 1,280 (4,800) 413 and 414, 40 of 700 462 and 444, 40 of 1,100 (12,960) 1,129 and 1,024,
//            12 of 2,520 1,882 and 1,746
//   d = 64:  80 of 512 (5,120) 351 and 359, 12 of 1,400 (5,808) 384 and 383, 24 of 1,100 (7,776) 506 and 477, 12 of 2,520 1,456 and 1,384
//   d = 32:  40 of 1,100 668 and 650, 12 of 2,048 788 and 811
static void launch_block_logits(const Geom& g, const double* Qbar, const double* Kbar, double scale, double* S, hipStream_t st) {
  const int n = (g.N + kTile - 1) / kTile;
  if (g.d >= 64 && (int64_t)n * n * g.B * g.H >= (g.d >= 128 ? 4608 : 5632)) {
    hipLaunchKernelGGL(scores_tile_kernel, dim3(n, n, g.B * g.H), dim3(256), 0, st, g, Qbar, Kbar, scale, S);
    return;
  }
  // the most rows a wavefront that still leave three workgroups a CU (eight rows) or two (four): four fit, and hide
  // the scalar loads
  launch_scores<8>(g, Qbar, Kbar, scale, S, 768, st) || launch_scores<4>(g, Qbar, Kbar, scale, S, 512, st) ||
      launch_scores<2>(g, Qbar, Kbar, scale, S, 0, st);
}

int launch_select(const Geom& g, const double* Qbar, const double* Kbar, double threshold, double stat_z,
                  double score_scale, int32_t* q2k_ptr, int32_t* q2k_idx, int32_t* k2q_ptr,
                  int32_t* k2q_idx, int64_t* nnz_dev, void* ws, hipStream_t st) {
  SelectWs w = carve(g, ws);
  const int BH = g.B * g.H;
  const size_t lds = (size_t)g.N * sizeof(unsigned long long);  // <= 64 KB
  if (g.N > 4096)
    if (int rc = allow_dynamic_lds<row_select_kernel<4, 32>>(lds)) return rc;
  launch_block_logits(g, Qbar, Kbar, score_scale, w.scores, st);
  launch_row_select(g, threshold, stat_z, w, st);
  if (g.rows <= kFewRows && g.N <= kFewBlocks) {
    hipLaunchKernelGGL(lists_kernel, dim3(1), dim3(1024), 0, st, g, w.mask, w.cnt, q2k_ptr, q2k_idx, k2q_ptr, k2q_idx, nnz_dev);
    return check_launch();
  }
  hipLaunchKernelGGL(scan_kernel, dim3(1), dim3(1024), 0, st, w.cnt, g.rows, q2k_ptr, nnz_dev);
  hipLaunchKernelGGL(expand_kernel, dim3((g.rows + 3) / 4), dim3(256), 0, st, g, w.mask, q2k_ptr, q2k_idx);
  if (k2q_ptr) {
    const int units = BH * ((g.N + kCols - 1) / kCols);
    hipLaunchKernelGGL(transpose_kernel<false>, dim3((units + 3) / 4), dim3(256), 0, st, g, w.mask, w.kcnt,
                       (const int32_t*)nullptr, (int32_t*)nullptr);
    hipLaunchKernelGGL(scan_kernel, dim3(1), dim3(1024), 0, st, w.kcnt, g.rows, k2q_ptr, (int64_t*)nullptr);
    hipLaunchKernelGGL(transpose_kernel<true>, dim3((units + 3) / 4), dim3(256), 0, st, g, w.mask, w.kcnt,
                       k2q_ptr, k2q_idx);
  }
  return check_launch();
}

}  // namespace bsa
