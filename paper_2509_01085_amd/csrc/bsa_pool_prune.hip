// Streaming kernels of the index-preparation stage: block mean pooling (Sec. 3.2.3) and
// query pruning by cosine similarity to the block center (Sec. 3.2.2, Eq. 2).
//
// Both are one pass over a [B,H,L,d] tensor and are bound by HBM bandwidth: a wavefront
// owns one 3D block (Bk token rows in Cw-token runs of contiguous memory) and does the fp64
// decision arithmetic on it.
//
// Bit-exactness contract with any other implementation of the same definition: sums run
// in ascending index order (tokens for pooling, channels for dot products) in fp64.  The
// inputs are fp32 or bf16, so every product of two inputs is exact in fp64 and a fused
// multiply-add rounds exactly like multiply-then-add; cos = dot / sqrt(|a|^2 * |c|^2) uses
// IEEE fp64 multiply, sqrt and divide.
#include <math.h>

#include "bsa_common.h"

namespace bsa {

// One wavefront per 3D block in both kernels, no workgroup barriers: many independent
// wavefronts per CU keep enough loads in flight to stream at HBM rate.

constexpr int kWaves = 4;  // wavefronts (= blocks) per workgroup

template <int ES>
__device__ inline void unpack(uint32_t w, double& lo, double& hi) {  // ES == 2: two bf16 channels of a word
  lo = (double)__uint_as_float(w << 16);
  hi = (double)__uint_as_float(w & 0xffff0000u);
}

// ------------------------------------------------------------------------------ pooling
// Lane l owns WL neighbouring 32-bit words of a token row (two bf16 channels or one fp32 channel each), the
// smallest WL with which 64 lanes cover the row (a second pass above 128 words): every load instruction of the
// wavefront reads one token's row segment, contiguous in memory, and the per-channel sums run over the tokens in
// ascending intra-block id, in registers.  No LDS but the table of row offsets.  Large grids are bound by HBM, small
// ones by the latency of a batch of loads: half a 64-token block at once, none of them behind a condition.
// Sixteen conditional loads a batch and one word a lane before, and now, microseconds: 3,072 tokens, 12 heads,
// d = 128, fp32 44 and 7.0, bf16 8.5 and 5.1; 23,296 tokens, bf16, 14.0 and 13.9 (5.1 TB/s).
// A batch past the end of a block reads its last row again, so it is no longer than short blocks: 8, 16 or 32 rows.
// 8 heads of 8,192 blocks, d = 128, in batches of 32 and now: fp32 1 token 81 and 31, 8 tokens 97 and 55, 16 tokens 110
// and 109; bf16 33 and 25, 35 and 32, 58 and 58.
template <int WL>
struct Words {
  typedef uint32_t type __attribute__((ext_vector_type(WL), aligned(4)));
};
// TB: token rows loaded ahead of the additions, the smallest that holds a block, or 32
template <int ES, int WL, int TB>
__global__ __launch_bounds__(64 * kWaves) void pool_kernel(Geom g, const uint8_t* X, double* Xbar) {
  constexpr int CW = 4 / ES;  // channels of a word
  typedef typename Words<WL>::type words_t;
  __shared__ uint32_t off[256];  // row offsets in words
  const int words = g.d * ES / 4;
  for (int t = threadIdx.x; t < g.Bk; t += 64 * kWaves) off[t] = (uint32_t)intra_offset(g, t) * (uint32_t)words;
  __syncthreads();  // the only workgroup barrier
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * kWaves + (threadIdx.x >> 6);  // (b*H + h)*N + i
  if (row >= g.rows) return;
  const int64_t bh = row / g.N;
  const int i = (int)(row % g.N);
  const uint32_t* base = reinterpret_cast<const uint32_t*>(X) + (bh * g.L + block_origin(g, i)) * (int64_t)words;
#pragma unroll 1
  for (int w0 = 0; w0 < words; w0 += 64 * WL) {
    const int w = w0 + WL * lane;
    const bool live = w < words;  // (words is a multiple of 4)
    const uint32_t* col = base + (live ? w : 0);
    double acc[WL * CW] = {};
    auto add = [&](words_t v) {  // ascending intra-block id
#pragma unroll
      for (int k = 0; k < WL; ++k) {
        uint32_t x;
        if constexpr (WL == 1) x = v[0]; else x = v[k];
        if constexpr (ES == 4) {
          acc[k] = __dadd_rn(acc[k], (double)__uint_as_float(x));
        } else {
          double lo, hi;
          unpack<ES>(x, lo, hi);
          acc[2 * k] = __dadd_rn(acc[2 * k], lo);
          acc[2 * k + 1] = __dadd_rn(acc[2 * k + 1], hi);
        }
      }
    };
    for (int r0 = 0; r0 < g.Bk; r0 += TB) {
      words_t v[TB];
#pragma unroll
      for (int u = 0; u < TB; ++u) v[u] = *reinterpret_cast<const words_t*>(col + off[min(r0 + u, g.Bk - 1)]);
      if (r0 + TB <= g.Bk) {
#pragma unroll
        for (int u = 0; u < TB; ++u) add(v[u]);
      } else {
#pragma unroll
        for (int u = 0; u < TB; ++u)
          if (r0 + u < g.Bk) add(v[u]);
      }
    }
    if (live) {
      const double bk = (double)g.Bk;
#pragma unroll
      for (int k = 0; k < WL * CW; ++k) Xbar[row * g.d + CW * w + k] = __ddiv_rn(acc[k], bk);
    }
  }
}

// ------------------------------------------------------------------------------ pruning
// Lane t owns token t of the block (Bk > 64: several passes).  The token rows pass through a
// per-wavefront LDS tile in groups of four sixteen-byte chunks: loaded row-contiguous (four lanes
// a row), read back one row per lane; the dot product with the center of the token's
// window and the squared norms accumulate over the channels in ascending order across the
// groups.  Four groups are in flight in registers, so a wavefront waits for memory once per 256 bytes of a
// row (a small grid is bound by that latency), and 5 KB of tile a wavefront let four of them sit on a SIMD instead of three
// (a large one is bound by the loads in flight and the fp64 rate).
// Ranking and quota are per window (Sec. 3.2.2, "Critical Token"); one window per
// block is the single-center method.
// Eight chunks a group, none requested ahead, the center's norm in every lane, before, and now, microseconds (bf16,
// d = 128, 64 tokens a block): 576 blocks 16.4 and 9.8, 4,368 41 and 22, 44,000 340 and 151; fp32, 576 blocks 26 and 10.
constexpr int kGroup = 4;                          // chunks of a row staged at a time
constexpr int kRowStride = kGroup * 16 + 16;       // LDS bytes per staged row (16 lanes' chunks take all banks)
constexpr int kTileBytes = 64 * kRowStride;

__device__ inline void wave_lds_sync() {  // LDS written by other lanes of this wavefront becomes readable
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// MAXB: the largest block (LDS per token)
// (four wavefronts a SIMD are what the sixteen loads leave registers for)
template <int ES, int MAXB>
__global__ __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(4, 4))) void prune_kernel(Geom g, const uint8_t* Q, int kw,
                                                           int32_t* keep_idx) {
  __shared__ __align__(16) uint8_t tiles[kWaves][kTileBytes];
  __shared__ __align__(16) double cosv[kWaves][MAXB];
  __shared__ int koff[MAXB];
  __shared__ short wid[MAXB];   // window of every intra-block token
  __shared__ short wcen[MAXB];  // critical token of that window (intra-block id)
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int t = threadIdx.x; t < g.Bk; t += 64 * kWaves) {
    koff[t] = intra_offset(g, t);
    const int w = window_of(g, t);
    wid[t] = (short)w;
    wcen[t] = (short)window_center(g, w);
  }
  __syncthreads();  // the only workgroup barrier; wavefronts are independent from here on
  const int64_t row = (int64_t)blockIdx.x * kWaves + wave;
  if (row >= g.rows) return;
  const int64_t bh = row / g.N;
  const int i = (int)(row % g.N);
  const int row_bytes = g.d * ES, cpr = row_bytes / 16, groups = (cpr + kGroup - 1) / kGroup;
  const int n_keep = kw * g.nwin;
  const uint8_t* base = Q + (bh * g.L + block_origin(g, i)) * (int64_t)row_bytes;
  uint8_t* tile = tiles[wave];

  for (int t0 = 0; t0 < g.Bk; t0 += 64) {
    const int nt = min(64, g.Bk - t0);
    const int cen = wcen[min(t0 + lane, g.Bk - 1)];  // this lane's window center
    const bool cen_staged = cen >= t0 && cen < t0 + nt;  // its row is part of this pass's tile
    const bool all_staged = __all(cen_staged);
    // load n of a group: chunk q of row (lane >> 2) + 16 n (rows and chunks past the end repeat the last)
    const int q = lane & 3;
    const uint8_t* src[kGroup];
#pragma unroll
    for (int n = 0; n < kGroup; ++n) src[n] = base + (int64_t)koff[t0 + min((lane >> 2) + 16 * n, nt - 1)] * row_bytes;
    typedef uint32_t words4 __attribute__((ext_vector_type(4)));
    auto request = [&](int grp, words4 (&v)[kGroup]) {
      const int c = min(grp * kGroup + q, cpr - 1);
#pragma unroll
      for (int n = 0; n < kGroup; ++n) v[n] = *reinterpret_cast<const words4*>(src[n] + 16 * c);
    };
    double dot = 0.0, na2 = 0.0, nc2 = 0.0;  // <q, q_c>, |q|^2, |q_c|^2: channels ascending
    auto chunk = [&](const uint4& xv, const uint4& cv, bool norm_c) {
      const uint32_t xw[4] = {xv.x, xv.y, xv.z, xv.w}, cw[4] = {cv.x, cv.y, cv.z, cv.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        double x[2], c[2];
        if (ES == 4) {
          x[0] = (double)__uint_as_float(xw[e]);
          c[0] = (double)__uint_as_float(cw[e]);
        } else {
          unpack<ES>(xw[e], x[0], x[1]);
          unpack<ES>(cw[e], c[0], c[1]);
        }
#pragma unroll
        for (int h = 0; h < 4 / ES; ++h) {
          dot = fma(x[h], c[h], dot);
          na2 = fma(x[h], x[h], na2);
          if (norm_c) nc2 = fma(c[h], c[h], nc2);
        }
      }
    };
    auto multiply = [&](int grp, const words4 (&v)[kGroup]) {
      if (grp >= groups) return;
      wave_lds_sync();  // everyone is done reading the previous group
#pragma unroll
      for (int n = 0; n < kGroup; ++n)
        *reinterpret_cast<words4*>(tile + ((lane >> 2) + 16 * n) * kRowStride + 16 * q) = v[n];
      wave_lds_sync();
      const int nq = min(kGroup, cpr - grp * kGroup);
      const uint8_t* own = tile + lane * kRowStride;
      if (all_staged) {  // the center's norm is that of its own lane
        const uint8_t* cr = tile + (cen - t0) * kRowStride;
        for (int k = 0; k < nq; ++k)
          chunk(*reinterpret_cast<const uint4*>(own + 16 * k), *reinterpret_cast<const uint4*>(cr + 16 * k), false);
      } else {
        for (int k = 0; k < nq; ++k) {
          const uint4 cv = cen_staged ? *reinterpret_cast<const uint4*>(tile + (cen - t0) * kRowStride + 16 * k)
                                      : *reinterpret_cast<const uint4*>(base + (int64_t)koff[cen] * row_bytes + 16 * (grp * kGroup + k));
          chunk(*reinterpret_cast<const uint4*>(own + 16 * k), cv, true);
        }
      }
    };
    for (int g0 = 0; g0 < groups; g0 += 4) {
      words4 v0[kGroup], v1[kGroup], v2[kGroup], v3[kGroup];
      request(g0, v0);  // (no conditions: the compiler would wait for a load at the end of one)
      request(g0 + 1, v1);
      request(g0 + 2, v2);
      request(g0 + 3, v3);
      multiply(g0, v0);
      multiply(g0 + 1, v1);
      multiply(g0 + 2, v2);
      multiply(g0 + 3, v3);
    }
    if (all_staged) nc2 = __shfl(na2, cen - t0);
    if (lane < nt) {
      const double den = __dsqrt_rn(__dmul_rn(na2, nc2));
      // A center takes no part in the ranking: NaN is ordered before nothing.  Any other token has to have a
      // place, or more than the quota would be kept: inf / inf (an infinity in Q) ranks last, by id.
      double c = NAN;
      if (t0 + lane != cen) c = fmin(den > 0.0 ? __ddiv_rn(dot, den) : 0.0, (double)INFINITY);  // (infinity for NaN)
      cosv[wave][t0 + lane] = c;
    }
  }
  wave_lds_sync();

  int base_pos = 0;  // retained tokens with a smaller id, over the passes so far
  for (int t0 = 0; t0 < g.Bk; t0 += 64) {
    const int t = t0 + lane;
    bool keep = false;
    if (t < g.Bk) {
      const int w = wid[t];
      const double ct = cosv[wave][t];
      int rank = 0;  // tokens of the window (center excluded) ordered before t: smaller cosine, then smaller id
#pragma unroll 8
      for (int u = 0; u < g.Bk; ++u) {
        const double cu = cosv[wave][u];
        rank += (wid[u] == w) & ((cu < ct) | ((cu == ct) & (u < t)));
      }
      keep = t == wcen[t] || rank < kw - 1;
    }
    const unsigned long long m = __ballot(keep);
    if (keep) keep_idx[row * n_keep + base_pos + __popcll(m & ((1ull << lane) - 1ull))] = t;
    base_pos += __popcll(m);
  }
}

template <int ES, int WL>
static void launch_pool_of(const Geom& g, const uint8_t* x, double* Xbar, hipStream_t st) {
  const dim3 grid((g.rows + kWaves - 1) / kWaves), block(64 * kWaves);
  if (g.Bk <= 8) hipLaunchKernelGGL((pool_kernel<ES, WL, 8>), grid, block, 0, st, g, x, Xbar);
  else if (g.Bk <= 16) hipLaunchKernelGGL((pool_kernel<ES, WL, 16>), grid, block, 0, st, g, x, Xbar);
  else hipLaunchKernelGGL((pool_kernel<ES, WL, 32>), grid, block, 0, st, g, x, Xbar);
}

int launch_pool(const Geom& g, int dtype, const void* X, double* Xbar, hipStream_t st) {
  const uint8_t* x = static_cast<const uint8_t*>(X);
  if (dtype == BSA_F32) {
    if (g.d > 64) launch_pool_of<4, 2>(g, x, Xbar, st);
    else launch_pool_of<4, 1>(g, x, Xbar, st);
  } else {
    if (g.d > 128) launch_pool_of<2, 2>(g, x, Xbar, st);
    else launch_pool_of<2, 1>(g, x, Xbar, st);
  }
  return check_launch();
}

int launch_prune(const Geom& g, int dtype, const void* Q, int window_quota, int32_t* keep_idx, hipStream_t st) {
  const uint8_t* q = static_cast<const uint8_t*>(Q);
  const dim3 grid((g.rows + kWaves - 1) / kWaves), block(64 * kWaves);
  const bool small = g.Bk <= 64;
  if (dtype == BSA_F32) {
    if (small) hipLaunchKernelGGL((prune_kernel<4, 64>), grid, block, 0, st, g, q, window_quota, keep_idx);
    else hipLaunchKernelGGL((prune_kernel<4, 256>), grid, block, 0, st, g, q, window_quota, keep_idx);
  } else {
    if (small) hipLaunchKernelGGL((prune_kernel<2, 64>), grid, block, 0, st, g, q, window_quota, keep_idx);
    else hipLaunchKernelGGL((prune_kernel<2, 256>), grid, block, 0, st, g, q, window_quota, keep_idx);
  }
  return check_launch();
}

}  // namespace bsa
