// Shape-generic sparse attention forward / backward (Eq. 5 with token filling, and its backward
// with the index sets held constant) on the fp32 matrix cores: true-fp32 inputs of any supported
// shape, and bf16 inputs of the shapes that the bf16 kernels do not cover (sums and probabilities
// stay fp32; where a product has a bf16 operand it runs on the bf16 instruction without loss, below).
//
// Instruction: v_mfma_f32_16x16x4_f32, D[16x16] += A[16x4] B[4x16]; lane l, i = l % 16, g = l / 16:
//   A: row i, k = g      B: column i, k = g      D: column i, rows 4 g + r in register r = 0..3
// Every product is an fp32 fused multiply-add, so the arithmetic is that of a vector-ALU kernel at
// four times its rate (64 flop per cycle and SIMD).  At that rate one operand register lasts 32
// cycles, so operands come straight from global memory (L1 / L2) in 16-byte loads and the kernels
// need neither LDS tiles nor barriers in their loops: the wavefronts of a workgroup take the
// entries of a list in turn, each with accumulators of its own, and these are summed once at the
// end, in a fixed order.
//
// Operand loads.  A contraction over channels may take them in any order that both operands
// share: step (s, e) lets lane group g supply channel 16 s + 4 g + e, so four steps are one
// 16-byte load of a row (row_frags).  A contraction over rows needs channels on the A row index:
// tile e of a 64-channel batch takes channel 64 b + 4 i + e as its row i, again one 16-byte load
// per lane and row (col_frags), and the D registers r, e then hold 16 consecutive channels.
// Register r of a D tile is the B operand of the row contraction as it stands (k slot g = row
// 4 g + r), so probabilities never leave their registers.
//
// Measured on a 3,072-token, 12-head fp32 layer (d = 128, half of the queries retained): forward
// 0.36 ms, dQ 0.48, dK/dV 0.72 against 2.50, 4.23 and 15.5 ms of the vector-ALU kernels before.
#include <math.h>

#include "bsa_common.h"

namespace bsa {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) short s16x4;

constexpr float kLog2e = 1.4426950408889634f;

// Backward workspace, one entry per retained row, rows of a block padded to a multiple of 16
struct GenericWs {
  float* g;      // [rows][nkp][d]  upstream gradient with the fill copies folded in
  float* lse2;   // [rows][nkp]     log-sum-exp in the exp2 domain, +inf on padding rows (P = 0)
  float* delta;  // [rows][nkp]     <g, o>
  int* tok;      // [rows][nkp]     token of the row
  int nkp;
  size_t bytes;
};
static GenericWs carve(const Geom& g, int n_keep, void* base) {
  GenericWs w;
  uint8_t* p = static_cast<uint8_t*>(base);
  w.nkp = (n_keep + 15) & ~15;
  const size_t n = (size_t)g.rows * w.nkp;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    uint8_t* q = p + off;
    off += (bytes + 255) & ~(size_t)255;
    return q;
  };
  w.g = reinterpret_cast<float*>(take(n * g.d * 4));
  w.lse2 = reinterpret_cast<float*>(take(n * 4));
  w.delta = reinterpret_cast<float*>(take(n * 4));
  w.tok = reinterpret_cast<int*>(take(n * 4));
  w.bytes = off;
  return w;
}
size_t bwd_workspace_generic(const Geom& g, int n_keep) { return carve(g, n_keep, nullptr).bytes; }

__device__ inline f32x4 mfma4(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// maximum / sum over the four lanes l, l ^ 16, l ^ 32, l ^ 48
__device__ inline float quad_max(float v) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ inline float quad_sum(float v) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ inline f32x4 load4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
__device__ inline f32x4 load4(const uint16_t* p) {
  const u32x2 v = *reinterpret_cast<const u32x2*>(p);
  return f32x4{__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u), __uint_as_float(v.y << 16),
               __uint_as_float(v.y & 0xffff0000u)};
}
__device__ inline f32x2 load2(const float* p) { return *reinterpret_cast<const f32x2*>(p); }
__device__ inline f32x2 load2(const uint16_t* p) {
  const uint32_t v = *reinterpret_cast<const uint32_t*>(p);
  return f32x2{__uint_as_float(v << 16), __uint_as_float(v & 0xffff0000u)};
}
__device__ inline void store4(float* p, f32x4 v) { *reinterpret_cast<f32x4*>(p) = v; }
__device__ inline void store4(uint16_t* p, f32x4 v) {
  u32x2 o;
  o.x = (uint32_t)f32_to_bf16(v[0]) | ((uint32_t)f32_to_bf16(v[1]) << 16);
  o.y = (uint32_t)f32_to_bf16(v[2]) | ((uint32_t)f32_to_bf16(v[3]) << 16);
  *reinterpret_cast<u32x2*>(p) = o;
}

// DS = number of 16-channel groups the kernel is compiled for (16 DS >= d).  Channels d .. 16 DS - 1
// are read from a clamped address; a channel contraction zeroes them in both operands (the data there
// may be infinite, and 0 * inf is not 0), a row contraction produces channels that are not stored.
__device__ inline int chan_or0(int ch, int d) { return ch < d ? ch : 0; }

// the smallest head dimension that takes DS groups: channels below it need no check
template <int DS>
constexpr int kMinD = DS == 2 ? 8 : DS == 4 ? 40 : DS == 5 ? 72 : DS == 6 ? 88 : DS == 8 ? 104 : DS == 12 ? 136 : 200;

// A or B operand of a channel contraction: this lane's row, DS loads of four channels.  FULL: d == 16 DS
template <int DS, bool FULL = false, typename T>
__device__ inline void row_frags(const T* row, int g, int d, f32x4 (&f)[DS]) {
#pragma unroll
  for (int s = 0; s < DS; ++s) {
    const int ch = 16 * s + 4 * g;
    f[s] = load4(row + chan_or0(ch, d));
    if (!FULL && 16 * s + 16 > kMinD<DS> && ch >= d) f[s] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
}

// A operand of a row contraction: channel tiles 0..DS-1 of this lane's row (k slot g), row index i.
// Full batches of four tiles by 16-byte loads, the remaining one to three tiles by 8 and 4.
template <int DS, typename T>
__device__ inline void col_frags(const T* row, int i, int d, float (&f)[DS]) {
  constexpr int NB = DS / 4, REM = DS % 4;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const f32x4 v = load4(row + chan_or0(64 * b + 4 * i, d));
#pragma unroll
    for (int e = 0; e < 4; ++e) f[4 * b + e] = v[e];
  }
  if (REM >= 2) {
    const f32x2 v = load2(row + chan_or0(64 * NB + 2 * i, d));
    f[4 * NB] = v[0];
    f[4 * NB + 1] = v[1];
  }
  if (REM & 1) f[DS - 1] = load_f32<T>(row + chan_or0(64 * NB + (REM >= 2 ? 32 : 0) + i, d));
}

// ---- bf16 operands on v_mfma_f32_16x16x32_bf16: 16 times the fp32 rate, fp32 accumulation.  A product
// of two bf16 values is exact in fp32, so K Q^T takes K and Q as they are.  An fp32 probability is the
// exact sum of three bf16 parts (24 bits of significand, eight a part, split by truncation), so V^T P^T
// is three products with V and rounds where the fp32 instruction rounds: in the accumulation.
// Matrix cycles of 16 x 16 logits at d = 128, forward: 64 + 192 against 2,048.  Error against fp64
// over seven shapes (24 to 128 keys a block, d = 64 .. 200; test_only_results_are_rounded): an element of O
// rounds to another bf16 value only within 0.35e-6 RMS of the midpoint, 0.70e-6 on the vector ALUs; LSE has
// an rms error of 0.32 to 0.35e-6 (0.30 to 0.37e-6).
// 32,760-token layer of 60-token blocks at inference: 3.90 -> 1.53 ms.
// Layout: A row i, B column i, k slot (g, t), t = 0..7; D as above.  A and B share the order of k.
__device__ inline f32x4 mfma32b(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
// v_mfma_f32_16x16x16_bf16: the same cycles for half the k slots, (g, t) with t = 0..3
__device__ inline f32x4 mfma16b(u32x2 a, u32x2 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, a), __builtin_bit_cast(s16x4, b), c, 0, 0, 0);
}
__device__ inline uint32_t halves_hi(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302); }  // {a.hi, b.hi}
__device__ inline uint32_t halves_lo(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x05040100); }  // {a.lo, b.lo}

// channel contraction, 32 channels a step: lane group g supplies channels 32 s + 8 g + t
template <int DS>
__device__ inline void row_frags_bf16(const uint16_t* row, int g, int d, u32x4 (&f)[(DS + 1) / 2]) {
#pragma unroll
  for (int s = 0; s < (DS + 1) / 2; ++s) {
    const int ch = 32 * s + 8 * g;
    f[s] = *reinterpret_cast<const u32x4*>(row + chan_or0(ch, d));
    if (32 * s + 32 > kMinD<DS> && ch >= d) f[s] = u32x4{0u, 0u, 0u, 0u};
  }
}

// row contraction: word k of a row holds this lane's channels of tiles 2 k (low half) and 2 k + 1,
// the channels that col_frags takes
template <int DS>
__device__ inline void col_words(const uint16_t* row, int i, int d, uint32_t (&w)[(DS + 1) / 2]) {
  constexpr int NB = DS / 4, REM = DS % 4;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const u32x2 v = *reinterpret_cast<const u32x2*>(row + chan_or0(64 * b + 4 * i, d));
    w[2 * b] = v.x;
    w[2 * b + 1] = v.y;
  }
  if (REM >= 2) w[2 * NB] = *reinterpret_cast<const uint32_t*>(row + chan_or0(64 * NB + 2 * i, d));
  if (REM & 1) w[DS / 2] = row[chan_or0(64 * NB + (REM >= 2 ? 32 : 0) + i, d)];
}

// A operand of channel tile c from the words of eight rows: k slots t = 0..3 and 4..7
template <int W>
__device__ inline u32x4 col_operand(const uint32_t (&w)[8][W], int c) {
  const int k = c >> 1;
  if (c & 1) return u32x4{halves_hi(w[0][k], w[1][k]), halves_hi(w[2][k], w[3][k]), halves_hi(w[4][k], w[5][k]), halves_hi(w[6][k], w[7][k])};
  return u32x4{halves_lo(w[0][k], w[1][k]), halves_lo(w[2][k], w[3][k]), halves_lo(w[4][k], w[5][k]), halves_lo(w[6][k], w[7][k])};
}

// x = part[0] + part[1] + part[2] for the k slots t = 0..3 (a) and 4..7 (b).  PROB: x >= 0, and where x is
// not zero a part that would be zero becomes 2^-126, so that an infinity in the other operand does not turn
// into NaN (where x is zero all parts are: 2^-126 of a value at the type's limit is not small).  Otherwise
// an infinite x leaves its other parts zero.
template <bool PROB>
__device__ inline void split3(f32x4 a, f32x4 b, u32x4 (&part)[3]) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    float x[2] = {k < 2 ? a[2 * k] : b[2 * k - 4], k < 2 ? a[2 * k + 1] : b[2 * k - 3]};
    const float whole[2] = {x[0], x[1]};  // (no rest is larger, so the median below is max(rest, 2^-126), 0 if x is 0)
#pragma unroll
    for (int n = 0; n < 3; ++n) {
      part[n][k] = halves_hi(__float_as_uint(x[0]), __float_as_uint(x[1]));
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const float rest = x[h] - __uint_as_float(__float_as_uint(x[h]) & 0xffff0000u);
        x[h] = PROB ? __builtin_amdgcn_fmed3f(rest, 0x1p-126f, whole[h]) : copysignf(fmaxf(fabsf(rest), 0.f), x[h]);  // (fmaxf drops a NaN)
      }
    }
  }
}

// writes accumulator tile ct (D layout, this lane: rows 4 g + r) into a row of channels
template <int DS, typename F>
__device__ inline void scatter_tile(const f32x4 (&acc)[DS], int g, F put /* (first channel, up to 4 values, n) */) {
  constexpr int NB = DS / 4, REM = DS % 4;
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      put(64 * b + 16 * g + 4 * r, f32x4{acc[4 * b][r], acc[4 * b + 1][r], acc[4 * b + 2][r], acc[4 * b + 3][r]});
  if (REM >= 2) {
    const f32x4 p = acc[4 * NB], q = acc[4 * NB + 1];
    put(64 * NB + 8 * g, f32x4{p[0], q[0], p[1], q[1]});
    put(64 * NB + 8 * g + 4, f32x4{p[2], q[2], p[3], q[3]});
  }
  if (REM & 1) put(64 * NB + (REM >= 2 ? 32 : 0) + 4 * g, acc[DS - 1]);
}

__device__ inline int kept_id(const Geom& g, const int32_t* keep_idx, int64_t row, int n_keep, int pos) {
  // clamped: a malformed keep list must not turn into an out-of-bounds access
  return g.dense ? pos : min(max(keep_idx[row * n_keep + pos], 0), g.Bk - 1);
}
__device__ inline int listed_block(const Geom& g, const int32_t* idx, int beg, int t) {
  return g.dense ? t : min(max(idx[beg + t], 0), g.N - 1);
}

constexpr int NWV = 4;  // wavefronts per workgroup

// ---------------------------------------------------------------------------- forward
// Workgroup: 16 NQT retained queries of one block; its wavefronts take the 64-key steps of the
// block's list in turn.  S^T = K Q^T (queries on the D column), online softmax in the exp2 domain,
// O^T += V^T P^T.
template <typename T, int DS, int NQT, int NS>
__global__ __launch_bounds__(64 * NWV, 2) void fwd_generic_kernel(Geom g, AttnArgs a) {
  constexpr int LDO = 16 * DS + 4;                  // padded row of the merge buffer
  extern __shared__ __align__(16) float osum[];     // [NQT * 16][LDO]
  __shared__ int koff[256];
  __shared__ short keeppos[256];                    // position of a token among the retained rows, -1 if pruned
  __shared__ float ml[NWV][NQT][2][16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, i16 = lane & 15, gq = lane >> 4;
  const int64_t row = blockIdx.x;
  const int64_t bh = row / g.N;
  const int ib = (int)(row % g.N);
  const int q0 = blockIdx.y * 16 * NQT;
  const int d = g.d;
  const T* Qh = static_cast<const T*>(a.Q) + bh * g.L * d;
  const T* Kh = static_cast<const T*>(a.K) + bh * g.L * d;
  const T* Vh = static_cast<const T*>(a.V) + bh * g.L * d;
  T* Oh = static_cast<T*>(a.O_out) + bh * g.L * d;
  float* Lh = a.LSE_out + bh * g.L;
  const int origin_q = block_origin(g, ib);

  if (tid < g.Bk) koff[tid] = intra_offset(g, tid);
  keeppos[tid] = -1;
  __syncthreads();
  if (tid < a.n_keep) keeppos[kept_id(g, a.keep_idx, row, a.n_keep, tid)] = (short)tid;

  constexpr bool kBf16 = sizeof(T) == 2;
  constexpr int S = (DS + 1) / 2;  // 32-channel steps, words of a row (bf16)
  f32x4 q[NQT][kBf16 ? 1 : DS];
  u32x4 qb[NQT][kBf16 ? S : 1];
#pragma unroll
  for (int t = 0; t < NQT; ++t) {
    const int pos = min(q0 + 16 * t + i16, a.n_keep - 1);
    const T* qrow = Qh + (int64_t)(origin_q + koff[kept_id(g, a.keep_idx, row, a.n_keep, pos)]) * d;
    if constexpr (kBf16) row_frags_bf16<DS>(qrow, gq, d, qb[t]);
    else row_frags<DS>(qrow, gq, d, q[t]);
  }
  const float c2 = a.sm_scale * kLog2e;
  // Exponents are taken relative to the largest logit so far, and that starts at a finite value: a wavefront
  // may begin with masked keys, and relative to -inf they would be NaN
  constexpr float kLowest = -3.4e38f;
  f32x4 o[NQT][DS];
  float m[NQT], l[NQT];
#pragma unroll
  for (int t = 0; t < NQT; ++t) {
    m[t] = kLowest;
    l[t] = 0.f;
#pragma unroll
    for (int c = 0; c < DS; ++c) o[t][c] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const int beg = g.dense ? 0 : a.q2k_ptr[row];
  const int cnt = g.dense ? g.N : a.q2k_ptr[row + 1] - beg;
  constexpr int KC = 16 * NS;            // keys per step
  const int nch = (g.Bk + KC - 1) / KC;  // steps per KV block
  for (int n = wave; n < cnt * nch; n += NWV) {
    const int t = n / nch, k0 = (n - t * nch) * KC;
    const int64_t origin = block_origin_fast(g, listed_block(g, a.q2k_idx, beg, t));
    const int nk = min(KC, g.Bk - k0), ns = kBf16 ? NS : (nk + 15) >> 4;  // keys and 16-key tiles of this step
    f32x4 s[NQT][NS];
    float mx[NQT];
#pragma unroll
    for (int u = 0; u < NQT; ++u) mx[u] = -INFINITY;
#pragma unroll
    for (int st = 0; st < NS; ++st) {
      if (st < ns) {
        const T* krow = Kh + (origin + koff[k0 + min(16 * st + i16, nk - 1)]) * d;
        f32x4 kf[kBf16 ? 1 : DS];
        u32x4 kb[kBf16 ? S : 1];
        if constexpr (kBf16) row_frags_bf16<DS>(krow, gq, d, kb);
        else row_frags<DS>(krow, gq, d, kf);
#pragma unroll
        for (int u = 0; u < NQT; ++u) {
          f32x4 acc = {0.f, 0.f, 0.f, 0.f};
          if constexpr (kBf16) {
#pragma unroll
            for (int c = 0; c < S; ++c) acc = mfma32b(kb[c], qb[u][c], acc);
          } else {
#pragma unroll
            for (int c = 0; c < DS; ++c)
#pragma unroll
              for (int e = 0; e < 4; ++e) acc = mfma4(kf[c][e], q[u][c][e], acc);
          }
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            if (16 * st + 4 * gq + r >= nk) acc[r] = -INFINITY;  // past the block's last key
            mx[u] = fmaxf(mx[u], acc[r]);
          }
          s[u][st] = acc;
        }
      }
    }
    // V words of key tiles st, st + 1 (bf16); those of the first two are requested ahead of the softmax
    uint32_t vw[8][S];
    auto load_v = [&](int st) {
      if constexpr (kBf16) {
#pragma unroll
        for (int r = 0; r < 8; ++r)
          if (st + (r >> 2) < NS)
            col_words<DS>(Vh + (origin + koff[k0 + min(16 * st + 16 * (r >> 2) + 4 * gq + (r & 3), nk - 1)]) * d, i16, d, vw[r]);
      }
    };
    load_v(0);
#pragma unroll
    for (int u = 0; u < NQT; ++u) {
      const float mnew = fmaxf(m[u], quad_max(mx[u]) * c2);  // c2 > 0: the maximum commutes with the scaling
      const float alpha = __builtin_amdgcn_exp2f(m[u] - mnew);
      float sum = 0.f;
#pragma unroll
      for (int st = 0; st < NS; ++st)
        if (st < ns)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            s[u][st][r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[u][st][r], c2, -mnew));
            sum += s[u][st][r];
          }
      l[u] = l[u] * alpha + sum;  // per lane; the four lanes of a query are summed at the end
      m[u] = mnew;
      if (__builtin_amdgcn_ballot_w64(alpha != 1.f)) {
#pragma unroll
        for (int c = 0; c < DS; ++c) o[u][c] *= alpha;
      }
    }
    // rows past the block's last key are zeroed: their P is zero, and 0 * inf would not be
    if constexpr (kBf16) {
#pragma unroll
      for (int st = 0; st < NS; st += 2) {
        if (st > 0) load_v(st);
        if (st + 2 > NS || 16 * st + 32 > nk) {
#pragma unroll
          for (int r = 0; r < 8; ++r) {
            const int key = 16 * st + 16 * (r >> 2) + 4 * gq + (r & 3);
#pragma unroll
            for (int k = 0; k < S; ++k) vw[r][k] = st + (r >> 2) < NS && key < nk ? vw[r][k] : 0u;
          }
        }
        u32x4 part[NQT][3];
#pragma unroll
        for (int u = 0; u < NQT; ++u)
          split3<true>(s[u][st], st + 1 < NS ? s[u][st + 1 < NS ? st + 1 : st] : f32x4{0.f, 0.f, 0.f, 0.f}, part[u]);
#pragma unroll
        for (int c = 0; c < DS; ++c) {
          const u32x4 va = col_operand(vw, c);
#pragma unroll
          for (int n = 2; n >= 0; --n)
#pragma unroll
            for (int u = 0; u < NQT; ++u) o[u][c] = mfma32b(va, part[u][n], o[u][c]);
        }
      }
    } else {
#pragma unroll
      for (int st = 0; st < NS; ++st) {
        if (st < ns) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int key = 16 * st + 4 * gq + r;
            float vf[DS];
            col_frags<DS>(Vh + (origin + koff[k0 + min(key, nk - 1)]) * d, i16, d, vf);
            if (16 * st + 16 > nk) {
#pragma unroll
              for (int c = 0; c < DS; ++c) vf[c] = key < nk ? vf[c] : 0.f;
            }
#pragma unroll
            for (int u = 0; u < NQT; ++u)
#pragma unroll
              for (int c = 0; c < DS; ++c) o[u][c] = mfma4(vf[c], s[u][st][r], o[u][c]);
          }
        }
      }
    }
  }
  // merge the wavefronts: m = max m_w, (l, O) = sum of (l_w, O_w) 2^(m_w - m), wavefronts in order (one
  // that met no key above -inf has l_w = O_w = 0)
#pragma unroll
  for (int u = 0; u < NQT; ++u) {
    l[u] = quad_sum(l[u]);
    if (gq == 0) {
      ml[wave][u][0][i16] = m[u];
      ml[wave][u][1][i16] = l[u];
    }
  }
  __syncthreads();
  float lse[NQT];
#pragma unroll
  for (int u = 0; u < NQT; ++u) {
    float mt = ml[0][u][0][i16], lt = 0.f;
#pragma unroll
    for (int w = 1; w < NWV; ++w) mt = fmaxf(mt, ml[w][u][0][i16]);
#pragma unroll
    for (int w = 0; w < NWV; ++w) lt += ml[w][u][1][i16] * __builtin_amdgcn_exp2f(ml[w][u][0][i16] - mt);
    // ln sum = (mt + log2 lt) sm_scale / c2, sum and quotient to twice fp32: times a rounded ln 2 it would keep
    // the rounding of c2, relative to the whole
    const float lg = __builtin_amdgcn_logf(lt), sum = mt + lg, k = a.sm_scale / c2;
    const float part = sum - mt, rest = ((mt - (sum - part)) + (lg - part)) * k + sum * (__builtin_fmaf(-k, c2, a.sm_scale) / c2);
    lse[u] = lt > 0.f ? __builtin_fmaf(sum, k, rest) : -INFINITY;
    // (no mass: an empty list gives zeros, a list of nothing but -inf logits NaN)
    const float w = lt > 0.f ? __builtin_amdgcn_exp2f(m[u] - mt) / lt : cnt > 0 ? NAN : 0.f;
#pragma unroll
    for (int c = 0; c < DS; ++c) o[u][c] *= w;
  }
  for (int w = 0; w < NWV; ++w) {
    if (wave == w) {
#pragma unroll
      for (int u = 0; u < NQT; ++u) {
        float* dst = osum + (16 * u + i16) * LDO;
        scatter_tile<DS>(o[u], gq, [&](int ch, f32x4 v) {
          if (w > 0) v += *reinterpret_cast<const f32x4*>(dst + ch);
          *reinterpret_cast<f32x4*>(dst + ch) = v;
        });
      }
    }
    __syncthreads();
  }
  if (wave == 0 && gq == 0) {
#pragma unroll
    for (int u = 0; u < NQT; ++u) ml[0][u][0][i16] = lse[u];
  }
  __syncthreads();
  // rows out, coalesced: a retained token takes its own row, a pruned one that of its window's
  // critical token (token filling), each written by the workgroup that holds the row
  const int nq = min(16 * NQT, a.n_keep - q0), dq4 = d >> 2;
  auto source = [&](int c) -> int {  // row of osum that token c receives, or < 0
    int p = keeppos[c];
    if (p < 0) p = g.dense ? -1 : keeppos[center_of(g, c)];
    p -= q0;
    return (p >= 0 && p < nq && p + q0 < a.n_keep) ? p : -1;
  };
  for (int e = tid; e < g.Bk * dq4; e += 64 * NWV) {
    const int c = e / dq4, ch = 4 * (e - c * dq4), p = source(c);
    if (p >= 0) store4(Oh + (int64_t)(origin_q + koff[c]) * d + ch, *reinterpret_cast<const f32x4*>(osum + p * LDO + ch));
  }
  if (tid < g.Bk) {
    const int p = source(tid);
    if (p >= 0) Lh[origin_q + koff[tid]] = ml[0][p >> 4][0][p & 15];
  }
}

// ------------------------------------------------------------- backward: preprocess
// g = dO of the retained row (+ for a window's critical token the dO of every pruned token of
// that window, ascending id); delta = <g, o>.  One wavefront per retained row, four channels a lane.
template <typename T>
__global__ __launch_bounds__(256) void bwd_pre_generic_kernel(Geom g, AttnArgs a, GenericWs w) {
  __shared__ short fill[256];  // window of a pruned token, -1 for a retained one
  __shared__ int koff[256];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t row = blockIdx.x;
  const int64_t bh = row / g.N;
  const T* dOh = static_cast<const T*>(a.dO) + bh * g.L * g.d;
  const T* Oh = static_cast<const T*>(a.O) + bh * g.L * g.d;
  const float* Lh = a.LSE_in + bh * g.L;
  const int64_t origin = block_origin(g, (int)(row % g.N));
  if (tid < g.Bk) {
    koff[tid] = intra_offset(g, tid);
    fill[tid] = g.dense ? -1 : (short)window_of(g, tid);
  }
  __syncthreads();
  if (tid < a.n_keep) fill[kept_id(g, a.keep_idx, row, a.n_keep, tid)] = -1;
  __syncthreads();
  const int ch = 4 * lane;
  for (int kp = blockIdx.y * 4 + wave; kp < w.nkp; kp += 4 * gridDim.y) {
    const int64_t e = row * w.nkp + kp;
    const int c = kept_id(g, a.keep_idx, row, a.n_keep, min(kp, a.n_keep - 1));
    const int64_t tok = origin + koff[c];
    f32x4 gv = {0.f, 0.f, 0.f, 0.f};
    float part = 0.f;
    if (ch < g.d && kp < a.n_keep) {
      gv = load4(dOh + tok * g.d + ch);
      const f32x4 ov = load4(Oh + tok * g.d + ch);
      if (!g.dense && c == center_of(g, c)) {
        const int win = window_of(g, c);
        for (int u0 = 0; u0 < g.Bk; u0 += 8) {  // eight loads in flight, added in ascending token id
          f32x4 x[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            const int v = min(u0 + u, g.Bk - 1);
            const bool use = u0 + u < g.Bk && fill[v] == win;
            x[u] = use ? load4(dOh + (origin + koff[v]) * g.d + ch) : f32x4{0.f, 0.f, 0.f, 0.f};
          }
#pragma unroll
          for (int u = 0; u < 8; ++u) gv += x[u];
        }
      }
      part = gv[0] * ov[0] + gv[1] * ov[1] + gv[2] * ov[2] + gv[3] * ov[3];
    }
    if (ch < g.d) *reinterpret_cast<f32x4*>(w.g + e * g.d + ch) = gv;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) part += __shfl_xor(part, o);
    if (lane == 0) {
      w.delta[e] = part;
      // padding: exp2(x - inf) = 0.  A row whose softmax has no value left LSE = -inf: its P is not finite, and
      // neither are the gradients it reaches (one with an empty list reaches none)
      w.lse2[e] = kp < a.n_keep ? Lh[tok] * kLog2e : INFINITY;
      w.tok[e] = (int)tok;
    }
  }
}

// Sums the wavefronts' accumulators of one [16 rows][channels] result in LDS, wavefronts in order:
// each of the SP wavefronts of a group (sub = 0..SP-1) adds its tiles to dst, the group's buffer.
template <int DS, int SP>
__device__ inline void sum_in_order(const f32x4 (&acc)[DS], float* dst_row, int sub, int gq) {
  for (int w = 0; w < SP; ++w) {
    if (sub == w)
      scatter_tile<DS>(acc, gq, [&](int ch, f32x4 v) {
        if (w > 0) v += *reinterpret_cast<const f32x4*>(dst_row + ch);
        *reinterpret_cast<f32x4*>(dst_row + ch) = v;
      });
    __syncthreads();
  }
}

// ------------------------------------------------------------------- backward: dQ
// As the forward, 16 queries a workgroup: S^T = K Q^T, dP^T = V G^T, dS^T = P^T (dP^T - delta),
// dQ^T += K^T dS^T.  bf16 tensors: 32 keys a step; G is split once, dS in each step.  A 3,024-token
// training layer of 24-token blocks (all its launches): 0.444 -> 0.359 ms; elements of dQ that are not
// the bf16 rounding of the exact result 0.016 -> 0.013 % (mean of the seven shapes above).
template <typename T, int DS, bool FULL>
__global__ __launch_bounds__(64 * NWV, DS <= 8 ? 2 : 1) void bwd_dq_generic_kernel(Geom g, AttnArgs a, GenericWs w) {
  constexpr int LDO = 16 * DS + 4;
  __shared__ __align__(16) float osum[16 * LDO];
  __shared__ int koff[256];
  __shared__ short keeppos[256];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, i16 = lane & 15, gq = lane >> 4;
  const int64_t row = blockIdx.x;
  const int64_t bh = row / g.N;
  const int ib = (int)(row % g.N);
  const int q0 = blockIdx.y * 16;
  const int d = g.d;
  const T* Qh = static_cast<const T*>(a.Q) + bh * g.L * d;
  const T* Kh = static_cast<const T*>(a.K) + bh * g.L * d;
  const T* Vh = static_cast<const T*>(a.V) + bh * g.L * d;
  T* dQh = static_cast<T*>(a.dQ) + bh * g.L * d;
  const int origin_q = block_origin(g, ib);
  if (tid < g.Bk) koff[tid] = intra_offset(g, tid);
  keeppos[tid] = -1;
  __syncthreads();
  if (tid < a.n_keep) keeppos[kept_id(g, a.keep_idx, row, a.n_keep, tid)] = (short)tid;

  const int64_t e = row * w.nkp + q0 + i16;  // this lane's query (padding rows: P = 0)
  constexpr bool kBf16 = sizeof(T) == 2;
  constexpr int S = (DS + 1) / 2;
  f32x4 q[kBf16 ? 1 : DS], gr[kBf16 ? 1 : DS], dq[DS];
  u32x4 qb[kBf16 ? S : 1], gb[kBf16 ? S : 1][3];
  if constexpr (kBf16) {
    row_frags_bf16<DS>(Qh + (int64_t)w.tok[e] * d, gq, d, qb);
#pragma unroll
    for (int c = 0; c < S; ++c) {
      const int ch = 32 * c + 8 * gq;
      const float* p = w.g + e * d + chan_or0(ch, d);
      f32x4 x = load4(p), y = load4(p + 4);
      if (32 * c + 32 > kMinD<DS> && ch >= d) x = y = f32x4{0.f, 0.f, 0.f, 0.f};
      split3<false>(x, y, gb[c]);
    }
  } else {
    row_frags<DS>(Qh + (int64_t)w.tok[e] * d, gq, d, q);
    row_frags<DS>(w.g + e * d, gq, d, gr);
  }
  const float lse2 = w.lse2[e], delta = w.delta[e];
#pragma unroll
  for (int c = 0; c < DS; ++c) dq[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  const float c2 = a.sm_scale * kLog2e;
  const int beg = g.dense ? 0 : a.q2k_ptr[row];
  const int cnt = g.dense ? g.N : a.q2k_ptr[row + 1] - beg;
  constexpr int KS = kBf16 ? 32 : 16;  // keys per step
  const int nst = (g.Bk + KS - 1) / KS;
  for (int n = wave; n < cnt * nst; n += NWV) {
    const int t = n / nst, k0 = (n - t * nst) * KS;
    const int64_t origin = block_origin_fast(g, listed_block(g, a.q2k_idx, beg, t));
    const int last = g.Bk - 1;
    if constexpr (kBf16) {
      f32x4 ds[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (k0 + 16 * h <= last) {
          const int64_t krow = (origin + koff[min(k0 + 16 * h + i16, last)]) * d;
          u32x4 kb[S], vb[S];
          row_frags_bf16<DS>(Kh + krow, gq, d, kb);
          row_frags_bf16<DS>(Vh + krow, gq, d, vb);
          f32x4 s = {0.f, 0.f, 0.f, 0.f}, dp = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int c = 0; c < S; ++c) {
            s = mfma32b(kb[c], qb[c], s);
#pragma unroll
            for (int x = 2; x >= 0; --x) dp = mfma32b(vb[c], gb[c][x], dp);
          }
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float v = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], c2, -lse2)) * (dp[r] - delta);
            ds[h][r] = k0 + 16 * h + 4 * gq + r > last ? 0.f : v;
          }
        }
      }
      uint32_t kw[8][S];
#pragma unroll
      for (int r = 0; r < 8; ++r)
        col_words<DS>(Kh + (origin + koff[min(k0 + (r >= 4 ? 16 : 0) + 4 * gq + (r & 3), last)]) * d, i16, d, kw[r]);
      u32x4 part[3];
      split3<false>(ds[0], ds[1], part);
#pragma unroll
      for (int c = 0; c < DS; ++c) {
        const u32x4 ka = col_operand(kw, c);
#pragma unroll
        for (int x = 2; x >= 0; --x) dq[c] = mfma32b(ka, part[x], dq[c]);
      }
    } else {
      const int64_t krow = (origin + koff[min(k0 + i16, last)]) * d;
      f32x4 kf[DS], vf[DS];
      row_frags<DS, FULL>(Kh + krow, gq, d, kf);
      row_frags<DS, FULL>(Vh + krow, gq, d, vf);
      f32x4 s = {0.f, 0.f, 0.f, 0.f}, dp = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < DS; ++c)
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          s = mfma4(kf[c][x], q[c][x], s);
          dp = mfma4(vf[c][x], gr[c][x], dp);
        }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float kc[DS];
        col_frags<DS>(Kh + (origin + koff[min(k0 + 4 * gq + r, last)]) * d, i16, d, kc);
        float ds = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], c2, -lse2)) * (dp[r] - delta);
        if (k0 + 4 * gq + r > last) ds = 0.f;
#pragma unroll
        for (int c = 0; c < DS; ++c) dq[c] = mfma4(kc[c], ds, dq[c]);
      }
    }
  }
  sum_in_order<DS, NWV>(dq, osum + i16 * LDO, wave, gq);
  const int nq = min(16, a.n_keep - q0), dq4 = d >> 2;
  for (int x = tid; x < g.Bk * dq4; x += 64 * NWV) {
    const int c = x / dq4, ch = 4 * (x - c * dq4), p = keeppos[c] - q0;
    T* out = dQh + (int64_t)(origin_q + koff[c]) * d + ch;
    if (p >= 0 && p < nq) store4(out, *reinterpret_cast<const f32x4*>(osum + p * LDO + ch) * a.sm_scale);
    else if (keeppos[c] < 0 && blockIdx.y == 0) store4(out, f32x4{0.f, 0.f, 0.f, 0.f});  // pruned: no part in the forward
  }
}

// --------------------------------------------------------------- backward: dK, dV
// Workgroup: KW 16-key tiles of one KV block (the owner of its gradients), NWV / KW wavefronts a
// tile, which take the query tiles of the block's k2q list in turn.  Keys on the D column, K and V
// of the tile in registers: S = Q K^T, dP = G V^T, dV^T += G^T P, dK^T += Q^T dS.
// bf16 tensors: S and dK on the bf16 instruction (dS in three parts, a tile of 16 queries fills its
// 16-slot form); dP and dV have the folded fp32 gradient as an operand, whose split would cost as much
// here as it saves, and stay on the fp32 one.  A 3,024-token training layer of 24-token blocks: 0.359 ->
// 0.315 ms; elements of dK that are not the bf16 rounding of the exact result 0.049 -> 0.046 %.
template <typename T, int DS, int KW, bool FULL>
__global__ __launch_bounds__(64 * NWV, DS <= 8 ? 2 : 1) void bwd_dkv_generic_kernel(Geom g, AttnArgs a, GenericWs w) {
  constexpr int LDO = 16 * DS + 4, SP = NWV / KW;
  __shared__ __align__(16) float osum[KW * 16 * LDO];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, i16 = lane & 15, gq = lane >> 4;
  const int kt = wave % KW, sub = wave / KW;
  const int64_t col = blockIdx.x;  // (b*H + h)*N + j
  const int64_t bh = col / g.N;
  const int j = (int)(col % g.N);
  const int k0 = (blockIdx.y * KW + kt) * 16;
  const int d = g.d;
  const T* Qh = static_cast<const T*>(a.Q) + bh * g.L * d;
  const T* Kh = static_cast<const T*>(a.K) + bh * g.L * d;
  const T* Vh = static_cast<const T*>(a.V) + bh * g.L * d;
  const int64_t ktok = (int64_t)block_origin(g, j) + intra_offset(g, min(k0 + i16, g.Bk - 1));
  constexpr bool kBf16 = sizeof(T) == 2;
  constexpr int S = (DS + 1) / 2;
  f32x4 kf[kBf16 ? 1 : DS], vf[DS], dk[DS], dv[DS];
  u32x4 kb[kBf16 ? S : 1];
  if constexpr (kBf16) row_frags_bf16<DS>(Kh + ktok * d, gq, d, kb);
  else row_frags<DS>(Kh + ktok * d, gq, d, kf);
  row_frags<DS>(Vh + ktok * d, gq, d, vf);
#pragma unroll
  for (int c = 0; c < DS; ++c) dk[c] = dv[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  const float c2 = a.sm_scale * kLog2e;
  const int beg = g.dense ? 0 : a.k2q_ptr[col];
  const int cnt = g.dense ? g.N : a.k2q_ptr[col + 1] - beg;
  const int nqt = w.nkp >> 4;  // query tiles per block
  if (k0 < g.Bk)
    for (int n = sub; n < cnt * nqt; n += SP) {
      const int t = n / nqt;
      const int64_t e0 = (bh * g.N + listed_block(g, a.k2q_idx, beg, t)) * w.nkp + (n - t * nqt) * 16;
      f32x4 s = {0.f, 0.f, 0.f, 0.f}, dp = {0.f, 0.f, 0.f, 0.f};
      if constexpr (kBf16) {
        u32x4 qb[S];
        f32x4 gf[DS];
        row_frags_bf16<DS>(Qh + (int64_t)w.tok[e0 + i16] * d, gq, d, qb);
        row_frags<DS, FULL>(w.g + (e0 + i16) * d, gq, d, gf);
#pragma unroll
        for (int c = 0; c < S; ++c) s = mfma32b(qb[c], kb[c], s);
#pragma unroll
        for (int c = 0; c < DS; ++c)
#pragma unroll
          for (int x = 0; x < 4; ++x) dp = mfma4(gf[c][x], vf[c][x], dp);
      } else {
        f32x4 qf[DS], gf[DS];
        row_frags<DS, FULL>(Qh + (int64_t)w.tok[e0 + i16] * d, gq, d, qf);
        row_frags<DS, FULL>(w.g + (e0 + i16) * d, gq, d, gf);
#pragma unroll
        for (int c = 0; c < DS; ++c)
#pragma unroll
          for (int x = 0; x < 4; ++x) {
            s = mfma4(qf[c][x], kf[c][x], s);
            dp = mfma4(gf[c][x], vf[c][x], dp);
          }
      }
      const f32x4 l4 = *reinterpret_cast<const f32x4*>(w.lse2 + e0 + 4 * gq), d4 = *reinterpret_cast<const f32x4*>(w.delta + e0 + 4 * gq);
      f32x4 ds;
      uint32_t qw[4][kBf16 ? S : 1];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float gc[DS];
        const int64_t e = e0 + 4 * gq + r;
        const T* qrow = Qh + (int64_t)w.tok[e] * d;
        col_frags<DS>(w.g + e * d, i16, d, gc);
        const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], c2, -l4[r]));
        ds[r] = p * (dp[r] - d4[r]);
        if constexpr (kBf16) {
          col_words<DS>(qrow, i16, d, qw[r]);
#pragma unroll
          for (int c = 0; c < DS; ++c) dv[c] = mfma4(gc[c], p, dv[c]);
        } else {
          float qc[DS];
          col_frags<DS>(qrow, i16, d, qc);
#pragma unroll
          for (int c = 0; c < DS; ++c) {
            dv[c] = mfma4(gc[c], p, dv[c]);
            dk[c] = mfma4(qc[c], ds[r], dk[c]);
          }
        }
      }
      if constexpr (kBf16) {
        u32x4 part[3];
        split3<false>(ds, f32x4{0.f, 0.f, 0.f, 0.f}, part);
#pragma unroll
        for (int c = 0; c < DS; ++c) {
          const int k = c >> 1;
          const u32x2 qa = c & 1 ? u32x2{halves_hi(qw[0][k], qw[1][k]), halves_hi(qw[2][k], qw[3][k])}
                                 : u32x2{halves_lo(qw[0][k], qw[1][k]), halves_lo(qw[2][k], qw[3][k])};
#pragma unroll
          for (int x = 2; x >= 0; --x) dk[c] = mfma16b(qa, u32x2{part[x].x, part[x].y}, dk[c]);
        }
      }
    }
  const int dq4 = d >> 2, kbase = blockIdx.y * KW * 16, nk = min(KW * 16, g.Bk - kbase);
  for (int pass = 0; pass < 2; ++pass) {
    if (pass == 0) sum_in_order<DS, SP>(dk, osum + (16 * kt + i16) * LDO, sub, gq);
    else sum_in_order<DS, SP>(dv, osum + (16 * kt + i16) * LDO, sub, gq);
    T* out = static_cast<T*>(pass == 0 ? a.dK : a.dV) + bh * g.L * d;
    const float scale = pass == 0 ? a.sm_scale : 1.f;
    for (int x = tid; x < nk * dq4; x += 64 * NWV) {
      const int c = x / dq4, ch = 4 * (x - c * dq4);
      store4(out + (int64_t)token_of(g, j, kbase + c) * d + ch, *reinterpret_cast<const f32x4*>(osum + c * LDO + ch) * scale);
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------------- launches
template <typename T, int DS, int NQT, int NS>
static int fwd_n(const Geom& g, const AttnArgs& a, hipStream_t st) {
  const size_t lds = (size_t)NQT * 16 * (16 * DS + 4) * 4;
  hipLaunchKernelGGL((fwd_generic_kernel<T, DS, NQT, NS>), dim3(g.rows, (a.n_keep + 16 * NQT - 1) / (16 * NQT)), dim3(64 * NWV), lds, st, g, a);
  return check_launch();
}

// two query tiles a wavefront (half the K and V loads per product) where both exist and their
// operands and accumulators (32 DS registers each way) leave two wavefronts per SIMD
template <typename T, int DS, int NS>
static int fwd_s(const Geom& g, const AttnArgs& a, hipStream_t st) {
  if constexpr (DS <= 8)
    if (a.n_keep > 16) return fwd_n<T, DS, 2, NS>(g, a, st);
  return fwd_n<T, DS, 1, NS>(g, a, st);
}

// 16-key tiles per step.  bf16: compiled in, so that no branch stands between the loads of a step; the
// block's tiles are spread evenly over its steps, and tiles past its end are masked.  fp32 takes up to
// four and skips those past the end: its time is that of the products.
// Compiled in against skipped, with the first V loads ahead of the softmax: 32,760-token layer of 60-token
// blocks 1.53 -> 1.31 ms, training layer of 24-token blocks 0.315 -> 0.307.
template <typename T, int DS>
static int fwd_t(const Geom& g, const AttnArgs& a, hipStream_t st) {
  if constexpr (sizeof(T) == 2) {
    const int tiles = (g.Bk + 15) / 16, steps = (tiles + 3) / 4, ns = (tiles + steps - 1) / steps;
    if (ns <= 2) return fwd_s<T, DS, 2>(g, a, st);
    if (ns == 3) return fwd_s<T, DS, 3>(g, a, st);
  }
  return fwd_s<T, DS, 4>(g, a, st);
}

template <typename T, int DS, bool FULL>
static int bwd_full(const Geom& g, const AttnArgs& a, hipStream_t st) {
  const GenericWs w = carve(g, a.n_keep, a.ws);
  const int nqt = w.nkp / 16, nkt = (g.Bk + 15) / 16;
  if (a.stages & BSA_BWD_PRE) hipLaunchKernelGGL((bwd_pre_generic_kernel<T>), dim3(g.rows, nqt), dim3(256), 0, st, g, a, w);
  if (a.stages & BSA_BWD_DQ) hipLaunchKernelGGL((bwd_dq_generic_kernel<T, DS, FULL && sizeof(T) == 4>), dim3(g.rows, nqt), dim3(64 * NWV), 0, st, g, a, w);
  if (a.stages & BSA_BWD_DKV) {
    // four key tiles a workgroup share the records they stream through the L1 (up to d = 128: their
    // result rows fit 64 KB of LDS); with too few workgroups to fill the chip the list of one tile
    // is spread over the four wavefronts instead.  Several tiles against one, d = 128, r = 0.5, us: fp32,
    // four tiles a block, 256 rows 79 / 61, 512 rows 120 / 151, 1,024 rows 906 / 1,001 (eight times the pairs);
    // bf16, two tiles, 256 rows 18 / 17, 512 rows 31 / 35.  The line is not right everywhere: a last group
    // that is mostly empty (three or five tiles) costs up to a quarter (fp32, five tiles, 1,024 rows 2,163 / 1,746).
    bool four = false;
    if constexpr (DS <= 8) four = (int64_t)g.rows * ((nkt + 3) / 4) >= 512 && nkt > 2;
    if (four) {
      if constexpr (DS <= 8)
        hipLaunchKernelGGL((bwd_dkv_generic_kernel<T, DS, 4, FULL>), dim3(g.rows, (nkt + 3) / 4), dim3(64 * NWV), 0, st, g, a, w);
    }
    else if ((int64_t)g.rows * ((nkt + 1) / 2) >= 512 && nkt > 1)
      hipLaunchKernelGGL((bwd_dkv_generic_kernel<T, DS, 2, FULL>), dim3(g.rows, (nkt + 1) / 2), dim3(64 * NWV), 0, st, g, a, w);
    else
      hipLaunchKernelGGL((bwd_dkv_generic_kernel<T, DS, 1, FULL>), dim3(g.rows, nkt), dim3(64 * NWV), 0, st, g, a, w);
  }
  return check_launch();
}

// Where d fills its groups there are instances without the selects that zero padding channels: fp32 dQ at d = 128
// 497 -> 478 us, dK/dV at 64 374 -> 370; bf16 dK/dV (the rows of G; its other operands need none) at d = 96, 45 keys
// a block, 483 -> 467
template <typename T, int DS>
static int bwd_t(const Geom& g, const AttnArgs& a, hipStream_t st) {
  return g.d == 16 * DS ? bwd_full<T, DS, true>(g, a, st) : bwd_full<T, DS, false>(g, a, st);
}

// the compiled numbers of 16-channel groups; a head dimension takes the next one up
#define BSA_BY_DS(fn, T)                              \
  do {                                                \
    const int n = (g.d + 15) / 16;                    \
    if (n <= 2) return fn<T, 2>(g, a, st);            \
    if (n <= 4) return fn<T, 4>(g, a, st);            \
    if (n <= 5) return fn<T, 5>(g, a, st);            \
    if (n <= 6) return fn<T, 6>(g, a, st);            \
    if (n <= 8) return fn<T, 8>(g, a, st);            \
    if (n <= 12) return fn<T, 12>(g, a, st);          \
    return fn<T, 16>(g, a, st);                       \
  } while (0)

int launch_fwd_generic(const Geom& g, int dtype, const AttnArgs& a, hipStream_t st) {
  if (dtype == BSA_F32) BSA_BY_DS(fwd_t, float);
  BSA_BY_DS(fwd_t, uint16_t);
}
int launch_bwd_generic(const Geom& g, int dtype, const AttnArgs& a, hipStream_t st) {
  if (dtype == BSA_F32) BSA_BY_DS(bwd_t, float);
  BSA_BY_DS(bwd_t, uint16_t);
}

}  // namespace bsa
