// dK, dV of the sparse attention (bf16 matrix cores): one workgroup owns one KV block.
//
//   dV^T += G^T P,  dK^T += Q^T dS,  with S = Q K^T, P = exp2(S c - LSE), dP = G V^T,
//   dS = P (dP - delta), over the records (32 retained query rows) of the block's k2q list.
//
// The four wavefronts of a workgroup take the records in turn, each with all 64 keys of the block:
// their K and V fragments (B operands) stay in 128 registers, the dK^T and dV^T accumulators fill
// the 256 accumulation registers, and the records stream through a private LDS ring.  There is no
// barrier in the loop and no wavefront ever multiplies for a list that is not its own; the four
// partial sums are added in wavefront order at the end.
//
// What bounds it: the matrix cores.  Every fragment read from LDS feeds two MFMAs (the two key
// halves): 32 fragments for 64 MFMAs of a record, against 48 for 32 in the two-blocks-per-workgroup
// kernel this replaces, whose K and V fragments came from LDS with every record and whose
// wavefronts idled on records that only the other block lists.  One wavefront per SIMD cannot lean
// on a neighbour to fill gaps, so the instruction order is fixed here: groups of two MFMAs
// (64 cycles) with a share of the vector work, LDS reads and DMA requests in between, nothing but
// fences separating the groups.  exp2 runs under the dP products, dS under the dV products; the dK
// products hide the requests.
//
// The 32 x 32 x 16 MFMA is written as inline assembly: the S and dP tiles must land in ordinary
// registers and the accumulators in accumulation registers, and the compiler takes one form for
// all.  The compiler does not know the hazards of an MFMA inside assembly.  Result to vector
// instruction, 12 wait states of 4 cycles: a tile's consumers are ordered behind a later MFMA that is
// at least two issue slots (64 cycles) away, through the tied operands below.  Vector instruction to
// MFMA operand, 2 wait states: the products whose operand was just converted start with a s_nop.
//
// Measured (MI355X, steady state): 33,280 tokens, 12 heads, d = 128, p = 0.9, half of the queries:
// 3.29 -> 2.63 ms (1,138 TFLOP/s; a long run of library products of random 8192^3 bf16 matrices reaches
// 1,410 on the same card).  The matrix cores are busy 55 % of the launch's cycles, which pass at 2.0 GHz;
// 3.5 GB come from beyond the L2 (86 % hits).  A wavefront issues an instruction in half of its cycles,
// a vector instruction in a third: what the MFMAs leave free, the exponentials take.
#include "bsa_pipe.h"

namespace bsa {

// the record's 256 bytes of row constants: sixteen lanes
__device__ inline void dma_tail(uint64_t sbase, uint32_t lane16, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\ts_mov_b64 exec, 0xffff\n\tglobal_load_lds_dwordx4 %0, %1\n\ts_mov_b64 exec, -1"
               :
               : "v"(lane16), "s"(sbase), "s"(lds)
               : "memory", "m0");
}

constexpr int kListCap = 8192;  // blocks per head at most

// D: channels (64 or 128), PACK: a record holds two query blocks of at most 16 rows.
template <int D, bool PACK>
__global__ __launch_bounds__(256, 1) void bwd_dkv_pipe_kernel(Geom g, AttnArgs a) {
  using R = BwdRec<D>;
  constexpr int NH = PBK / 32;  // 32-key halves of the KV block
  constexpr int RB = D * 2, DT = D / 32, DS = D / 16, NT = NH * DT;
  constexpr int ND = 32 * RB / 1024;        // DMA instructions of a record's Q (or G) rows
  constexpr int NF = 2 * DS + 4 * DT;       // fragments of a record in order of use
  constexpr int RING = DT == 2 ? 2 : 4;     // fragments read ahead (64 cycles each)
  static_assert(NF % RING == 0 && 2 * DT - RING >= 2, "the ring wraps into the next record");
  static_assert(8 * R::BYTES >= NT * 16 * 1024, "the record ring doubles as the reduction buffer");
  extern __shared__ __align__(16) uint8_t smem[];  // [4 wavefronts][2 records] | list
  uint16_t* list = reinterpret_cast<uint16_t*>(smem + 8 * R::BYTES);

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = lane >> 5, col = lane & 31;
  const int units = g.rows, per = units >> 3, rest = units & 7, xcd = blockIdx.x & 7, nth = blockIdx.x >> 3;
  if (nth >= per + (xcd < rest ? 1 : 0)) return;
  const int unit = xcd * per + min(xcd, rest) + nth;  // neighbouring KV blocks share an XCD's L2
  const int64_t bh = unit / g.N;
  const int j = unit % g.N;
  const int nqt = a.n_keep > 32 ? 2 : 1;                       // records per query block
  const int nrec = PACK ? (g.N + 1) / 2 : g.N * nqt;           // records of a head
  const uint16_t* Kh = static_cast<const uint16_t*>(a.K) + bh * g.L * D;
  const uint16_t* Vh = static_cast<const uint16_t*>(a.V) + bh * g.L * D;
  const uint8_t* ws = static_cast<const uint8_t*>(a.ws) + bh * nrec * (int64_t)R::BYTES;

  // K and V fragments (B operands): lane (col, grp) holds channels 16 s + 8 grp .. +7 of key 32 h + col.
  // Requested ahead of the list, whose loads they overlap.
  bf16x8 kf[NH][DS], vf[NH][DS];
  const int origin = block_origin(g, j);
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    const int64_t first = (origin + intra_offset(g, 32 * h + col)) * (int64_t)D + 8 * grp;
#pragma unroll
    for (int s = 0; s < DS; ++s) {
      kf[h][s] = as_frag(*reinterpret_cast<const u32x4*>(Kh + first + 16 * s));
      vf[h][s] = as_frag(*reinterpret_cast<const u32x4*>(Vh + first + 16 * s));
    }
  }

  // The block's list as a set: bits in LDS, then entries in ascending order (a duplicate counts once, a
  // block id out of range not at all).  Entries are query blocks; packed: pairs, with two bits for
  // its members (bits 14, 15).
  uint32_t* bits = reinterpret_cast<uint32_t*>(smem);  // one word a thread; in the record ring, not in use yet
  int* base = reinterpret_cast<int*>(bits + kListCap / 32);  // entries ahead of a word's, then their number
  bits[tid] = g.dense ? (tid * 32 + 32 <= g.N ? 0xffffffffu : tid * 32 < g.N ? (1u << (g.N - tid * 32)) - 1u : 0u) : 0u;
  __syncthreads();
  if (!g.dense) {
    const int beg = a.k2q_ptr[unit], end = a.k2q_ptr[unit + 1];
    for (int t = beg + tid; t < end; t += 256) {
      const int b = a.k2q_idx[t];
      if ((unsigned)b < (unsigned)g.N) atomicOr(&bits[b >> 5], 1u << (b & 31));
    }
    __syncthreads();
  }
  auto heads = [&](uint32_t w) { return PACK ? (w | (w >> 1)) & 0x55555555u : w; };  // a bit for every entry
  if (wave == 0) {
    int n[4], sum = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      n[k] = sum;
      sum += __popc(heads(bits[4 * lane + k]));
    }
    int upto = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int v = __shfl_up(upto, off);
      if (lane >= off) upto += v;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) base[4 * lane + k] = upto - sum + n[k];
    if (lane == 63) base[256] = upto;
  }
  __syncthreads();
  const int cnt = base[256];
  for (int t = tid; t < (PACK ? (g.N + 1) / 2 : g.N); t += 256) {
    const int b = PACK ? 2 * t : t, bit = b & 31;
    const uint32_t w = bits[b >> 5], hd = heads(w);
    if ((hd >> bit) & 1u)
      list[base[b >> 5] + __popc(hd & ((1u << bit) - 1u))] = (uint16_t)(PACK ? t | (((w >> bit) & 3u) << 14) : t);
  }

#pragma unroll
  for (int h = 0; h < NH; ++h)
#pragma unroll
    for (int s = 0; s < DS; ++s) {  // waited for here, not in the loop
      settle(kf[h][s]);
      settle(vf[h][s]);
    }
  f32x16 dk[NH][DT], dv[NH][DT];
#pragma unroll
  for (int h = 0; h < NH; ++h)
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) dk[h][dt][r] = dv[h][dt][r] = 0.f;
  __syncthreads();  // the list is whole, the ring free
  const int items = __builtin_amdgcn_readfirstlane(cnt * nqt);
  const int mine = (items - wave + 3) >> 2;  // items wave, wave + 4, ...
  const float c2 = a.sm_scale * kLog2e;

  if (mine > 0) {
    const uint32_t lds0 = uniform_lds(smem + wave * 2 * R::BYTES);
    const uint32_t lane16 = lane * 16;
    const int qshift = nqt - 1;
    auto entry = [&](int i) { return (int)list[(wave + 4 * min(i, mine - 1)) >> qshift]; };
    auto rec_of = [&](int e, int i) {  // wave-uniform record number of item i with list entry e
      const int t = wave + 4 * min(i, mine - 1);
      return PACK ? (e & 0x3fff) : (e << qshift) | (t & qshift);
    };
    auto src_of = [&](int rec) { return uniform64(ws + rec * (int64_t)R::BYTES); };
    // requests: Q rows (with the row constants) and G rows of a record into ring slot `b`
    auto dma_rows = [&](uint64_t src, uint32_t dst, auto N) {
      constexpr int n = decltype(N)::value;
      dma_kb<1024 * (n & 3)>(src + 4096 * (n >> 2), lane16, dst + 4096 * (n >> 2));
    };
    int e0 = __builtin_amdgcn_readfirstlane(entry(0)), e1 = __builtin_amdgcn_readfirstlane(entry(1));
    uint64_t src1 = src_of(rec_of(e1, 1));
    {
      const uint64_t src0 = src_of(rec_of(e0, 0));
      static_for<0, ND>([&](auto N) { dma_rows(src0 + R::GC, lds0 + R::GC, N); });
      static_for<0, ND>([&](auto N) { dma_rows(src0 + R::QC, lds0 + R::QC, N); });
      dma_tail(src0 + R::LS, lane16, lds0 + R::LS);
      static_for<0, ND>([&](auto N) { dma_rows(src1 + R::GC, lds0 + R::BYTES + R::GC, N); });
    }
    int flip = R::BYTES;  // from the current ring slot to the other
    uint32_t cur = lds0;  // the current slot
    // LDS offsets of the fragments (see bsa_mfma.h for the swizzle): row fragments of row col,
    // transposed ones of rows 8 h + 4 grp + .., channel tile dt; row constants of this lane's rows
    int koffs[DS], voffs[2][DT], dlo = lds0 + 16 * grp;
#pragma unroll
    for (int s = 0; s < DS; ++s) koffs[s] = lds0 + col * RB + (((2 * s + grp) ^ swz<D>(col)) << 4);
    const int L16 = lane & 15, q16 = lane >> 4, rsub = L16 >> 2, jj = L16 & 3;
    const int cl = 2 * (q16 & 1) + (jj >> 1), rhi = D == 128 ? rsub : (rsub >> 1);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
        voffs[h][dt] = lds0 + (8 * h + 4 * grp + rsub) * RB + ((((dt ^ rhi) << 2) | (cl ^ (2 * h + grp))) << 4) + 8 * (jj & 1);
    // fragment f of a record: Q rows, G rows, G^T and Q^T ((16-row step, channel tile) order)
    auto frag = [&](auto F) -> bf16x8 {
      constexpr int f = decltype(F)::value;
      if constexpr (f < DS) return frag_at(koffs[f] + R::QC);
      else if constexpr (f < 2 * DS) return frag_at(koffs[f - DS] + R::GC);
      else {
        constexpr int v = f - 2 * DS, w = v % (2 * DT), dt = w % DT, base = (v < 2 * DT ? R::GC : R::QC) + 16 * (w / DT) * RB;
        return frag_tr_at(voffs[0][dt] + base, voffs[1][dt] + base);
      }
    };
    bf16x8 fr[RING];
    auto refill = [&](auto F) {  // the ring slot of fragment f takes the one RING ahead, at the end the next record's
      constexpr int f = decltype(F)::value;
      fr[f % RING] = frag(std::integral_constant<int, (f + RING) % NF>{});
    };
    wait_vm<ND>();  // the first record has landed
    static_for<0, RING>([&](auto F) { fr[decltype(F)::value] = frag(F); });
    BSA_FENCE();
    for (int i = 0; i < mine; ++i) {
      const int e2v = entry(i + 2);
      const uint32_t other = cur + flip;
      f32x16 s[NH], dp[NH];
      bf16x8 pf[NH][2], df[NH][2];
      // ---- S = Q K^T; requests of the next record's Q rows
      static_for<0, DS>([&](auto KK) {
        constexpr int k = decltype(KK)::value;
        static_for<0, NH>([&](auto HH) {
          constexpr int h = decltype(HH)::value;
          if constexpr (k == 0) mfma_first(s[h], fr[k % RING], kf[h][k]);
          else mfma_next(s[h], fr[k % RING], kf[h][k]);
          if constexpr (h == 0) {  // (behind an MFMA of its own: a request may wait for the vector memory port)
            BSA_FENCE();
            static_for<k * ND / DS, (k + 1) * ND / DS>([&](auto N) { dma_rows(src1 + R::QC, other + R::QC, N); });
            BSA_FENCE();
          }
        });
        refill(KK);
        if constexpr (k == DS - 1) dma_tail(src1 + R::LS, lane16, other + R::LS);
        if constexpr (k == DS - 2) {
          int own[2] = {dlo, dlo};
          asm("" : "+v"(own[1]));
#pragma unroll
          for (int r4 = 0; r4 < 4; ++r4) {
#pragma unroll
            for (int h = 0; h < NH; ++h) {  // one read each: a copy of the other's registers would cost vector instructions
              const f32x4 v = f4_at(own[h] + R::DL + 32 * r4);
#pragma unroll
              for (int e = 0; e < 4; ++e) dp[h][4 * r4 + e] = v[e];
            }
          }
        }
        BSA_FENCE();
      });
      // ---- dP - delta = G V^T - delta; P under it
      static_for<0, DS>([&](auto KK) {
        constexpr int k = decltype(KK)::value, ra = 16 * k / DS, rz = 16 * (k + 1) / DS;
        const std::integral_constant<int, DS + k> F{};
        float lse[rz - ra];
#pragma unroll
        for (int r = ra; r < rz; ++r) {
          if (r == ra || r % 4 == 0) {
            const f32x4 v = f4_at(dlo + R::LS + 32 * (r / 4));
#pragma unroll
            for (int q = r; q < rz && q < (r / 4) * 4 + 4; ++q)  // packed: rows of a block that does not list this one have P = 0
              lse[q - ra] = PACK && !((e0 >> (14 + q / 8)) & 1) ? INFINITY : v[q % 4];
          }
        }
#pragma unroll
        for (int h = 0; h < NH; ++h) {
          if (k == 0) mfma_next(dp[h], fr[F % RING], vf[h][k], s[h]);
          else mfma_next(dp[h], fr[F % RING], vf[h][k]);
#pragma unroll
          for (int r = ra; r < rz; ++r) s[h][r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[h][r], c2, -lse[r - ra]));
        }
        if (k == DS - 2) {
#pragma unroll
          for (int h = 0; h < NH; ++h) pf[h][0] = d_to_b(s[h], 0);
        }
        refill(F);
        BSA_FENCE();
      });
      // ---- dV^T += G^T P; dS under it
      static_for<0, 2 * DT>([&](auto VV) {
        constexpr int v = decltype(VV)::value, dt = v % DT, ra = 16 * v / (2 * DT), rz = 16 * (v + 1) / (2 * DT);
        const std::integral_constant<int, 2 * DS + v> F{};
        static_for<0, NH>([&](auto HH) {
          constexpr int h = decltype(HH)::value;
          mfma_acc<h == 0 && v % DT == 0>(dv[h][dt], fr[F % RING], pf[h][v / DT]);
          if (v == 0) order_behind(dp[h]);
#pragma unroll
          for (int r = ra; r < rz; ++r) dp[h][r] = s[h][r] * dp[h][r];
        });
        if (v == 0) {
#pragma unroll
          for (int h = 0; h < NH; ++h) pf[h][1] = d_to_b(s[h], 1);
        }
        if (v == 2 * DT - 2) {
#pragma unroll
          for (int h = 0; h < NH; ++h) df[h][0] = d_to_b(dp[h], 0);
        }
        refill(F);
        BSA_FENCE();
      });
      // ---- dK^T += Q^T dS; requests of the G rows two records ahead (this record's are free now)
      const int e2 = __builtin_amdgcn_readfirstlane(e2v);
      const uint64_t src2 = src_of(rec_of(e2, i + 2));
      static_for<0, 2 * DT>([&](auto VV) {
        constexpr int v = decltype(VV)::value, dt = v % DT;
        const std::integral_constant<int, 2 * DS + 2 * DT + v> F{};
        if constexpr (v == 2 * DT - RING) {  // the next record has landed once only these G rows are outstanding
          wait_vm<(2 * DT - RING) * ND / (2 * DT)>();
#pragma unroll
          for (int q = 0; q < DS; ++q) koffs[q] += flip;
        }
        static_for<0, NH>([&](auto HH) {
          constexpr int h = decltype(HH)::value;
          mfma_acc<h == 0 && v % DT == 0>(dk[h][dt], fr[F % RING], df[h][v / DT]);
          if constexpr (h == 0) {
            BSA_FENCE();
            static_for<v * ND / (2 * DT), (v + 1) * ND / (2 * DT)>([&](auto N) { dma_rows(src2 + R::GC, cur + R::GC, N); });
            BSA_FENCE();
          }
        });
        if (v == 0) {
#pragma unroll
          for (int h = 0; h < NH; ++h) df[h][1] = d_to_b(dp[h], 1);
        }
        refill(F);
        BSA_FENCE();
      });
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) voffs[h][dt] += flip;
      dlo += flip;
      cur = other;
      flip = -flip;
      e0 = e1;
      e1 = e2;
      src1 = src2;
    }
    BSA_WAIT_VM(0);
    asm volatile("s_nop 15\n\ts_nop 15");  // the last accumulations land before anything reads them
#pragma unroll
    for (int h = 0; h < NH; ++h)
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) asm volatile("" : "+a"(dk[h][dt]), "+a"(dv[h][dt]));
  }

  // sum of the four wavefronts, in order, through the idle ring: dK then dV.  Of at most two items the last
  // two wavefronts have none, and their zeros stay out: a 256-token layer at d = 128, where this sum is a
  // good part of the launch, 13.8 -> 12.9 us with 16 queries a block, 14.5 -> 14.0 with 32 (with the loads
  // above); no difference from 3,000 tokens up.
  f32x4* red = reinterpret_cast<f32x4*>(smem) + lane;  // [tile][wavefront][4][64]
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    __syncthreads();
    if (wave < 2 || items > 2) {
#pragma unroll
      for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
          const f32x16& acc = pass ? dv[h][dt] : dk[h][dt];
#pragma unroll
          for (int r4 = 0; r4 < 4; ++r4)
            red[(((h * DT + dt) * 4 + wave) * 4 + r4) * 64] = f32x4{acc[4 * r4], acc[4 * r4 + 1], acc[4 * r4 + 2], acc[4 * r4 + 3]};
        }
    }
    __syncthreads();
    uint16_t* out = static_cast<uint16_t*>(pass ? a.dV : a.dK) + bh * g.L * D;
    const float scale = pass ? 1.f : a.sm_scale;
    auto put = [&](auto N) {
      constexpr int n = decltype(N)::value;
      for (int t = wave * NT / 4; t < (wave + 1) * NT / 4; ++t) {
        const int key = 32 * (t / DT) + col;
        const int64_t tok = origin + intra_offset(g, key);
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          f32x4 v = red[(t * 16 + r4) * 64];
#pragma unroll
          for (int w = 1; w < n; ++w) v += red[(t * 16 + 4 * w + r4) * 64];
          const int ch = 32 * (t % DT) + 8 * r4 + 4 * grp;
          u32x2 o;
          o.x = pack_bf16(v[0] * scale, v[1] * scale);
          o.y = pack_bf16(v[2] * scale, v[3] * scale);
          *reinterpret_cast<u32x2*>(out + tok * D + ch) = o;
        }
      }
    };
    if (items > 2) put(std::integral_constant<int, 4>{});
    else put(std::integral_constant<int, 2>{});
  }
}

template <int D>
static size_t lds_bytes(const Geom& g) { return (size_t)8 * BwdRec<D>::BYTES + (size_t)g.N * 2; }

template <int D, bool PACK>
static int launch_t(const Geom& g, const AttnArgs& a, hipStream_t st) {
  hipLaunchKernelGGL((bwd_dkv_pipe_kernel<D, PACK>), dim3((g.rows + 7) / 8 * 8), dim3(256), lds_bytes<D>(g), st, g, a);
  return check_launch();
}

// the dynamic LDS of the launch below, for the caller to take ahead of every launch of the backward
int grant_bwd_dkv_pipe(const Geom& g, const AttnArgs& a) {
  if (g.d == 128)
    return a.pack ? allow_dynamic_lds<bwd_dkv_pipe_kernel<128, true>>(lds_bytes<128>(g))
                  : allow_dynamic_lds<bwd_dkv_pipe_kernel<128, false>>(lds_bytes<128>(g));
  return a.pack ? allow_dynamic_lds<bwd_dkv_pipe_kernel<64, true>>(lds_bytes<64>(g))
                : allow_dynamic_lds<bwd_dkv_pipe_kernel<64, false>>(lds_bytes<64>(g));
}

int launch_bwd_dkv_pipe(const Geom& g, const AttnArgs& a, hipStream_t st) {
  if (g.d == 128) return a.pack ? launch_t<128, true>(g, a, st) : launch_t<128, false>(g, a, st);
  return a.pack ? launch_t<64, true>(g, a, st) : launch_t<64, false>(g, a, st);
}

}  // namespace bsa
