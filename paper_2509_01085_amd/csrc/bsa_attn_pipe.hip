// bf16 MFMA kernels that walk lists with a barrier a tile (Bk = 64, d = 128 or 64): the forward of launches whose lists are short
// (bsa_attn_fwd.hip has the other one; the choice is at the end of this file) and the backward's dQ.
//
// A workgroup owns four consecutive query blocks of a head and walks the union of their KV
// lists in ascending order (Eq. 5: each query block multiplies only the tiles on its own
// list).  K/V tiles stream from the raster layout straight into an LDS ring by global->LDS
// DMA (no staging registers, no transposition pass: the tile format of bsa_mfma.h serves both
// the row fragments of K and the transposed fragments of V) while earlier tiles are being
// multiplied; one barrier per tile.  Forward, per tile and wavefront (32 queries on the MFMA column
// index): S^T = K Q^T, online softmax in the exp2 domain, O^T += V^T P^T.
//
//   n_keep <= 32 : four wavefronts (one per query block), two tiles in the ring, two
//                  workgroups per CU: while one waits at its barrier the other multiplies;
//   n_keep  > 32 : eight wavefronts, two per query block splitting its queries, four tiles
//                  in the ring, one workgroup per CU (also the dense baseline's shape).
//   n_keep <= 16 : as the first, but a wavefront carries two query blocks (16 MFMA columns
//                  each) and the workgroup eight.
// Token filling (Sec. 3.2.2) happens in the epilogue: the rows of the critical tokens (one per
// window of the block) are parked in LDS and copied to their windows' pruned positions.
#include "bsa_pipe.h"

namespace bsa {

bool mfma_supported(const Geom& g, int dtype, int n_keep) {
  return dtype == BSA_BF16 && g.Bk == PBK && (g.d == 128 || g.d == 64) && n_keep <= PBK;
}

// The walk: a whole unit, or one segment of a split unit, whose unnormalised accumulators, running maxima and sums go
// to a.part (fwd_combine_kernel merges them).
// PACK (n_keep <= 16): a wavefront carries two query blocks, 16 columns of its 32-column MFMA
// tile each, so a workgroup covers eight blocks; a tile that only one of the two lists holds
// is masked (-inf) in the other block's columns.
template <int D, bool SPLITQ, bool PACK>
__global__ __launch_bounds__(SPLITQ ? 512 : 256, 2) void fwd_pipe_kernel(Geom g, AttnArgs a) {
  static_assert(!(PACK && SPLITQ), "packing is for short retained sets");
  constexpr int PG = PACK ? 2 * bsa::PG : bsa::PG;  // query blocks per workgroup
  constexpr int NT = SPLITQ ? 512 : 256;  // threads
  constexpr int NB = SPLITQ ? 4 : 2;      // LDS ring depth (tiles)
  constexpr int RB = D * 2;               // bytes per tile row
  constexpr int CPR = D / 8;              // 16-byte chunks per row
  constexpr int TILE = PBK * RB;          // bytes of one K (or V) tile
  constexpr int NI = PBK * CPR / NT;      // DMA instructions per thread per K (or V) tile
  constexpr int DT = D / 32, DS = D / 16;
  extern __shared__ __align__(16) uint8_t smem[];
  uint8_t* ring = smem;                                                  // [NB][K tile | V tile]
  uint32_t* masks = reinterpret_cast<uint32_t*>(smem + NB * 2 * TILE);   // [PG][W]
  __shared__ int koff[PBK];
  __shared__ float cen_lse[PG][PBK];  // per window
  __shared__ uint32_t keepbits[PG][2];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int grp = lane >> 5, col = lane & 31;
  // Eight wavefronts: the two of a query block are neighbours, so they sit on two SIMDs (a
  // workgroup's wavefronts go round the four) and a tile that one block lists occupies two matrix cores.
  // With both on one SIMD (wavefronts w and w + 4) the others idled for such a tile: 23,296 tokens, 12 heads,
  // d = 64, every query retained, half of the blocks listed: 1.69 ms against 1.56, dQ 1.86 against 1.62.
  const int sub = SPLITQ ? (wave & 1) : 0;                 // which 32 queries of the block
  const int qb0 = PACK ? 2 * wave : SPLITQ ? (wave >> 1) : wave;  // the wavefront's (first) query block within the workgroup
  const int qb = PACK ? qb0 + (col >> 4) : qb0;            // the lane's
  constexpr int NOWN = PACK ? 2 : 1;
  constexpr int NW = NT / 64;              // wavefronts
  constexpr int NREG = (D / 32) * 16 + 2;  // floats per lane of a partial result: O^T tile, m, l
  const int ngroups = (g.N + PG - 1) / PG;
  Item it;
  if (!item_of(blockIdx.x, ngroups * g.B * g.H, a.split_S, a.split_n, it)) return;
  if (lists_are_long(g, a)) return;
  const int unit = it.unit;
  const int64_t bh = unit / ngroups;
  const int i0 = (unit % ngroups) * PG + qb0;  // the wavefront's first query block
  const int i = (unit % ngroups) * PG + qb;    // the lane's query block
  const bool valid = i < g.N;
  const int64_t row = bh * g.N + i;
  const int W = (g.N + 31) / 32;
  const uint16_t* Qh = static_cast<const uint16_t*>(a.Q) + bh * g.L * D;
  const uint16_t* Kh = static_cast<const uint16_t*>(a.K) + bh * g.L * D;
  const uint16_t* Vh = static_cast<const uint16_t*>(a.V) + bh * g.L * D;
  uint16_t* Oh = static_cast<uint16_t*>(a.O_out) + bh * g.L * D;
  float* Lh = a.LSE_out + bh * g.L;

  if (tid < PBK) koff[tid] = intra_offset(g, tid);
  for (int k = tid; k < PG * W; k += NT) masks[k] = 0u;
  if (tid < 2 * PG) keepbits[tid >> 1][tid & 1] = 0u;
  __syncthreads();
  if (sub == 0) {
#pragma unroll
    for (int o2 = 0; o2 < NOWN; ++o2) {  // the wavefront's own list(s)
      const int ib = i0 + o2, ql = qb0 + o2;
      if (ib >= g.N) continue;
      if (g.dense) {
        for (int w = lane; w < W; w += 64)
          masks[ql * W + w] = (w * 32 + 32 <= g.N) ? 0xffffffffu : ((1u << (g.N - w * 32)) - 1u);
      } else {
        const int64_t rw = bh * g.N + ib;
        const int beg = a.q2k_ptr[rw], cnt = a.q2k_ptr[rw + 1] - beg;
        for (int t = lane; t < cnt; t += 64) {
          const int j = a.q2k_idx[beg + t];
          if ((unsigned)j < (unsigned)g.N) atomicOr(&masks[ql * W + (j >> 5)], 1u << (j & 31));
        }
      }
    }
  }

  // DMA plan of this thread: LDS slot (tid + NT n) of a tile is position p of row r and
  // receives chunk p ^ swz<D>(r) of that row from global memory.
  uint32_t goff[NI];  // bytes, relative to the block origin
#pragma unroll
  for (int n = 0; n < NI; ++n) {
    const int slot = tid + NT * n, r = slot / CPR, c = (slot % CPR) ^ swz<D>(r);
    goff[n] = (uint32_t)(koff[r] * D + c * 8) * 2u;
  }
  const uint32_t lds_wave = uniform_lds(ring + wave * 1024);
  auto issue = [&](int jb, int b) {  // addresses: scalar base of the block + the lane's offset; nothing vector per instruction
    const int64_t origin = (int64_t)block_origin_fast(g, jb) * D;
    const uint64_t kbase = uniform64(Kh + origin), vbase = uniform64(Vh + origin);
    const uint32_t kdst = lds_wave + b * 2 * TILE;
#pragma unroll
    for (int n = 0; n < NI; ++n) dma16_raw(kbase, goff[n], kdst + n * (NT * 16));
#pragma unroll
    for (int n = 0; n < NI; ++n) dma16_raw(vbase, goff[n], kdst + TILE + n * (NT * 16));
  };

  // Q^T fragments (B operand): lane (col, grp) holds channels 16 s + 8 grp .. +7 of its query
  const int qpos = PACK ? (col & 15) : 32 * sub + col;
  int qid = -1, qtok = 0;
  if (valid && qpos < a.n_keep) {
    qid = g.dense ? qpos : min(max(a.keep_idx[row * a.n_keep + qpos], 0), PBK - 1);
    qtok = block_origin(g, i) + koff[qid];
    atomicOr(&keepbits[qb][qid >> 5], 1u << (qid & 31));
  }
  bf16x8 qf[DS];
#pragma unroll
  for (int s = 0; s < DS; ++s) {
    u32x4 v = {0u, 0u, 0u, 0u};
    if (qid >= 0) v = *reinterpret_cast<const u32x4*>(Qh + (int64_t)qtok * D + 16 * s + 8 * grp);
    qf[s] = as_frag(v);
  }
#pragma unroll
  for (int s = 0; s < DS; ++s) settle(qf[s]);

  // per-lane LDS offsets of the two fragment kinds
  int koffs[DS];  // row fragment of tile row (32 kt + col): chunk 2 s + grp, swizzled
#pragma unroll
  for (int s = 0; s < DS; ++s) koffs[s] = col * RB + (((2 * s + grp) ^ swz<D>(col)) << 4);
  // transposed fragment (channel tile dt, 16-row step ks, half h): lane L of a 16-lane group
  // points at 8 bytes of tile row 16 ks + 8 h + 4 grp + L/4, channels 32 dt + 16 (q16&1) + 4 (L%4) .. +3
  const int L16 = lane & 15, q16 = lane >> 4, rsub = L16 >> 2, jj = L16 & 3;
  const int cl = 2 * (q16 & 1) + (jj >> 1), rhi = D == 128 ? rsub : (rsub >> 1);
  int voffs[2][DT];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
      voffs[h][dt] = (8 * h + 4 * grp + rsub) * RB + ((((dt ^ rhi) << 2) | (cl ^ (2 * h + grp))) << 4) + 8 * (jj & 1);

  f32x16 o[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;
  // The running maximum starts at a finite value: relative to -inf the exponents of a tile of nothing but -inf
  // logits would be NaN, and wherever a walk or a segment of one begins with it, it has to weigh nothing (packed: a
  // block that has seen no key yet stays at -inf, and the exponents are relative to 0).  The sum starts at -0, which
  // the first tile turns into +0 or more.
  constexpr float kLowest = PACK ? -INFINITY : -3.4e38f;
  float m = kLowest, l = PACK ? 0.f : -0.f;
  const float c2 = a.sm_scale * kLog2e;
  __syncthreads();
  if (it.nseg > 1 && a.split_by_lists) {  // (at the top, the prologue would wait for these loads)
    it.nseg = min(it.nseg, max(2, pairs_of(g, a.q2k_ptr, unit, ngroups, PG) / kSegPairs));
    if (it.seg >= it.nseg) return;
  }

  // partial results of split unit sidx: [segment][wavefront][NREG][64 lanes] floats
  float* part = it.sidx >= 0 ? a.part + ((int64_t)it.sidx * a.split_S * NW + wave) * (NREG * 64) + lane : nullptr;
  WalkN<PG, NOWN> walk(masks, W, qb0);  // runs NB-1 tiles ahead of the multiplication; `pending` remembers
  int issued = 0;                      // for the tiles in flight which of this wavefront's lists have them (2 bits a tile)
  uint32_t pending = 0;
  if (it.nseg > 1) walk.restrict_to(it.seg, it.nseg);
#pragma unroll
  for (int k = 0; k < NB - 1; ++k) {
    uint32_t mk = 0;
    const int jb = walk.next(mk);
    if (jb >= 0) {
      issue(jb, k);
      pending |= mk << (2 * k);
      ++issued;
    }
  }
  for (int t = 0; t < issued; ++t) {
    // tile t must have landed; up to NB-2 younger tiles may stay in flight (2*NI DMAs each)
    const int ahead = issued - t - 1;
    if (NB >= 4 && ahead >= 2) {
      static_assert(2 * NI == 4 || 2 * NI == 2 || NB < 4, "wait immediates below assume 2 or 4 DMAs per tile");
      if (2 * NI == 4) BSA_WAIT_VM(8); else BSA_WAIT_VM(4);
    } else if (NB >= 3 && ahead == 1) {
      if (2 * NI == 4) BSA_WAIT_VM(4); else BSA_WAIT_VM(2);
    } else {
      BSA_WAIT_VM(0);
    }
    raw_barrier();  // tile t visible to all; everyone is done with tile t-1, whose buffer is refilled now
    {
      uint32_t mn = 0;
      const int jn = walk.next(mn);
      if (jn >= 0) {
        issue(jn, (t + NB - 1) & (NB - 1));
        pending |= mn << (2 * (NB - 1));
        ++issued;
      }
    }
    const uint32_t mbits = pending & 3u;
    const bool mine = mbits != 0;
    pending >>= 2;
    if (mine) {
      // 64 keys x this wavefront's 32 queries.  The 4*DS A fragments of the tile (K rows for
      // both key halves, then V^T) are read from LDS through a ring of RING register
      // fragments, RING MFMAs ahead of their use.  Matrix, vector and LDS instructions of a
      // SIMD co-execute only in part on this chip (measured: the tile's mix keeps the matrix
      // core at most 62 % busy with two wavefronts that never wait), and the LDS -> MFMA chain is
      // the critical path of a tile, so the vector work per tile is kept minimal.
      const uint8_t* Kb = ring + (t & (NB - 1)) * 2 * TILE;
      const uint8_t* Vb = Kb + TILE;
      constexpr int RING = 8, NF = 2 * DS + 4 * DT;
      auto frag = [&](int f) -> bf16x8 {
        if (f < 2 * DS) return lds_frag(reinterpret_cast<const uint16_t*>(Kb + 32 * (f / DS) * RB + koffs[f % DS]));
        const int v = f - 2 * DS, ks = v / DT, dt = v % DT;
        return lds_frag_tr(Vb + voffs[0][dt] + 16 * ks * RB, Vb + voffs[1][dt] + 16 * ks * RB);
      };
      bf16x8 fr[RING];
#pragma unroll
      for (int f = 0; f < RING; ++f) fr[f] = frag(f);
      BSA_FENCE();
      f32x16 s[2];
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int r = 0; r < 16; ++r) s[kt][r] = 0.f;
#pragma unroll
      for (int f = 0; f < 2 * DS; ++f) {
        s[f / DS] = mfma32(fr[f % RING], qf[f % DS], s[f / DS]);
        if (f + RING < NF) fr[f % RING] = frag(f + RING);
        if (f & 1) BSA_FENCE();
      }
      if (PACK && mbits != 3u && !((mbits >> (col >> 4)) & 1u)) {  // the tile is not on this lane's block's list
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
          for (int r = 0; r < 16; ++r) s[kt][r] = -INFINITY;
      }
      float mx = s[0][0];
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[kt][r]);
      mx = pair_max(mx);
      const float mtrue = fmaxf(m, mx * c2);  // c2 > 0: the maximum commutes with the scaling
      const float mnew = (PACK && mtrue == -INFINITY) ? 0.f : mtrue;
      const float alpha = __builtin_amdgcn_exp2f(m - mnew);
      float sum0 = 0.f, sum1 = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        s[0][r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[0][r], c2, -mnew));
        s[1][r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[1][r], c2, -mnew));
        sum0 += s[0][r];
        sum1 += s[1][r];
      }
      l = l * alpha + (sum0 + sum1);  // per-lane partial; the lane pair is summed at the end
      m = mtrue;
      if (__builtin_amdgcn_ballot_w64(alpha != 1.f)) {  // rescale only when some row's maximum moved
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
      }
      bf16x8 pf[4];
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) pf[ks] = d_to_b(s[ks >> 1], ks & 1);
      BSA_FENCE();
#pragma unroll
      for (int f = 2 * DS; f < NF; ++f) {
        const int v = f - 2 * DS;  // V^T fragments in (key step, channel tile) order: consecutive MFMAs hit different accumulators
        o[v % DT] = mfma32(fr[f % RING], pf[v / DT], o[v % DT]);
        if (f + RING < NF) fr[f % RING] = frag(f + RING);
        if (f & 1) BSA_FENCE();
      }
    }
  }

  if (it.nseg > 1) {  // a segment: leave the partial result, the combine launch finishes the unit
    float* ps = part + (int64_t)it.seg * NW * NREG * 64;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) ps[(dt * 16 + r) * 64] = o[dt][r];
    ps[(NREG - 2) * 64] = m;
    ps[(NREG - 1) * 64] = l;
    return;
  }
  // epilogue: normalise, store the retained rows, park the rows of the windows' critical tokens
  // (in the tile ring, idle now) for the fill
  uint16_t* cen_rows = reinterpret_cast<uint16_t*>(smem);  // [PG][nwin][D]
  const float ltot = pair_sum(l);
  // No mass: an empty list gives zeros, a list of nothing but -inf logits NaN (packed, where a tile of the other
  // block's list counts as one of them, zeros for both).
  const float inv = ltot > 0.f ? 1.f / ltot : PACK || __builtin_signbit(ltot) ? 0.f : NAN;
  const float lse = ltot > 0.f ? (m + __builtin_amdgcn_logf(ltot)) * kLn2 : -INFINITY;
  __syncthreads();  // every wavefront is done with the ring
  if (qid >= 0) {
    const int win = window_of(g, qid);
    const bool is_center = !g.dense && qid == window_center(g, win);
    uint16_t* park = cen_rows + ((size_t)qb * g.nwin + win) * D;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        u32x2 v;
        v.x = pack_bf16(o[dt][4 * r4 + 0] * inv, o[dt][4 * r4 + 1] * inv);
        v.y = pack_bf16(o[dt][4 * r4 + 2] * inv, o[dt][4 * r4 + 3] * inv);
        const int ch = 32 * dt + 8 * r4 + 4 * grp;
        *reinterpret_cast<u32x2*>(Oh + (int64_t)qtok * D + ch) = v;
        if (is_center) *reinterpret_cast<u32x2*>(park + ch) = v;
      }
    if (grp == 0) {
      Lh[qtok] = lse;
      if (is_center) cen_lse[qb][win] = lse;
    }
  }
  __syncthreads();
  // token filling: lane c of the block's first wavefront owns intra-block token c and, if it
  // was pruned, copies the row of its window's critical token
  if (!g.dense && sub == 0) {
#pragma unroll
    for (int o2 = 0; o2 < NOWN; ++o2) {  // the wavefront's own block(s)
      const int ib = i0 + o2, ql = qb0 + o2;
      if (ib >= g.N) continue;
      const bool kept = (keepbits[ql][lane >> 5] >> (lane & 31)) & 1u;
      const int win = window_of(g, lane);
      const bool have = (keepbits[ql][window_center(g, win) >> 5] >> (window_center(g, win) & 31)) & 1u;
      if (!kept && have) {
        const int64_t tok = block_origin(g, ib) + koff[lane];
        const uint16_t* src = cen_rows + ((size_t)ql * g.nwin + win) * D;
#pragma unroll
        for (int q = 0; q < D / 8; ++q)
          *reinterpret_cast<u32x4*>(Oh + tok * D + 8 * q) = *reinterpret_cast<const u32x4*>(src + 8 * q);
        Lh[tok] = cen_lse[ql][win];
      }
    }
  }
}

// =====================================================================================
// Backward, same streaming scheme.  Three kernels, no floating-point atomics:
//   pre   per query block: retained Q rows and the folded upstream gradient g (dO of the
//         row; for the center row plus the dO of every pruned token, the gradient of the
//         fill copy) as bf16 tiles in the swizzled LDS format, delta = <g, O> and LSE in the
//         exp2 domain: one contiguous record per query block in the workspace.
//   dQ    the forward's walk (four query blocks per workgroup, union of their KV lists):
//         S^T = K Q^T, dP^T = V G^T, dS^T = P^T (dP^T - delta), dQ^T += K^T dS^T, one key half
//         at a time; K^T comes from the same K tile through transposed LDS reads.
//   dKV   bsa_attn_dkv.hip: a workgroup owns one KV block and streams its list's records.
// =====================================================================================

template <int D, int NQT>
__global__ __launch_bounds__(256) void bwd_pre_pipe_kernel(Geom g, AttnArgs a) {
  using R = BwdRec<D>;
  constexpr int NQ = 32 * NQT;
  constexpr int CPR = D / 8;       // 16-byte chunks per row
  constexpr int RPP = 256 / CPR;   // rows covered by one pass of the workgroup (a row = CPR adjacent lanes)
  extern __shared__ __align__(16) float fold_mem[];
  float* partial = fold_mem;                // [RPP][D] column sums of pruned dO rows, per row group
  float* foldw = fold_mem + RPP * D;        // [nwin][D] the same, complete, per window
  __shared__ int keepflag[PBK];
  __shared__ int qtok[NQ];
  __shared__ short qwin[NQ];   // window whose critical token the retained row is, or -1
  __shared__ int koff[PBK];
  __shared__ short wtok[PBK];     // tokens grouped by window, ascending id inside a window
  const int tid = threadIdx.x;
  const int c = tid % CPR, rg = tid / CPR;
  const int64_t row = blockIdx.x;
  const int64_t bh = row / g.N;
  const int i = row % g.N;
  const uint16_t* Qh = static_cast<const uint16_t*>(a.Q) + bh * g.L * D;
  const uint16_t* Oh = static_cast<const uint16_t*>(a.O) + bh * g.L * D;
  const uint16_t* dOh = static_cast<const uint16_t*>(a.dO) + bh * g.L * D;
  const float* Lh = a.LSE_in + bh * g.L;
  // a.pack (n_keep <= 16): two query blocks share a record, rows 0..15 the even block's, 16..31 the odd one's
  const int64_t recno = a.pack ? bh * ((g.N + 1) / 2) + (i >> 1) : row * NQT;
  const int r0 = a.pack ? 16 * (i & 1) : 0, nrows = a.pack ? 16 : NQ;
  uint8_t* rec0 = static_cast<uint8_t*>(a.ws) + recno * (int64_t)R::BYTES;
  const int origin = block_origin(g, i);

  if (tid < PBK) {
    koff[tid] = intra_offset(g, tid);
    keepflag[tid] = 0;
    if (!g.dense) {  // position of token tid inside its window: raster order of its local coordinates
      const int cw = tid % g.Cw, ch = (tid / g.Cw) % g.Ch, ct = tid / (g.Cw * g.Ch);
      const int k = ((ct % g.Wt) * g.Wh + ch % g.Wh) * g.Ww + cw % g.Ww;
      wtok[window_of(g, tid) * g.Wk + k] = (short)tid;
    }
  }
  __syncthreads();
  if (tid < NQ) {
    int k = -1;
    if (tid < a.n_keep) k = g.dense ? tid : min(max(a.keep_idx[row * a.n_keep + tid], 0), PBK - 1);
    qtok[tid] = k >= 0 ? origin + koff[k] : -1;
    qwin[tid] = (short)((k >= 0 && !g.dense && center_of(g, k) == k) ? window_of(g, k) : -1);
    if (k >= 0) keepflag[k] = 1;
  }
  __syncthreads();

  // Gradient of the fill copies: per window, the dO rows of its pruned tokens summed per
  // channel.  G row groups share a window: each adds every G-th token of the window in
  // ascending id, then the groups' sums are added in order.
  if (!g.dense) {
    const int G = g.nwin >= RPP ? 1 : RPP / g.nwin;  // row groups per window
    const int WB = g.nwin >= RPP ? RPP : g.nwin;     // windows per batch
    for (int w0 = 0; w0 < g.nwin; w0 += WB) {
      const int w = w0 + rg / G, sub = rg % G;
      float acc[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = 0.f;
      if (rg < WB * G && w < g.nwin) {
        for (int k = sub; k < g.Wk; k += G) {
          const int u = wtok[w * g.Wk + k];
          if (keepflag[u]) continue;
          const u32x4 pv = *reinterpret_cast<const u32x4*>(dOh + (int64_t)(origin + koff[u]) * D + 8 * c);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            acc[2 * e] += __uint_as_float(pv[e] << 16);
            acc[2 * e + 1] += __uint_as_float(pv[e] & 0xffff0000u);
          }
        }
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) partial[rg * D + 8 * c + e] = acc[e];
      __syncthreads();
      for (int t = tid; t < WB * D; t += 256) {
        const int wl = t / D, ch = t % D;
        if (w0 + wl < g.nwin) {
          float sum = 0.f;
          for (int k = 0; k < G; ++k) sum += partial[(wl * G + k) * D + ch];
          foldw[(w0 + wl) * D + ch] = sum;
        }
      }
      __syncthreads();
    }
  }

  // a last block without a partner also writes the partner's half of the record: padding rows
  const int nwrite = (a.pack && (i & 1) == 0 && i + 1 == g.N) ? 32 : nrows;
  for (int q = rg; q < nwrite; q += RPP) {
    const int tok = q < nrows ? qtok[q] : -1;
    u32x4 qv = {0u, 0u, 0u, 0u}, gv = {0u, 0u, 0u, 0u};
    float dsum = 0.f;
    if (tok >= 0) {
      qv = *reinterpret_cast<const u32x4*>(Qh + (int64_t)tok * D + 8 * c);
      gv = *reinterpret_cast<const u32x4*>(dOh + (int64_t)tok * D + 8 * c);
      const u32x4 ov = *reinterpret_cast<const u32x4*>(Oh + (int64_t)tok * D + 8 * c);
      float gf[8];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        gf[2 * e] = __uint_as_float(gv[e] << 16);
        gf[2 * e + 1] = __uint_as_float(gv[e] & 0xffff0000u);
      }
      const int w = qwin[q];
      if (w >= 0) {  // a window's critical token: its own dO plus its window's fill copies
#pragma unroll
        for (int e = 0; e < 8; ++e) gf[e] += foldw[w * D + 8 * c + e];
#pragma unroll
        for (int e = 0; e < 4; ++e) gv[e] = pack_bf16(gf[2 * e], gf[2 * e + 1]);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        dsum += gf[2 * e] * __uint_as_float(ov[e] << 16);
        dsum += gf[2 * e + 1] * __uint_as_float(ov[e] & 0xffff0000u);
      }
    }
    const int rq = (r0 + q) & 31;      // row of the record
    uint8_t* rec = rec0 + (NQT == 2 ? (q >> 5) * R::BYTES : 0);
    const int pos = c ^ swz<D>(rq);    // chunk position inside the swizzled row
    *reinterpret_cast<u32x4*>(rec + R::QC + rq * R::RB + pos * 16) = qv;
    *reinterpret_cast<u32x4*>(rec + R::GC + rq * R::RB + pos * 16) = gv;
#pragma unroll
    for (int msk = 1; msk < CPR; msk <<= 1) dsum += __shfl_xor(dsum, msk);  // the row's CPR lanes
    if (c == 0) {
      // padding rows, and rows whose list was empty (LSE = -inf): +inf, so that exp2(x - inf) = 0
      const float lse = tok >= 0 ? Lh[tok] : INFINITY;
      reinterpret_cast<float*>(rec + R::LS)[rq] = lse == -INFINITY ? INFINITY : lse * kLog2e;
      reinterpret_cast<float*>(rec + R::DL)[rq] = -dsum;  // as dK/dV adds it
    }
  }
}

// ------------------------------------------------------------------------------- dQ
// COMBINE as in the forward: segments of a split unit leave their dQ^T sums in a.part.
// PACK as in the forward: two query blocks per wavefront when n_keep <= 16.
template <int D, bool SPLITQ, bool COMBINE, bool PACK>
__global__ __launch_bounds__(SPLITQ ? 512 : 256, 2) void bwd_dq_pipe_kernel(Geom g, AttnArgs a) {
  static_assert(!(PACK && SPLITQ), "packing is for short retained sets");
  constexpr int PG = PACK ? 2 * bsa::PG : bsa::PG;  // query blocks per workgroup
  using R = BwdRec<D>;
  constexpr int NT = SPLITQ ? 512 : 256;
  constexpr int NB = SPLITQ ? 4 : 2;
  constexpr int RB = D * 2, CPR = D / 8, TILE = PBK * RB, NI = PBK * CPR / NT;
  constexpr int DT = D / 32, DS = D / 16;
  extern __shared__ __align__(16) uint8_t smem[];
  uint8_t* ring = smem;                                                  // [NB][K tile | V tile]
  uint32_t* masks = reinterpret_cast<uint32_t*>(smem + NB * 2 * TILE);   // [PG][W]
  __shared__ int koff[PBK];
  __shared__ uint32_t keepbits[PG][2];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int grp = lane >> 5, col = lane & 31;
  const int sub = SPLITQ ? (wave & 1) : 0;  // as in the forward
  const int qb0 = PACK ? 2 * wave : SPLITQ ? (wave >> 1) : wave;  // the wavefront's (first) query block within the workgroup
  const int qb = PACK ? qb0 + (col >> 4) : qb0;  // the lane's
  constexpr int NOWN = PACK ? 2 : 1;
  constexpr int NW = NT / 64;          // wavefronts
  constexpr int NREG = (D / 32) * 16;  // floats per lane of a partial result: the dQ^T tile
  const int ngroups = (g.N + PG - 1) / PG;
  Item it;
  if (COMBINE ? !split_item_of(blockIdx.x, ngroups * g.B * g.H, a.split_S, a.split_n, it)
              : !item_of(blockIdx.x, ngroups * g.B * g.H, a.split_S, a.split_n, it))
    return;
  const int unit = it.unit;
  const int64_t bh = unit / ngroups;
  const int i0 = (unit % ngroups) * PG + qb0;
  const int i = (unit % ngroups) * PG + qb;
  const bool valid = i < g.N;
  const int64_t row = bh * g.N + i;
  const int W = (g.N + 31) / 32;
  const uint16_t* Kh = static_cast<const uint16_t*>(a.K) + bh * g.L * D;
  const uint16_t* Vh = static_cast<const uint16_t*>(a.V) + bh * g.L * D;
  uint16_t* dQh = static_cast<uint16_t*>(a.dQ) + bh * g.L * D;
  // packed: the wavefront's two blocks (i0 even) share one record, and the lane's row in it is its column
  const uint8_t* rec = static_cast<const uint8_t*>(a.ws) +
                       (PACK ? bh * ((g.N + 1) / 2) + (i0 >> 1) : SPLITQ ? row * 2 + sub : row) * (int64_t)R::BYTES;

  if (tid < PBK) koff[tid] = intra_offset(g, tid);
  if (!COMBINE)
    for (int k = tid; k < PG * W; k += NT) masks[k] = 0u;
  if (tid < 2 * PG) keepbits[tid >> 1][tid & 1] = 0u;
  __syncthreads();
  if (!COMBINE && sub == 0) {
#pragma unroll
    for (int o2 = 0; o2 < NOWN; ++o2) {  // the wavefront's own list(s)
      const int ib = i0 + o2, ql = qb0 + o2;
      if (ib >= g.N) continue;
      if (g.dense) {
        for (int w = lane; w < W; w += 64)
          masks[ql * W + w] = (w * 32 + 32 <= g.N) ? 0xffffffffu : ((1u << (g.N - w * 32)) - 1u);
      } else {
        const int64_t rw = bh * g.N + ib;
        const int beg = a.q2k_ptr[rw], cnt = a.q2k_ptr[rw + 1] - beg;
        for (int t = lane; t < cnt; t += 64) {
          const int j = a.q2k_idx[beg + t];
          if ((unsigned)j < (unsigned)g.N) atomicOr(&masks[ql * W + (j >> 5)], 1u << (j & 31));
        }
      }
    }
  }
  uint32_t goff[NI];  // bytes, relative to the block origin
#pragma unroll
  for (int n = 0; n < NI; ++n) {
    const int slot = tid + NT * n, r = slot / CPR, c = (slot % CPR) ^ swz<D>(r);
    goff[n] = (uint32_t)(koff[r] * D + c * 8) * 2u;
  }
  const uint32_t lds_wave = uniform_lds(ring + wave * 1024);
  auto issue = [&](int jb, int b) {  // addresses: scalar base of the block + the lane's offset; nothing vector per instruction
    const int64_t origin = (int64_t)block_origin_fast(g, jb) * D;
    const uint64_t kbase = uniform64(Kh + origin), vbase = uniform64(Vh + origin);
    const uint32_t kdst = lds_wave + b * 2 * TILE;
#pragma unroll
    for (int n = 0; n < NI; ++n) dma16_raw(kbase, goff[n], kdst + n * (NT * 16));
#pragma unroll
    for (int n = 0; n < NI; ++n) dma16_raw(vbase, goff[n], kdst + TILE + n * (NT * 16));
  };

  // Q^T and G^T fragments (B operands) and the row constants, from the query block's record
  const int qpos = PACK ? (col & 15) : 32 * sub + col;
  const int rrow = col;  // row of the record
  int qid = -1, qtok = 0;
  float lse2 = INFINITY, delta = 0.f;
  if (valid && qpos < a.n_keep) {
    qid = g.dense ? qpos : min(max(a.keep_idx[row * a.n_keep + qpos], 0), PBK - 1);
    qtok = block_origin(g, i) + koff[qid];
    atomicOr(&keepbits[qb][qid >> 5], 1u << (qid & 31));
    lse2 = reinterpret_cast<const float*>(rec + R::LS)[rrow];
    delta = -reinterpret_cast<const float*>(rec + R::DL)[rrow];
  }
  bf16x8 qf[DS], gf[DS];
#pragma unroll
  for (int s = 0; s < DS; ++s) {
    u32x4 qv = {0u, 0u, 0u, 0u}, gv = {0u, 0u, 0u, 0u};
    if (!COMBINE && qid >= 0) {
      const int off = rrow * RB + (((2 * s + grp) ^ swz<D>(rrow)) << 4);
      qv = *reinterpret_cast<const u32x4*>(rec + R::QC + off);
      gv = *reinterpret_cast<const u32x4*>(rec + R::GC + off);
    }
    qf[s] = as_frag(qv);
    gf[s] = as_frag(gv);
  }
  settle(lse2);
  settle(delta);
#pragma unroll
  for (int s = 0; s < DS; ++s) {
    settle(qf[s]);
    settle(gf[s]);
  }

  int koffs[DS];
#pragma unroll
  for (int s = 0; s < DS; ++s) koffs[s] = col * RB + (((2 * s + grp) ^ swz<D>(col)) << 4);
  const int L16 = lane & 15, q16 = lane >> 4, rsub = L16 >> 2, jj = L16 & 3;
  const int cl = 2 * (q16 & 1) + (jj >> 1), rhi = D == 128 ? rsub : (rsub >> 1);
  int voffs[2][DT];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
      voffs[h][dt] = (8 * h + 4 * grp + rsub) * RB + ((((dt ^ rhi) << 2) | (cl ^ (2 * h + grp))) << 4) + 8 * (jj & 1);

  f32x16 dq[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) dq[dt][r] = 0.f;
  const float c2 = a.sm_scale * kLog2e;
  __syncthreads();
  if (it.nseg > 1 && a.split_by_lists) {  // (at the top, the prologue would wait for these loads)
    it.nseg = min(it.nseg, max(2, pairs_of(g, a.q2k_ptr, unit, ngroups, PG) / kSegPairs));
    if (it.seg >= it.nseg) return;
  }

  // partial results of split unit sidx: [segment][wavefront][NREG][64 lanes] floats
  float* part = it.sidx >= 0 ? a.part + ((int64_t)it.sidx * a.split_S * NW + wave) * (NREG * 64) + lane : nullptr;
  if (COMBINE) {
    for (int sg = 0; sg < it.nseg; ++sg) {
      const float* ps = part + (int64_t)sg * NW * NREG * 64;
      float v[NREG];  // all loads of the segment in flight together
#pragma unroll
      for (int k = 0; k < NREG; ++k) v[k] = __builtin_nontemporal_load(ps + k * 64);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) dq[dt][r] += v[dt * 16 + r];
    }
  }
  WalkN<PG, NOWN> walk(masks, W, qb0);
  int issued = 0;
  uint32_t pending = 0;  // two bits per tile in flight: which of the wavefront's lists hold it
  if (!COMBINE) {
    if (it.nseg > 1) walk.restrict_to(it.seg, it.nseg);
#pragma unroll
    for (int k = 0; k < NB - 1; ++k) {
      uint32_t mk = 0;
      const int jb = walk.next(mk);
      if (jb >= 0) {
        issue(jb, k);
        pending |= mk << (2 * k);
        ++issued;
      }
    }
  }
  for (int t = 0; t < issued; ++t) {
    const int ahead = issued - t - 1;
    if (NB >= 4 && ahead >= 2) {
      if (2 * NI == 4) BSA_WAIT_VM(8); else BSA_WAIT_VM(4);
    } else if (NB >= 3 && ahead == 1) {
      if (2 * NI == 4) BSA_WAIT_VM(4); else BSA_WAIT_VM(2);
    } else {
      BSA_WAIT_VM(0);
    }
    raw_barrier();
    {
      uint32_t mn = 0;
      const int jn = walk.next(mn);
      if (jn >= 0) {
        issue(jn, (t + NB - 1) & (NB - 1));
        pending |= mn << (2 * (NB - 1));
        ++issued;
      }
    }
    const uint32_t mbits = pending & 3u;
    const bool mine = mbits != 0;
    pending >>= 2;
    if (mine) {
      const uint8_t* Kb = ring + (t & (NB - 1)) * 2 * TILE;
      const uint8_t* Vb = Kb + TILE;
      // packed: a tile that is not on this lane's block's list contributes P = 0
      const float lse_t = (PACK && !((mbits >> (col >> 4)) & 1u)) ? INFINITY : lse2;
      // one key half (32 keys) at a time: 2*DS row fragments (K, V alternating), then 2*DT
      // transposed K fragments; a ring of RING register fragments runs ahead of the MFMAs
      constexpr int RING = 8, NF = 2 * DS + 2 * DT;
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        auto frag = [&](int f) -> bf16x8 {
          if (f < 2 * DS) {
            const uint8_t* base = (f & 1) ? Vb : Kb;
            return lds_frag(reinterpret_cast<const uint16_t*>(base + 32 * kt * RB + koffs[f >> 1]));
          }
          const int v = f - 2 * DS, h = v / DT, dt = v % DT, ks = 2 * kt + h;
          return lds_frag_tr(Kb + voffs[0][dt] + 16 * ks * RB, Kb + voffs[1][dt] + 16 * ks * RB);
        };
        bf16x8 fr[RING];
#pragma unroll
        for (int f = 0; f < RING; ++f) fr[f] = frag(f);
        BSA_FENCE();
        f32x16 s, dp;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = dp[r] = 0.f;
#pragma unroll
        for (int f = 0; f < 2 * DS; ++f) {
          if (f & 1) dp = mfma32(fr[f % RING], gf[f >> 1], dp);
          else s = mfma32(fr[f % RING], qf[f >> 1], s);
          if (f + RING < NF) fr[f % RING] = frag(f + RING);
          if (f & 1) BSA_FENCE();
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], c2, -lse_t));
          s[r] = p * (dp[r] - delta);
        }
        const bf16x8 d0 = d_to_b(s, 0), d1 = d_to_b(s, 1);
        BSA_FENCE();
#pragma unroll
        for (int f = 2 * DS; f < NF; ++f) {
          const int v = f - 2 * DS;
          dq[v % DT] = mfma32(fr[f % RING], (v / DT) ? d1 : d0, dq[v % DT]);
          if (f + RING < NF) fr[f % RING] = frag(f + RING);
          if (f & 1) BSA_FENCE();
        }
      }
    }
  }

  if (!COMBINE && it.nseg > 1) {
    float* ps = part + (int64_t)it.seg * NW * NREG * 64;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) ps[(dt * 16 + r) * 64] = dq[dt][r];
    return;
  }
  if (qid >= 0) {
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        u32x2 v;
        v.x = pack_bf16(dq[dt][4 * r4 + 0] * a.sm_scale, dq[dt][4 * r4 + 1] * a.sm_scale);
        v.y = pack_bf16(dq[dt][4 * r4 + 2] * a.sm_scale, dq[dt][4 * r4 + 3] * a.sm_scale);
        *reinterpret_cast<u32x2*>(dQh + (int64_t)qtok * D + 32 * dt + 8 * r4 + 4 * grp) = v;
      }
  }
  __syncthreads();
  // pruned queries take no part in the forward: zero gradient rows
  if (!g.dense && sub == 0) {
#pragma unroll
    for (int o2 = 0; o2 < NOWN; ++o2) {  // the wavefront's own block(s)
      const int ib = i0 + o2, ql = qb0 + o2;
      if (ib >= g.N) continue;
      const bool kept = (keepbits[ql][lane >> 5] >> (lane & 31)) & 1u;
      if (!kept) {
        const int64_t tok = block_origin(g, ib) + koff[lane];
        const u32x4 z = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int q = 0; q < D / 8; ++q) *reinterpret_cast<u32x4*>(dQh + tok * D + 8 * q) = z;
      }
    }
  }
}

// floats per lane of one wavefront's partial result
constexpr int fwd_part_regs(int d) { return (d / 32) * 16 + 2; }
constexpr int dq_part_regs(int d) { return (d / 32) * 16; }

// pack: the packed variant (two query blocks per wavefront, eight per workgroup)
static bool fwd_packs(const Geom& g, int n_keep) { return n_keep <= 16 && !g.dense; }
static SplitPlan pipe_plan(const Geom& g, int n_keep, bool allow, bool pack = false) {
  const bool splitq = n_keep > 32;
  const int pg = pack ? 2 * PG : PG;
  return plan_split(((g.N + pg - 1) / pg) * g.B * g.H, kCUs * (splitq ? 1 : 2), g.N, allow);
}

template <int D, int NQT, bool PACK>
static int launch_bwd_pipe_t(const Geom& g, AttnArgs a, hipStream_t st) {
  using R = BwdRec<D>;
  constexpr bool SPLITQ = NQT == 2;
  constexpr int PGK = PACK ? 2 * PG : PG;
  const int W = (g.N + 31) / 32;
  a.pack = PACK ? 1 : 0;
  const size_t lds_q = (size_t)(SPLITQ ? 4 : 2) * 2 * PBK * D * 2 + (size_t)PGK * W * 4;
  const int nrec_head = PACK ? (g.N + 1) / 2 : g.N;
  const size_t nrec = (size_t)g.B * g.H * nrec_head * NQT;  // records in the workspace
  if (int rc = allow_dynamic_lds<bwd_dq_pipe_kernel<D, SPLITQ, false, PACK>>(lds_q)) return rc;
  if (int rc = grant_bwd_dkv_pipe(g, a)) return rc;
  if (a.stages & BSA_BWD_PRE)  // LDS: per-row-group partial sums + per-window sums of the fill gradient
    hipLaunchKernelGGL((bwd_pre_pipe_kernel<D, NQT>), dim3(g.rows), dim3(256), (size_t)(256 / (D / 8) + g.nwin) * D * 4, st, g, a);
  if (a.stages & BSA_BWD_DQ) {
    const SplitPlan p = pipe_plan(g, a.n_keep, !g.dense, PACK);
    a.split_S = p.S;
    a.split_n = p.n;
    a.split_by_lists = p.by_lists;
    a.part = reinterpret_cast<float*>(static_cast<uint8_t*>(a.ws) + (size_t)R::BYTES * nrec);  // behind the records
    hipLaunchKernelGGL((bwd_dq_pipe_kernel<D, SPLITQ, false, PACK>), dim3(p.grid), dim3(SPLITQ ? 512 : 256), lds_q, st, g, a);
    if (p.units)
      hipLaunchKernelGGL((bwd_dq_pipe_kernel<D, SPLITQ, true, PACK>), dim3(p.units), dim3(SPLITQ ? 512 : 256), 0, st, g, a);
  }
  if (a.stages & BSA_BWD_DKV)
    if (int rc = launch_bwd_dkv_pipe(g, a, st)) return rc;
  return check_launch();
}

int launch_bwd_pipe(const Geom& g, const AttnArgs& a, hipStream_t st) {
  const bool two = a.n_keep > 32;
  if (fwd_packs(g, a.n_keep)) return g.d == 128 ? launch_bwd_pipe_t<128, 1, true>(g, a, st) : launch_bwd_pipe_t<64, 1, true>(g, a, st);
  if (g.d == 128) return two ? launch_bwd_pipe_t<128, 2, false>(g, a, st) : launch_bwd_pipe_t<128, 1, false>(g, a, st);
  return two ? launch_bwd_pipe_t<64, 2, false>(g, a, st) : launch_bwd_pipe_t<64, 1, false>(g, a, st);
}

size_t bwd_workspace_pipe(const Geom& g, int n_keep) {
  const bool two = n_keep > 32;
  const size_t per_rec = g.d == 128 ? BwdRec<128>::BYTES : BwdRec<64>::BYTES;
  const SplitPlan p = pipe_plan(g, n_keep, !g.dense, fwd_packs(g, n_keep));
  const size_t partials = (size_t)p.units * p.S * (two ? 8 : 4) * dq_part_regs(g.d) * 64 * sizeof(float);
  const size_t nrec = fwd_packs(g, n_keep) ? (size_t)g.B * g.H * ((g.N + 1) / 2) : (size_t)g.rows * (two ? 2 : 1);
  return per_rec * nrec + partials;  // records | dQ partials
}

// The other forward kernel's plan keeps to the same workspace.
size_t fwd_workspace_pipe(const Geom& g, int n_keep) {
  if (g.dense) return 0;
  const SplitPlan p = pipe_plan(g, n_keep, true, fwd_packs(g, n_keep));
  return (size_t)p.units * p.S * (n_keep > 32 ? 8 : 4) * fwd_part_regs(g.d) * 64 * sizeof(float);
}

template <int D, bool SPLITQ, bool PACK>
static size_t fwd_pipe_lds(const Geom& g) {
  return (size_t)(SPLITQ ? 4 : 2) * 2 * PBK * D * 2 + (size_t)(PACK ? 2 * PG : PG) * ((g.N + 31) / 32) * 4;
}

// calls f with the constants of the kernel
template <typename F>
static int for_fwd_pipe(const Geom& g, int n_keep, F f) {
  using std::bool_constant;
  auto go = [&](auto D) {
    if (fwd_packs(g, n_keep)) return f(D, bool_constant<false>{}, bool_constant<true>{});
    return n_keep > 32 ? f(D, bool_constant<true>{}, bool_constant<false>{}) : f(D, bool_constant<false>{}, bool_constant<false>{});
  };
  return g.d == 128 ? go(std::integral_constant<int, 128>{}) : go(std::integral_constant<int, 64>{});
}

static int launch_pipe(const Geom& g, AttnArgs a, FwdSplit& split, hipStream_t st) {
  const bool pack = fwd_packs(g, a.n_keep);
  const SplitPlan p = pipe_plan(g, a.n_keep, !g.dense && a.fwd_ws != nullptr, pack);
  split = FwdSplit{p.S, p.n, p.by_lists, pack ? 2 * PG : PG};
  a.split_S = p.S;
  a.split_n = p.n;
  a.split_by_lists = p.by_lists;
  return for_fwd_pipe(g, a.n_keep, [&](auto D, auto SPLITQ, auto PACK) {
    hipLaunchKernelGGL((fwd_pipe_kernel<D, SPLITQ, PACK>), dim3(p.grid), dim3(SPLITQ ? 512 : 256), (fwd_pipe_lds<D, SPLITQ, PACK>(g)), st, g, a);
    return check_launch();
  });
}

// Two forward kernels.  The one of bsa_attn_fwd.hip (walk) costs some 15 us a unit whatever its lists, the one above (pipe) half of
// that under another workgroup's walk, but more a tile.  What walk does for the keys that weigh most in a row costs the more, the sharper
// the logits.  Figures: us, pipe / walk, 12 heads, selected lists of so many blocks on fields with noise of 0.3 (with noise of 1.0).
struct FwdChoice {
  bool walk, pipe;
  int from;  // both are launched, and one ends at once (2 us): walk works from so many listed blocks a row on
};

static FwdChoice choose_forward(const Geom& g, int n_keep) {
  const bool half = fwd_packs(g, n_keep), two = g.dense || n_keep > 32, one = !half && !two;  // tiles a block
  const int units = fwd_walk_units(g, n_keep);
  if (units <= kCUs) {
    // Within one round walk takes a workgroup a unit and no combine launch.  d = 128, 4 heads of 128 blocks, 23 and 72 listed: two
    // tiles a block 66 / 56, 113 / 101 (67 / 63, 114 / 113), one 46 / 41, 72 / 69 (47 / 45, 73 / 74), half 49 / 40, 60 / 57
    // (49 / 41, 61 / 60); half a tile, 12 heads, 72 listed: 134 / 116 (136 / 131).  But pipe, with less than two tiles a block,
    // - where the chip is full of short walks: 48 blocks, 18 and 36 listed, one tile: 46 / 44, 52 / 54 (47 / 50, 53 / 62), half
    //   46 / 46, 47 / 50 (45 / 48, 47 / 55); d = 64, 4 heads of 128 blocks, 71 and 92 listed, one tile: 49 / 49, 54 / 56 (49 / 55, 54 / 62), but
    //   half, 43, 71 and 92: 39 / 35, 43 / 42, 44 / 46 (40 / 39, 44 / 47, 44 / 48);
    // - where units shrink to a block or four and pipe has several segments for each: 1 head, 520 blocks, half a tile, 48, 200 and 520
    //   listed (independent logits with a deviation of 2): 80 / 78, 146 / 176, 196 / 280; 256 blocks, one tile, 200 listed: 88 / 95;
    // and below 16 blocks, where lists are short whatever the threshold (2 heads of 12 blocks, 3 and 12 listed: 16 / 18, 23 / 23).
    const bool full = !two && g.rows >= 512 && g.N <= (one && g.d == 64 ? 128 : 64);
    const bool lone = !two && g.N >= 256 && g.rows <= 640, few = g.N < 16 && !g.dense;
    const bool walk = !full && !lone && !few;
    return {walk, !walk, 0};
  }
  // Beyond, the lists decide, and how long they are is known on the device only.  d = 128:
  // two tiles, 364 blocks, 26, 57 and 179 listed: 500 / 455, 886 / 720, 1944 / 1720 (507 / 534, 889 / 816, 2023 / 1873);
  // one, 26, 57 and 179: 283 / 292, 484 / 444, 1052 / 956 (285 / 328, 489 / 504, 1097 / 1035), 1,100 blocks, 52: 1392 / 1392 (1432 / 1446);
  // half, 26, 57 and 179: 252 / 238, 400 / 370, 664 / 645 (256 / 259, 399 / 395, 671 / 699), 520 blocks, 28: 434 / 344 (434 / 381).
  // d = 64: two tiles, 364 blocks, 27 and 59: 366 / 339, 647 / 526 (363 / 386, 644 / 591); one tile or less hardly ever (520 blocks, one, 29,
  // 67 and 346: 235 / 301, 435 / 494, 1435 / 1594).
  // Fewer blocks: two tiles, 192 blocks, 26, 51 and 161: 233 / 256, 374 / 367, 822 / 814; one, 252 blocks, 27, 56: 206 / 212, 336 / 311 (206 / 242,
  // 346 / 353), 192 blocks, 92: 300 / 337; half, 192 blocks, 26: 175 / 126, but with little more than two rounds of units (24 heads,
  // independent logits, 64 listed) 352 / 424.  Dense, from where the block count is a list's length.
  const int from = g.dense ? (g.d == 128 ? 56 : 40) : two ? 32 : g.d == 64 ? g.N + 1 : one ? 48 : 24;
  const int shortest = g.dense ? 0 : two ? 256 : one ? 320 : units < 2 * kCUs ? 192 : 320;
  const bool walk = g.N >= from && g.N >= shortest;
  return {walk, !walk || !g.dense, from};
}

int launch_fwd_pipe(const Geom& g, const AttnArgs& args, hipStream_t st) {
  AttnArgs a = args;
  const bool splitq = a.n_keep > 32, pack = fwd_packs(g, a.n_keep);
  const auto [walk, pipe, from] = choose_forward(g, a.n_keep);
  a.fwd_long = walk && pipe ? from : 0;
  a.part = static_cast<float*>(a.fwd_ws);
  if (walk)
    if (int rc = grant_fwd_walk(g, a)) return rc;
  if (pipe)
    if (int rc = for_fwd_pipe(g, a.n_keep, [&](auto D, auto SPLITQ, auto PACK) {
          return allow_dynamic_lds<fwd_pipe_kernel<D, SPLITQ, PACK>>(fwd_pipe_lds<D, SPLITQ, PACK>(g));
        }))
      return rc;
  const SplitPlan p = pipe_plan(g, a.n_keep, !g.dense, pack);
  FwdSplit sw{1, 0, 0, 0}, sp{1, 0, 0, 0};
  if (walk)
    if (int rc = launch_fwd_walk(g, a, p.units * p.S * (splitq ? 2 : 1), sw, st)) return rc;
  if (pipe)
    if (int rc = launch_pipe(g, a, sp, st)) return rc;
  return launch_fwd_combine(g, a, sw, sp, st);
}

}  // namespace bsa
