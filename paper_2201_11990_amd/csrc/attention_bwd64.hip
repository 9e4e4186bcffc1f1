// Backward of the fused causal attention with 16 own rows to a wave: bf16 head size 64 and, with P and dS in fp32 (EXACT), head sizes up to 64 and the short sequences of the others up to 192
// (attention_bwd.hip has the rest and says which), with the tiles and fragments of attention_fwd16.hip.
//
// dP = da v^T,  dS = P o (dP - D) with D_t = da_t . a_t,  dq = scale dS k,  dk = scale dS^T q,  dv = P^T da, on 16x16x32 MFMAs with 16 own rows to a wave:
//   dq      : S^T and dP^T = V dO^T with the query on the lane column, dQ^T += K^T dS^T.
//   dk / dv : S = Q K^T, dP = dO V^T with the key on the lane column, dV^T += dO^T P, dK^T += Q^T dS.
// The vector unit bounds it: a tile's exponentials and dS take longer than its MFMAs at head size 64 (the matrix pipes work 36 % of the time), and what hides latency is the number of waves, for which these kernels are
// small (24 waves to a compute unit).  The kernels of attention_bwd.hip, with 32 own rows to a wave and 8 to 16 waves to a unit, took 50 us instead of
// 56 at 2048 tokens x 16 heads and 153 instead of 167 at 4 times that, but 29 instead of 24 at 1024 x 20, 20 instead of 17.6 at 512 x 48 and 12 instead of 9.4 at 128 x 128.
#include "attention_tiles.h"

namespace mtnlg {

namespace {

// The backward kernels: a workgroup owns one 64-row block (queries for dq, keys for dk / dv), 16 rows to each of waves 0-3
// and again to waves 4-7: the two halves of the workgroup take the first and the last 32 rows of every streamed
// tile, and their partial results are merged through LDS at the end.  Half the tile per wave halves the registers
// of its scores and its chain per tile, and no wave idles while the mask leaves work to the other half only.  Blocks are
// handed out in the order of falling work, so a compute unit that got a long block gets a short one after it.  Measured with
// paired blocks and whole tiles before, dq + dk/dv at 2048 tokens x 16 heads: 75 us, now 56.  (In the forward kernel of attention_fwd16.hip, which has fewer registers to
// save, the merge costs more than it gives.)

// Over many sequences the work evens out by itself, and what a workgroup costs besides its tiles counts instead.  PAIRED has half the workgroups: waves 0-3
// and 4-7 own blocks p and nb - 1 - p and take whole tiles, as in attention_fwd16.hip, with nothing to merge.
template <bool PAIRED>
struct BackwardBlocks {
  int block;      // this wave's 64-row block
  int lo, hi;     // lowest and highest of the workgroup's
  bool idle;      // wave-uniform: this wave owns no rows
  __device__ BackwardBlocks(int s, int order, int wave) {
    lo = order;
    hi = PAIRED ? row_blocks(s) - 1 - order : order;
    block = wave >> 2 ? hi : lo;
    idle = PAIRED && wave >> 2 && hi == lo;
  }
  static __host__ __device__ int count(int s) { return PAIRED ? (row_blocks(s) + 1) / 2 : row_blocks(s); }
};

// Partial accumulators of waves 4-7 to waves 0-3 through LDS: 16-byte slots per lane, conflict-free.
__device__ __forceinline__ f32x4 *merge_slots(char *smem, int wave, int lane, int blocks) {
  return reinterpret_cast<f32x4 *>(smem) + (wave & 3) * (blocks * 64) + lane;
}

// ------------------------------------------------------------------ backward: dq (and D)
template <int D, bool PAIRED, bool EXACT>
__device__ __forceinline__ void dq_block(unsigned place, char *smem, int b, int s, int n, int head_dim, int group, float scale,
                                         const bf16 *__restrict__ qkv, const bf16 *__restrict__ a, const float *__restrict__ lse,
                                         const bf16 *__restrict__ da, bf16 *__restrict__ dqkv, float *__restrict__ Dvec) {
  using T = Tile<D>;
  constexpr int KK = D / 32, DB = D / 16, STAGE = 2 * T::BYTES;
  constexpr int NB = PAIRED ? 4 : 2, NS = NB / 2;   // 16-row blocks and 32-row slots of a tile that a wave takes
  const HeadBlock hb(b, n, group, BackwardBlocks<PAIRED>::count(s), place);
  const int j = hb.head, bi = hb.batch;
  if (hb.none) return;
  // from the thread number: as in the forward kernel
  const BackwardBlocks<PAIRED> bb(s, PAIRED ? hb.order : row_blocks(s) - 1 - hb.order, threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, g = lane >> 4, lr = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // a scalar
  const int d = EXACT ? head_dim : D;
  const int64_t ld = (int64_t)n * 3 * d, pld = (int64_t)n * d;
  const bf16 *base = qkv + (int64_t)bi * s * ld + (int64_t)j * 3 * d;
  const int qw = bb.block * 64 + ((threadIdx.x >> 6) & 3) * 16;
  const int k_half = PAIRED ? 0 : (wave >> 2) * 32;   // first key of a tile that this wave takes
  const float f = EXACT ? scale : scale * kLog2e;
  typename T::Lane ln(lane);
  const uint32_t smem_addr = lds_address(smem);

  const int q = qw + lr, qc = q < s ? q : s - 1;
  bf16x8 qf[KK], dof[KK];
  float dsum = 0.0f;
  f32x4 diag = {0.0f, 0.0f, 0.0f, 0.0f};
  const bf16 *dah = da + (int64_t)bi * s * pld + (int64_t)j * d;
  {
    const bf16 *ar = a + ((int64_t)bi * s + qc) * pld + (int64_t)j * d;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const int col = 32 * kk + 8 * g;
      qf[kk] = row_chunk<EXACT>(base + (int64_t)qc * ld, col, d);
      dof[kk] = row_chunk<EXACT>(dah + (int64_t)qc * pld, col, d);
      const bf16x8 av = row_chunk<EXACT>(ar, col, d);
      if constexpr (EXACT) {   // D on the diagonal of a dO^T, by the same MFMAs as dP: where a row has one key (a = v) the two cancel exactly
        diag = MFMA16(av, dof[kk], diag);
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) dsum += (float)dof[kk][i] * (float)av[i];
      }
    }
    if constexpr (EXACT) {
      const float mine = (lr & 2) ? ((lr & 1) ? diag[3] : diag[2]) : ((lr & 1) ? diag[1] : diag[0]);
      dsum = __shfl(mine, 16 * (lr >> 2) + lr, 64);
    } else {
      dsum = quad_sum(dsum);
    }
  }
  float lsf = lse[((int64_t)bi * n + j) * s + qc];
  if constexpr (!EXACT) lsf *= kLog2e;
  if (q < s && g == 0 && (PAIRED ? !bb.idle : wave < 4)) Dvec[((int64_t)bi * n + j) * s + q] = EXACT ? dsum : -dsum;   // as the dk/dv kernel starts its accumulators, or subtracts it

  f32x4 dq[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int e = 0; e < 4; ++e) dq[db][e] = 0.0f;

  const int ntiles = bb.hi + 1;
  // tile DMAs as in the forward kernel
  constexpr int IPW = T::NI;   // DMA instructions per wave and tile
  const int quarter = wave & 3, half = wave >> 2;
  TileStream kv(base + d + half * d, ((int64_t)s * ld - (j * 3 + 1 + half) * d) * 2, 64 * ld * 2);
  uint32_t dma_off[IPW];
#pragma unroll
  for (int i = 0; i < IPW; ++i) dma_off[i] = T::dma_offset((uint32_t)(ld * 2), quarter, lane, i, d);
  auto issue_one = [&](auto tag, int st, int i) {   // instruction i of the stream's next tile into ring stage st
    constexpr int TAG = decltype(tag)::value;
    dma16<TAG>(kv.rsrc(), smem_addr + st * STAGE + half * T::BYTES + (quarter * IPW + i) * 1024, dma_off[i]);
  };
  constexpr int STEPS = NS * (KK + DB / 2);   // MFMA steps of a tile
  auto issue_step = [&](int step, int st) {
#pragma unroll
    for (int i = 0; i < IPW; ++i)
      if (i >= (step ? dma_by<IPW, STEPS>(step - 1) : 0) && i < dma_by<IPW, STEPS>(step)) issue_one(Spread{}, st, i);
  };
  auto issue = [&](int st) {
#pragma unroll
    for (int i = 0; i < IPW; ++i) issue_one(Burst{}, st, i);
  };
  issue(0);
  kv.advance();
  issue(1);
  kv.advance();
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    arrive(qf[kk]);
    arrive(dof[kk]);
  }
  arrive(lsf);
  arrive(dsum);
  int cur = 0;
  for (int it = 0; it < ntiles; ++it) {
    wait_and_barrier<IPW>();
    ln.here();
    const int nn = cur == 0 ? 2 : cur - 1;
    const char *Kt = smem + cur * STAGE + k_half * (T::ROWS16 / 16), *Vt = Kt + T::BYTES;
    const int kv0 = it * 64 + k_half;
    if (bb.idle || kv0 > qw + 15) {
      issue(nn);
    } else {
      f32x4 sc[NB], pc[NB];   // pc accumulates dP - D (EXACT: dP)
#pragma unroll
      for (int kb = 0; kb < NB; ++kb) {
        const float start = EXACT ? 0.0f : -dsum;
        pc[kb] = f32x4{start, start, start, start};
#pragma unroll
        for (int e = 0; e < 4; ++e) sc[kb][e] = 0.0f;
      }
      {  // step i: k-step i / NS, key blocks 2 (i % NS) and + 1
        constexpr int P = 2;   // steps that the reads run ahead
        bf16x8 kfr[P + 1][2], vfr[P + 1][2];
        pipelined<NS * KK, P>(
            [&](int i) {
#pragma unroll
              for (int h = 0; h < 2; ++h) {
                kfr[i % (P + 1)][h] = T::nat(Kt, ln, 2 * (i % NS) + h, i / NS);
                vfr[i % (P + 1)][h] = T::nat(Vt, ln, 2 * (i % NS) + h, i / NS);
              }
            },
            [&](int i) {
#pragma unroll
              for (int h = 0; h < 2; ++h) {
                const int kb = 2 * (i % NS) + h;
                sc[kb] = MFMA16(kfr[i % (P + 1)][h], qf[i / NS], sc[kb]);
                pc[kb] = MFMA16(vfr[i % (P + 1)][h], dof[i / NS], pc[kb]);
              }
            },
            [&](int i) { issue_step(i, nn); });
      }
      // dS^T = P^T o (dP^T - D); element (kb, e): key kv0 + 16 kb + 4 g + e, query qc
      constexpr int PT = 3, HB = DB / 2;
      bf16x8 ktr[PT + 1][2];
      auto load = [&](int i) {   // step i: key slot i / HB, output blocks 2 (i % HB) and + 1
#pragma unroll
        for (int h = 0; h < 2; ++h) ktr[i % (PT + 1)][h] = T::tr(Kt, ln, 2 * (i % HB) + h, i / HB);
      };
      pipelined_start<NS * HB, PT>(load);
      if (kv0 + 16 * NB - 1 > qw) {  // wave-uniform: diagonal (or past-the-end keys) among this wave's keys
#pragma unroll
        for (int kb = 0; kb < NB; ++kb)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (kv0 + 16 * kb + 4 * g + e > qc) sc[kb][e] = -INFINITY;
      }
#pragma unroll
      for (int kb = 0; kb < NB; ++kb)
#pragma unroll
        for (int e = 0; e < 4; ++e) sc[kb][e] = weight<EXACT>(sc[kb][e], f, lsf) * (EXACT ? pc[kb][e] - dsum : pc[kb][e]);
      Parts<EXACT ? 3 : 1> df[NS];
#pragma unroll
      for (int ks = 0; ks < NS; ++ks) df[ks] = weights<EXACT>(sc[2 * ks], sc[2 * ks + 1]);
      pipelined_run<NS * HB, PT>(
          load,
          [&](int i) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
              dq[2 * (i % HB) + h] = mma_weights(ktr[i % (PT + 1)][h], df[i / HB], dq[2 * (i % HB) + h]);
          },
          [&](int i) { issue_step(NS * KK + i, nn); });
    }
    kv.advance();
    cur = cur == 2 ? 0 : cur + 1;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  bf16 *out = dqkv + ((int64_t)bi * s + q) * ld + (int64_t)j * 3 * d;
  float z = 0.0f;   // EXACT: NaN where a result is not finite
  auto store = [&](int db, const f32x4 &sum) {
    if (EXACT && db * 16 + 4 * g >= d) return;
    bf16x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float x = (EXACT ? sum[e] * PARTS_UNSCALE : sum[e]) * scale;
      if constexpr (EXACT) z = fmaf(x, 0.0f, z);
      v[e] = (bf16)x;
    }
    *reinterpret_cast<bf16x4 *>(out + db * 16 + 4 * g) = v;
  };
  if constexpr (PAIRED) {
    if (q < s && !bb.idle) {
#pragma unroll
      for (int db = 0; db < DB; ++db) store(db, dq[db]);
    }
    return;
  }
  __syncthreads();   // the rings are no longer read
  f32x4 *slots = merge_slots(smem, wave, lane, DB);
  if (wave >= 4) {
#pragma unroll
    for (int db = 0; db < DB; ++db) slots[db * 64] = dq[db];
  }
  __syncthreads();
  if (wave < 4 && q < s) {
#pragma unroll
    for (int db = 0; db < DB; ++db) store(db, dq[db] + slots[db * 64]);
  }
  if constexpr (EXACT) {
    if (wave < 4 && !all_finite(z))
      redo_dq<bf16, D>(base, ld, dah, pld, s, d, scale, q, qw + 15 < s ? qw + 15 : s - 1, lse[((int64_t)bi * n + j) * s + qc], dsum, g, out);
  }
}

// ------------------------------------------------------------------ backward: dk, dv
// OWN_D: D is computed here (a: read then), not taken from the dq kernel.
template <int D, bool PAIRED, bool EXACT, bool OWN_D>
__device__ __forceinline__ void dkv_block(unsigned place, char *smem, int b, int s, int n, int head_dim, int group, float scale,
                                          const bf16 *__restrict__ qkv, const bf16 *__restrict__ a, const float *__restrict__ lse,
                                          const float *__restrict__ Dvec, const bf16 *__restrict__ da, bf16 *__restrict__ dqkv) {
  static_assert(!OWN_D || (!PAIRED && !EXACT), "as it is used");
  using T = Tile<D>;
  constexpr int KK = D / 32, DB = D / 16, STAGE = 2 * T::BYTES + 512;   // Q tile, dO tile, lse[64], D[64]
  constexpr int NB = PAIRED ? 4 : 2, NS = NB / 2;   // as in the dq kernel
  const HeadBlock hb(b, n, group, BackwardBlocks<PAIRED>::count(s), place);
  const int j = hb.head, bi = hb.batch;
  if (hb.none) return;
  const BackwardBlocks<PAIRED> bb(s, hb.order, threadIdx.x >> 6);   // (from the thread number: as in the forward kernels)
  const int lane = threadIdx.x & 63, g = lane >> 4, lr = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // a scalar
  const int d = EXACT ? head_dim : D;
  const int64_t ld = (int64_t)n * 3 * d, pld = (int64_t)n * d;
  const bf16 *base = qkv + (int64_t)bi * s * ld + (int64_t)j * 3 * d;
  const bf16 *dab = da + (int64_t)bi * s * pld + (int64_t)j * d;
  const int kw = bb.block * 64 + ((threadIdx.x >> 6) & 3) * 16;
  const int q_half = PAIRED ? 0 : (wave >> 2) * 32;   // first query of a tile that this wave takes
  const float f = EXACT ? scale : scale * kLog2e;
  typename T::Lane ln(lane);
  const uint32_t smem_addr = lds_address(smem);

  const int key = kw + lr, keyc = key < s ? key : s - 1;
  bf16x8 kf[KK], vf[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    kf[kk] = row_chunk<EXACT>(base + (int64_t)keyc * ld + d, 32 * kk + 8 * g, d);
    vf[kk] = row_chunk<EXACT>(base + (int64_t)keyc * ld + 2 * d, 32 * kk + 8 * g, d);
  }
  f32x4 dk[DB], dv[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int e = 0; e < 4; ++e) dk[db][e] = dv[db][e] = 0.0f;

  const int t_first = bb.lo, ntiles = row_blocks(s) - t_first;
  // tile DMAs as in the forward kernel (Q tile and dO tile), plus one instruction per wave for the
  // tile's lse values (even waves) or -D values (odd waves); those arrive four times over, so that every wave
  // issues the same number of memory operations, which the counted waits rely on
  constexpr int IPW = T::NI;
  const int quarter = wave & 3, half = wave >> 2;
  const int64_t pitch = half ? pld : ld, row0 = (int64_t)t_first * 64;
  TileStream qo(half ? dab + row0 * pld : base + row0 * ld, ((s - row0) * pitch - (half ? j : 3 * j) * d) * 2, 64 * pitch * 2);
  TileStream stats(((wave & 1) && !OWN_D ? Dvec : lse) + ((int64_t)bi * n + j) * s + row0, (s - row0) * 4, 256);
  uint32_t dma_off[IPW];
#pragma unroll
  for (int i = 0; i < IPW; ++i) dma_off[i] = T::dma_offset((uint32_t)(pitch * 2), quarter, lane, i, d);
  auto issue_one = [&](auto tag, int st, int i) {   // i == IPW: the statistics
    constexpr int TAG = decltype(tag)::value;
    const uint32_t stage = smem_addr + st * STAGE;
    if (i == IPW) {
      dma4<TAG>(stats.rsrc(), stage + 2 * T::BYTES + (wave & 1) * 256, lane * 4);
    } else {
      dma16<TAG>(qo.rsrc(), stage + half * T::BYTES + (quarter * IPW + i) * 1024, dma_off[i < IPW ? i : 0]);
    }
  };
  constexpr int STEPS = NS * (KK + DB);   // MFMA steps of a tile; the statistics count as instruction IPW
  auto issue_step = [&](int step, int st) {
#pragma unroll
    for (int i = 0; i <= IPW; ++i)
      if (i >= (step ? dma_by<IPW + 1, STEPS>(step - 1) : 0) && i < dma_by<IPW + 1, STEPS>(step)) issue_one(Spread{}, st, i);
  };
  auto advance = [&] {
    qo.advance();
    stats.advance();
  };
  auto issue = [&](int st) {
#pragma unroll
    for (int i = 0; i <= IPW; ++i) issue_one(Burst{}, st, i);
  };
  issue(0);
  advance();
  issue(1);
  advance();
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    arrive(kf[kk]);
    arrive(vf[kk]);
  }
  float *const own_d = reinterpret_cast<float *>(smem + 3 * STAGE);   // -D of the rows from the first tile on
  if constexpr (OWN_D) {
    const bf16 *ah = a + (int64_t)bi * s * pld + (int64_t)j * d;
    for (int row = (threadIdx.x >> 2); row < ntiles * 64; row += 128) {   // four lanes to a row
      const int64_t at = (int64_t)(row0 + row < s ? row0 + row : s - 1) * pld + (threadIdx.x & 3) * 8;
      float t = 0.0f;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        const bf16x8 x = *reinterpret_cast<const bf16x8 *>(dab + at + 32 * kk), y = *reinterpret_cast<const bf16x8 *>(ah + at + 32 * kk);
#pragma unroll
        for (int e = 0; e < 8; ++e) t += (float)x[e] * (float)y[e];
      }
      t += __shfl_xor(t, 1, 64);
      t += __shfl_xor(t, 2, 64);
      if ((threadIdx.x & 3) == 0) own_d[row] = -t;
    }
  }
  int cur = 0;
  for (int it = 0; it < ntiles; ++it) {
    wait_and_barrier<IPW + 1>();
    ln.here();
    const int nn = cur == 0 ? 2 : cur - 1;
    const char *Qt = smem + cur * STAGE + q_half * (T::ROWS16 / 16), *Ot = Qt + T::BYTES;
    const float *stat = reinterpret_cast<const float *>(smem + cur * STAGE + 2 * T::BYTES) + q_half;
    const int q0 = (t_first + it) * 64 + q_half;
    if (bb.idle || q0 + 16 * NB - 1 < kw) {  // wave-uniform: none of this wave's queries sees one of its keys
      issue(nn);
    } else {
      f32x4 sc[NB], pc[NB];   // pc accumulates dP - D (EXACT: dP)
#pragma unroll
      for (int qb = 0; qb < NB; ++qb) {
        if constexpr (EXACT) pc[qb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        else pc[qb] = *reinterpret_cast<const f32x4 *>((OWN_D ? own_d + it * 64 + q_half : stat + 64) + 16 * qb + 4 * g);
#pragma unroll
        for (int e = 0; e < 4; ++e) sc[qb][e] = 0.0f;
      }
      {  // step i: k-step i / NS, query blocks 2 (i % NS) and + 1
        constexpr int P = 2;
        bf16x8 qfr[P + 1][2], ofr[P + 1][2];
        pipelined<NS * KK, P>(
            [&](int i) {
#pragma unroll
              for (int h = 0; h < 2; ++h) {
                qfr[i % (P + 1)][h] = T::nat(Qt, ln, 2 * (i % NS) + h, i / NS);
                ofr[i % (P + 1)][h] = T::nat(Ot, ln, 2 * (i % NS) + h, i / NS);
              }
            },
            [&](int i) {
#pragma unroll
              for (int h = 0; h < 2; ++h) {
                const int qb = 2 * (i % NS) + h;
                sc[qb] = MFMA16(qfr[i % (P + 1)][h], kf[i / NS], sc[qb]);
                pc[qb] = MFMA16(ofr[i % (P + 1)][h], vf[i / NS], pc[qb]);
              }
            },
            [&](int i) { issue_step(i, nn); });
      }
      // element (qb, e): query q0 + 16 qb + 4 g + e, key `key`
      constexpr int PT = 3;
      bf16x8 otr[PT + 1], qtr[PT + 1];
      auto load = [&](int i) {   // step i: query slot i / DB, output block i % DB
        otr[i % (PT + 1)] = T::tr(Ot, ln, i % DB, i / DB);
        qtr[i % (PT + 1)] = T::tr(Qt, ln, i % DB, i / DB);
      };
      pipelined_start<NS * DB, PT>(load);
      if (q0 < kw + 16 || q0 + 16 * NB - 1 >= s) {  // wave-uniform: diagonal or past-the-end queries
#pragma unroll
        for (int qb = 0; qb < NB; ++qb)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int qq = q0 + 16 * qb + 4 * g + e;
            if (qq < key || qq >= s) sc[qb][e] = -INFINITY;
          }
      }
#pragma unroll
      for (int qb = 0; qb < NB; ++qb) {
        if constexpr (EXACT) pc[qb] -= *reinterpret_cast<const f32x4 *>(stat + 64 + 16 * qb + 4 * g);
        const f32x4 ls = *reinterpret_cast<const f32x4 *>(stat + 16 * qb + 4 * g);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          sc[qb][e] = weight<EXACT>(sc[qb][e], f, EXACT ? ls[e] : ls[e] * kLog2e);
          pc[qb][e] *= sc[qb][e];
        }
      }
      Parts<EXACT ? 3 : 1> pf[NS], df[NS];
#pragma unroll
      for (int ks = 0; ks < NS; ++ks) {
        pf[ks] = weights<EXACT>(sc[2 * ks], sc[2 * ks + 1]);
        df[ks] = weights<EXACT>(pc[2 * ks], pc[2 * ks + 1]);
      }
      pipelined_run<NS * DB, PT>(
          load,
          [&](int i) {
            dv[i % DB] = mma_weights(otr[i % (PT + 1)], pf[i / DB], dv[i % DB]);
            dk[i % DB] = mma_weights(qtr[i % (PT + 1)], df[i / DB], dk[i % DB]);
          },
          [&](int i) { issue_step(NS * KK + i, nn); });
    }
    advance();
    cur = cur == 2 ? 0 : cur + 1;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  bf16 *out = dqkv + ((int64_t)bi * s + key) * ld + (int64_t)j * 3 * d;
  float z = 0.0f;   // EXACT: NaN where a result is not finite
  auto store = [&](int db, const f32x4 &sk, const f32x4 &sv) {
    if (EXACT && db * 16 + 4 * g >= d) return;
    bf16x4 ok, ov;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float x = (EXACT ? sk[e] * PARTS_UNSCALE : sk[e]) * scale, y = EXACT ? sv[e] * PARTS_UNSCALE : sv[e];
      if constexpr (EXACT) z = fmaf(x, 0.0f, fmaf(y, 0.0f, z));
      ok[e] = (bf16)x;
      ov[e] = (bf16)y;
    }
    *reinterpret_cast<bf16x4 *>(out + d + db * 16 + 4 * g) = ok;
    *reinterpret_cast<bf16x4 *>(out + 2 * d + db * 16 + 4 * g) = ov;
  };
  if constexpr (PAIRED) {
    if (key < s && !bb.idle) {
#pragma unroll
      for (int db = 0; db < DB; ++db) store(db, dk[db], dv[db]);
    }
    return;
  }
  __syncthreads();   // the rings are no longer read
  f32x4 *slots = merge_slots(smem, wave, lane, 2 * DB);
  if (wave >= 4) {
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      slots[db * 64] = dk[db];
      slots[(DB + db) * 64] = dv[db];
    }
  }
  __syncthreads();
  if (wave < 4 && key < s) {
#pragma unroll
    for (int db = 0; db < DB; ++db) store(db, dk[db] + slots[db * 64], dv[db] + slots[(DB + db) * 64]);
  }
  if constexpr (EXACT) {
    if (wave < 4 && !all_finite(z)) {
      const int64_t st = ((int64_t)bi * n + j) * s;
      redo_dk<bf16, D>(base, ld, dab, pld, s, d, scale, kw, key, lse + st, [&](int t) { return Dvec[st + t]; }, g, out);
      redo_dv<bf16, D>(base, ld, dab, pld, s, d, scale, kw, key, lse + st, g, out);
    }
  }
}

template <int D, bool PAIRED, bool EXACT>
__global__ __launch_bounds__(512) void attn_bwd64_dq_kernel(BackwardArgs w) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  dq_block<D, PAIRED, EXACT>(blockIdx.x, smem, w.b, w.s, w.n, w.head_dim, w.group, w.scale, w.qkv, w.a, w.lse, w.da, w.dqkv, w.Dvec);
}
template <int D, bool PAIRED, bool EXACT>
__global__ __launch_bounds__(512) void attn_bwd64_dkv_kernel(BackwardArgs w) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  dkv_block<D, PAIRED, EXACT, false>(blockIdx.x, smem, w.b, w.s, w.n, w.head_dim, w.group, w.scale, w.qkv, w.a, w.lse, w.Dvec, w.da, w.dqkv);
}
// Both in one launch (attention_bwd64 says when): the first half of a grid row's workgroups (dk / dv, the longer ones) compute D for themselves.
__global__ __launch_bounds__(512) void attn_bwd64_kernel(BackwardArgs w) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const unsigned half = gridDim.x / 2;
  if (blockIdx.x < half)
    dkv_block<64, false, false, true>(blockIdx.x, smem, w.b, w.s, w.n, w.head_dim, w.group, w.scale, w.qkv, w.a, w.lse, nullptr, w.da, w.dqkv);
  else
    dq_block<64, false, false>(blockIdx.x - half, smem, w.b, w.s, w.n, w.head_dim, w.group, w.scale, w.qkv, w.a, w.lse, w.da, w.dqkv, w.Dvec);
}

template <int D, bool PAIRED, bool EXACT>
int launch_two(const BackwardArgs &in, hipStream_t st) {
  constexpr int smem_dq = 3 * 2 * Tile<D>::BYTES, smem_dkv = smem_dq + 3 * 512;
  static_assert(smem_dkv >= 4 * 2 * (D / 16) * 1024, "the merge of the two halves fits the rings");
  static unsigned long long attr_done = 0;
  int device;
  if (!attr_is_set(attr_done, &device)) {
    MTNLG_TRY(set_lds(attn_bwd64_dq_kernel<D, PAIRED, EXACT>, smem_dq));
    MTNLG_TRY(set_lds(attn_bwd64_dkv_kernel<D, PAIRED, EXACT>, smem_dkv));
    attr_mark_set(attr_done, device);
  }
  BackwardArgs w = in;
  const int count = BackwardBlocks<PAIRED>::count(w.s);
  w.group = HeadBlock::group(w.b, w.n, count, PAIRED || D >= 128 ? 32 : 128, PAIRED ? 511 : 2047);
  const dim3 grid = HeadBlock::grid(w.b, w.n, w.group, count);
  LaunchScope scope(MTNLG_K_ATTN_BWD, st);
  attn_bwd64_dq_kernel<D, PAIRED, EXACT><<<grid, 512, smem_dq, st>>>(w);
  MTNLG_TRY(check_launch());
  attn_bwd64_dkv_kernel<D, PAIRED, EXACT><<<grid, 512, smem_dkv, st>>>(w);
  return check_launch();
}

constexpr int ONE_LAUNCH_ROWS = 4096;   // what their D has room for in LDS
int launch_one(const BackwardArgs &in, hipStream_t st) {
  BackwardArgs w = in;
  const int count = row_blocks(w.s);
  w.group = HeadBlock::group(w.b, w.n, count, 32, 2047);
  constexpr int rings = 3 * (2 * Tile<64>::BYTES + 512);
  static unsigned long long attr_done = 0;
  int device;
  if (!attr_is_set(attr_done, &device)) {
    MTNLG_TRY(set_lds(attn_bwd64_kernel, rings + ONE_LAUNCH_ROWS * (int)sizeof(float)));
    attr_mark_set(attr_done, device);
  }
  dim3 grid = HeadBlock::grid(w.b, w.n, w.group, count);
  grid.x *= 2;
  LaunchScope scope(MTNLG_K_ATTN_BWD, st);
  attn_bwd64_kernel<<<grid, 512, rings + count * 64 * (int)sizeof(float), st>>>(w);
  return check_launch();
}

}  // namespace

// Two blocks of a head in each workgroup: only for sequences of two blocks, of which those that come here have more than 384 heads (512 heads, s = 80 26.0 us by
// halves, 23.3 paired; but 300, s = 192 31.2, 36.7).
// One launch where all workgroups of either kernel run at once, so that both kernels' would leave units idle one after the other: a second
// D for every tile costs less than that and the launch.  us, two launches / one: 2 x 257 tokens 13.3 / 8.7; by blocks of all heads together (s 192 to 1024): 512 1.16 to
// 1.19 times as fast, 768 1.11, 1024 0.96 (two blocks of 70 to 128 rows: 256 1.22 to 1.35, 384 0.92 to 1.10, 512 0.92 to 1.01, 768 1.13 to 1.20).  Beyond s 960 D takes the LDS of
// the third workgroup: up to 256 blocks 1.19 to 1.44 times as fast from s 1030 to 4096, 384 1.11 to 1.33, 512 0.92 to 1.17, 768 0.94 to 1.06.
int attention_bwd64(int b, int s, int n, float scale, const void *qkv, const void *a, const float *lse, const void *da, void *dqkv, void *ws, hipStream_t st) {
  const BackwardArgs w{b, s, n, 64, 0, scale, (const bf16 *)qkv, (const bf16 *)a, lse, (const bf16 *)da, (bf16 *)dqkv, (float *)ws};
  if (s <= ONE_LAUNCH_ROWS && (int64_t)b * n * row_blocks(s) <= (s > 1024 ? 256 : 768)) return launch_one(w, st);
  return row_blocks(s) == 2 ? launch_two<64, true, false>(w, st) : launch_two<64, false, false>(w, st);
}

int attention_bwd_exact64(int b, int s, int n, int d, float scale, const void *qkv, const void *a, const float *lse, const void *da, void *dqkv, void *ws,
                          hipStream_t st) {
  const BackwardArgs w{b, s, n, d, 0, scale, (const bf16 *)qkv, (const bf16 *)a, lse, (const bf16 *)da, (bf16 *)dqkv, (float *)ws};
  switch ((d + 31) / 32) {
    case 1: return launch_two<32, false, true>(w, st);
    case 2: return launch_two<64, false, true>(w, st);
    case 3: return launch_two<96, false, true>(w, st);
    case 4: return launch_two<128, false, true>(w, st);
    case 5: return launch_two<160, false, true>(w, st);
    case 6: return launch_two<192, false, true>(w, st);
    default: return MTNLG_UNSUPPORTED_SHAPE;
  }
}

}  // namespace mtnlg
