// Fused causal softmax attention on the gfx950 matrix cores, forward: the calls where rows of 16 to a wave beat those of attention_mfma.hip (which says what is computed, and
// how, and which calls these are): with P in fp32 (EXACT) some head sizes, short sequences and a few others, else short sequences.
//
// Eight waves.  A workgroup owns 128 queries, 16 per wave, held in registers as MFMA B operands; K and V stream through LDS in tiles of 64 rows, brought in by LDS DMA three
// tiles deep, one workgroup barrier per tile.  What bounds it: no single unit.  Between two barriers a wave runs LDS reads, MFMAs, the softmax and the
// DMA issue in one chain, and the waves of a workgroup run it in step, so the times of the four add up.  All products are v_mfma_f32_16x16x32_bf16 with the
// streamed tile as the A operand, so a product block comes out as C[tile row 4 (lane/16) + i][own row lane%16], i = 0..3; the k slots of the
// second product are ordered to match (slot (g, e) of a 32-row step = tile row 4g + e for e < 4, 16 + 4g + e - 4 otherwise).
#include "attention_tiles.h"

namespace mtnlg {

namespace {

// Which rows a wave of the forward kernel owns.
// Under the causal mask a 64-row block b works on b + 1 of the 64-row tiles the workgroup streams, so blocks taken in order
// would leave the workgroups of a head with 1 .. s/64 tiles of work.  The two halves of a workgroup therefore take
// blocks p and nb - 1 - p (nb blocks of 64 rows in the sequence): every workgroup then computes nb + 1 wave-halves
// of tiles, and while only one half has work in a tile it has the compute unit to itself.  With an
// odd nb the middle block is alone in its workgroup and the other half only helps to move tiles.
struct PairedBlocks {
  int row0;        // first row of this wave
  int last_tile;   // highest 64-row block of the workgroup: it streams tiles 0 .. last
  bool idle;       // wave-uniform: this wave owns no rows
  __device__ PairedBlocks(int s, int pair, int wave) {
    const int lo = pair, hi = row_blocks(s) - 1 - pair, half = wave >> 2;
    row0 = (half ? hi : lo) * 64 + (wave & 3) * 16;
    last_tile = hi;
    idle = half && hi == lo;
  }
  static __host__ __device__ int count(int s) { return (row_blocks(s) + 1) / 2; }
};

template <int D, bool EXACT>
__global__ __launch_bounds__(512) void attn_fwd16_kernel(int b, int s, int n, int head_dim, int group, float scale, const bf16 *__restrict__ qkv,
                                                        bf16 *__restrict__ a, float *__restrict__ lse) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  using T = Tile<D>;
  constexpr int KK = D / 32, DB = D / 16, STAGE = 2 * T::BYTES;
  const HeadBlock hb(b, n, group, PairedBlocks::count(s), blockIdx.x);
  const int j = hb.head, bi = hb.batch;
  if (hb.none) return;
  const int lane = threadIdx.x & 63, g = lane >> 4, lr = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // a scalar
  const int d = EXACT ? head_dim : D;
  const int64_t ld = (int64_t)n * 3 * d;
  const bf16 *base = qkv + (int64_t)bi * s * ld + (int64_t)j * 3 * d;
  // From the thread number and not the scalar: with a scalar condition for masked tiles the compiler lays the tile's code out per path and holds more registers.
  const PairedBlocks rb(s, hb.order, threadIdx.x >> 6);
  const int qw = rb.row0;
  const float c = scale * kLog2e, f = EXACT ? scale : c;
  typename T::Lane ln(lane);
  const uint32_t smem_addr = lds_address(smem);

  bf16x8 qf[KK];
  const int q = qw + lr, qc = q < s ? q : s - 1;
#pragma unroll
  for (int kk = 0; kk < KK; ++kk)
    qf[kk] = row_chunk<EXACT>(base + (int64_t)qc * ld, 32 * kk + 8 * g, d);
  f32x4 o[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int e = 0; e < 4; ++e) o[db][e] = 0.0f;
  float m = -INFINITY, l = 0.0f;   // l: this lane's share of the row sum

  const int ntiles = rb.last_tile + 1;
  // Waves 0-3 bring the K tile, waves 4-7 the V tile, 16 rows each.  The DMAs of tile it + 2 are spread over
  // the MFMA steps of tile it (dma_by).
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
  constexpr int STEPS = 2 * KK + DB;   // MFMA steps of a tile
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
  for (int kk = 0; kk < KK; ++kk) arrive(qf[kk]);
  int cur = 0;
  for (int it = 0; it < ntiles; ++it) {
    wait_and_barrier<IPW>();   // tile it landed everywhere, tile it-1 no longer read
    ln.here();
    const int nn = cur == 0 ? 2 : cur - 1;   // stage of tile it + 2
    const char *Kt = smem + cur * STAGE, *Vt = Kt + T::BYTES;
    const int kv0 = it * 64;
    if (rb.idle || kv0 > qw + 15) {  // wave-uniform: every (query, key) pair of this wave is masked
      issue(nn);
    } else {
      f32x4 sc[4];
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int e = 0; e < 4; ++e) sc[kb][e] = 0.0f;
      {  // step i: k-step i / 2, key blocks 2 (i % 2) and 2 (i % 2) + 1
        bf16x8 kfr[4][2];
        pipelined<2 * KK, 3>(
            [&](int i) {
#pragma unroll
              for (int h = 0; h < 2; ++h) kfr[i & 3][h] = T::nat(Kt, ln, 2 * (i & 1) + h, i >> 1);
            },
            [&](int i) {
#pragma unroll
              for (int h = 0; h < 2; ++h)
                sc[2 * (i & 1) + h] = MFMA16(kfr[i & 3][h], qf[i >> 1], sc[2 * (i & 1) + h]);
            },
            [&](int i) { issue_step(i, nn); });
      }
      // element (kb, e): key kv0 + 16 kb + 4 g + e, query qc
      if (kv0 + 63 > qw) {  // wave-uniform: this tile crosses the diagonal for some row
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (kv0 + 16 * kb + 4 * g + e > qc) sc[kb][e] = -INFINITY;
      }
      // m tracks the running maximum of the raw scores; exponents are taken in base 2 with the
      // scale folded in: p = 2^(s c - m c).
      float mx = -INFINITY;
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int e = 0; e < 4; ++e) mx = fmaxf(mx, sc[kb][e]);
      mx = quad_max(mx);
      // The reference maximum only follows when the row maximum has outgrown it by more than
      // 2^8 in the exponent's units (any reference gives the same sums; this one keeps p <= 256
      // and makes rescaling O rare).  Finite from the first tile on: key 0 is never masked.
      const float m_new = mx * c > m * c + 8.0f ? mx : m;
      const float mc = EXACT ? product_of(m_new, scale) : m_new * c;
      float rs = 0.0f;
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float p = weight<EXACT>(sc[kb][e], f, mc);
          sc[kb][e] = p;
          rs += p;
        }
      const float alpha = EXACT ? exact_exp((m - m_new) * scale) : fast_exp2((m - m_new) * c);
      l = l * alpha + rs;
      m = m_new;
      if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {  // a reference maximum moved: rescale O
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int e = 0; e < 4; ++e) o[db][e] *= alpha;
      }
      {  // step i: key half i / (DB / 2), output blocks 2 (i % (DB / 2)) and + 1
        Parts<EXACT ? 3 : 1> pf[2];
        bf16x8 vfr[4][2];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) pf[ks] = weights<EXACT>(sc[2 * ks], sc[2 * ks + 1]);
        constexpr int HB = DB / 2;
        pipelined<2 * HB, 3>(
            [&](int i) {
#pragma unroll
              for (int h = 0; h < 2; ++h) vfr[i & 3][h] = T::tr(Vt, ln, 2 * (i % HB) + h, i / HB);
            },
            [&](int i) {
#pragma unroll
              for (int h = 0; h < 2; ++h)
                o[2 * (i % HB) + h] = mma_weights(vfr[i & 3][h], pf[i / HB], o[2 * (i % HB) + h]);
            },
            [&](int i) { issue_step(2 * KK + i, nn); });
      }
    }
    kv.advance();
    cur = cur == 2 ? 0 : cur + 1;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the look-ahead tiles, which nobody reads

  const float lsum = quad_sum(l);
  bf16 *out = a + ((int64_t)bi * s + q) * ((int64_t)n * d) + (int64_t)j * d;
  float *out_lse = lse + ((int64_t)bi * n + j) * s + q;
  float z = 0.0f;   // EXACT: NaN where a result is not finite
  if (q < s && !rb.idle) {
    const float inv = EXACT ? 1.0f / lsum * PARTS_UNSCALE : 1.0f / lsum;
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      if (EXACT && db * 16 + 4 * g >= d) continue;
      bf16x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float x = o[db][e] * inv;
        if constexpr (EXACT) z = fmaf(x, 0.0f, z);
        v[e] = (bf16)x;
      }
      *reinterpret_cast<bf16x4 *>(out + db * 16 + 4 * g) = v;
    }
    if (g == 0) *out_lse = EXACT ? plus_log(product_of(m, scale), lsum) : (m * c + log2f(lsum)) * kLn2;
  }
  if constexpr (EXACT) {
    if (!all_finite(z)) redo_fwd<bf16, D>(base, ld, s, d, scale, q, qw + 15 < s ? qw + 15 : s - 1, g, out, out_lse);
  }
}

template <int D, bool EXACT>
int fwd16_launch(int b, int s, int n, int d, float scale, const void *qkv, void *a, float *lse, hipStream_t st) {
  constexpr int smem = 3 * 2 * Tile<D>::BYTES;
  static unsigned long long attr_done = 0;
  int device;
  if (!attr_is_set(attr_done, &device)) {
    MTNLG_TRY(set_lds(attn_fwd16_kernel<D, EXACT>, smem));
    attr_mark_set(attr_done, device);
  }
  const int count = PairedBlocks::count(s), group = HeadBlock::group(b, n, count, 32, D >= 128 ? 511 : 768);   // (768: 3 a compute unit)
  LaunchScope scope(MTNLG_K_ATTN_FWD, st);
  attn_fwd16_kernel<D, EXACT><<<HeadBlock::grid(b, n, group, count), 512, smem, st>>>(b, s, n, d, group, scale, (const bf16 *)qkv, (bf16 *)a, lse);
  return check_launch();
}

}  // namespace

int attention_fwd_mfma16(int b, int s, int n, int d, float scale, const void *qkv, void *a, float *lse, hipStream_t stream) {
  switch (d) {
    case 64: return fwd16_launch<64, false>(b, s, n, d, scale, qkv, a, lse, stream);
    case 128: return fwd16_launch<128, false>(b, s, n, d, scale, qkv, a, lse, stream);
    case 160: return fwd16_launch<160, false>(b, s, n, d, scale, qkv, a, lse, stream);
    default: return MTNLG_UNSUPPORTED_SHAPE;
  }
}

int attention_fwd_exact16(int b, int s, int n, int d, float scale, const void *qkv, void *a, float *lse, hipStream_t stream) {
  switch ((d + 31) / 32) {
    case 1: return fwd16_launch<32, true>(b, s, n, d, scale, qkv, a, lse, stream);
    case 2: return fwd16_launch<64, true>(b, s, n, d, scale, qkv, a, lse, stream);
    case 3: return fwd16_launch<96, true>(b, s, n, d, scale, qkv, a, lse, stream);
    case 4: return fwd16_launch<128, true>(b, s, n, d, scale, qkv, a, lse, stream);
    case 5: return fwd16_launch<160, true>(b, s, n, d, scale, qkv, a, lse, stream);
    case 6: return fwd16_launch<192, true>(b, s, n, d, scale, qkv, a, lse, stream);
    default: return MTNLG_UNSUPPORTED_SHAPE;
  }
}

}  // namespace mtnlg
