// Fused causal softmax attention on the gfx950 matrix cores (bf16 in, fp32 softmax and accumulation): forward, for head sizes 64, 128 and 160; and
// with P in fp32 (EXACT) for the others up to 192.  Backward: attention_bwd.hip, attention_bwd64.hip.
//
//   S = scale * q k^T (causal),  P = rowsoftmax(S),  a = P v,  lse = log sum exp(S)
//
// Eight waves.  A workgroup owns 128 or 256 queries, 16 or 32 per wave, held in registers as MFMA B operands (groups of 16, one row per lane
// column); K and V stream through LDS in tiles of 64 rows, brought in by LDS DMA (buffer_load ... lds, no staging
// registers) three tiles deep, one workgroup barrier per tile.  What bounds it: no single unit.  Between two barriers a
// wave runs LDS reads, MFMAs, the softmax and the DMA issue in one chain, and the waves of a workgroup run it in step, so
// the times of the four add up; taking any one out shortened a tile by no more than that one's own time.
//
// All products are v_mfma_f32_16x16x32_bf16 with the streamed tile as the A operand, so a product block comes out as
// C[tile row 4 (lane/16) + i][own row lane%16], i = 0..3: S^T = K Q^T; the softmax statistics of a query live in the four lanes that
// share lane%16; P^T packed to bf16 is directly the B operand of O^T += V^T P^T.  That product contracts over the tile's rows.  Its A operand is read
// from the same natural [row][D] tile with the transposing LDS read (ds_read_b64_tr_b16: a
// 16-lane group reads 4 tile rows x 16 columns, each lane receives the 4 row values of its
// column); the k slots of that MFMA are ordered to match the accumulator layout of the
// first product (slot (g, e) of a 32-row step = tile row 4g + e for e < 4, 16 + 4g + e - 4
// otherwise), so P never leaves the registers and nothing is transposed in software.
// No atomics: every output element has one owner, results are run-to-run identical.
//
// EXACT: any head size d that is a multiple of 8, in tiles of D = d rounded up to 32 columns (the DMA brings zeros past d).  P is
// not rounded to bf16: it goes into the second product as three bf16 parts that add up to it (common.h: Parts; scaled, so of any size), three MFMAs
// where the other kernels have one.  2 x 1024 tokens, 16 heads of 96: 103 us on the fp32 instructions without LDS (attention_f32.hip), 24 here.  Inputs that are
// not finite take the slow path of attention_redo.h.
#include "attention_tiles.h"

namespace mtnlg {

namespace {

// Which rows a wave of the forward kernel owns.
// Under the causal mask a 64-row block b works on b + 1 of the 64-row tiles the workgroup streams, so blocks taken in order
// would leave the workgroups of a head with 1 .. s/64 tiles of work.  The two halves of a workgroup therefore take
// blocks p and nb - 1 - p (nb blocks of 64 G rows in the sequence): every workgroup then computes nb + 1 wave-halves
// of tiles, and while only one half has work in a tile it has the compute unit to itself.  With an
// odd nb the middle block is alone in its workgroup and the other half only helps to move tiles.
template <int G>
struct PairedBlocks {
  int row0;        // first row of this wave
  int last_tile;   // highest 64-row block of the workgroup: it streams tiles 0 .. last
  bool idle;       // wave-uniform: this wave owns no rows
  __device__ PairedBlocks(int s, int pair, int wave) {
    const int nb = (s + 63) / 64, nblk = (nb + G - 1) / G;
    const int lo = pair, hi = nblk - 1 - pair, half = wave >> 2;
    row0 = (half ? hi : lo) * (64 * G) + (wave & 3) * (16 * G);
    last_tile = hi * G + G - 1 < nb ? hi * G + G - 1 : nb - 1;
    idle = half && hi == lo;
  }
  static __host__ __device__ int count(int s) { return (((s + 63) / 64 + G - 1) / G + 1) / 2; }
};

// ------------------------------------------------------------------ forward
template <int D, int G, bool EXACT>
__global__ __launch_bounds__(512) void attn_fwd_kernel(int b, int s, int n, int head_dim, int group, float scale, const bf16 *__restrict__ qkv,
                                                      bf16 *__restrict__ a, float *__restrict__ lse) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  using T = Tile<D>;
  constexpr int KK = D / 32, DB = D / 16, STAGE = 2 * T::BYTES;
  const HeadBlock hb(b, n, group, PairedBlocks<G>::count(s), blockIdx.x);
  const int j = hb.head, bi = hb.batch;
  if (hb.none) return;
  const int lane = threadIdx.x & 63, g = lane >> 4, lr = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // a scalar
  const int d = EXACT ? head_dim : D;
  const int64_t ld = (int64_t)n * 3 * d;
  const bf16 *base = qkv + (int64_t)bi * s * ld + (int64_t)j * 3 * d;
  // From the thread number and not the scalar: with a scalar condition for masked tiles the compiler lays the tile's code
  // out per path and holds 60 registers more (head size 160, 32 rows per wave: 256 and 27 spilled, 163 us; now 208, 105).
  const PairedBlocks<G> rb(s, hb.order, threadIdx.x >> 6);
  const int qw = rb.row0;
  const float c = scale * kLog2e, f = EXACT ? scale : c;
  typename T::Lane ln(lane);
  const uint32_t smem_addr = lds_address(smem);

  int qc[G];
  bf16x8 qf[G][KK];
#pragma unroll
  for (int qg = 0; qg < G; ++qg) {
    const int q = qw + 16 * qg + lr;
    qc[qg] = q < s ? q : s - 1;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
      qf[qg][kk] = row_chunk<EXACT>(base + (int64_t)qc[qg] * ld, 32 * kk + 8 * g, d);
  }
  f32x4 o[G][DB];
#pragma unroll
  for (int qg = 0; qg < G; ++qg)
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int e = 0; e < 4; ++e) o[qg][db][e] = 0.0f;
  float m[G], l[G];   // l: this lane's share of the row sum
#pragma unroll
  for (int qg = 0; qg < G; ++qg) {
    m[qg] = -INFINITY;
    l[qg] = 0.0f;
  }

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
  for (int qg = 0; qg < G; ++qg)
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) arrive(qf[qg][kk]);
  int cur = 0;
  for (int it = 0; it < ntiles; ++it) {
    wait_and_barrier<IPW>();   // tile it landed everywhere, tile it-1 no longer read
    ln.here();
    const int nn = cur == 0 ? 2 : cur - 1;   // stage of tile it + 2
    const char *Kt = smem + cur * STAGE, *Vt = Kt + T::BYTES;
    const int kv0 = it * 64;
    if (rb.idle || kv0 > qw + (16 * G - 1)) {  // wave-uniform: every (query, key) pair of this wave is masked
      issue(nn);
    } else {
      f32x4 sc[G][4];
#pragma unroll
      for (int qg = 0; qg < G; ++qg)
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
          for (int e = 0; e < 4; ++e) sc[qg][kb][e] = 0.0f;
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
#pragma unroll
                for (int qg = 0; qg < G; ++qg)
                  sc[qg][2 * (i & 1) + h] = MFMA16(kfr[i & 3][h], qf[qg][i >> 1], sc[qg][2 * (i & 1) + h]);
            },
            [&](int i) { issue_step(i, nn); });
      }
      // element (qg, kb, e): key kv0 + 16 kb + 4 g + e, query qc[qg]
      if (kv0 + 63 > qw) {  // wave-uniform: this tile crosses the diagonal for some row
#pragma unroll
        for (int qg = 0; qg < G; ++qg)
#pragma unroll
          for (int kb = 0; kb < 4; ++kb)
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (kv0 + 16 * kb + 4 * g + e > qc[qg]) sc[qg][kb][e] = -INFINITY;
      }
      // m tracks the running maximum of the raw scores; exponents are taken in base 2 with the
      // scale folded in: p = 2^(s c - m c).
      float alpha[G];
#pragma unroll
      for (int qg = 0; qg < G; ++qg) {
        float mx = -INFINITY;
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
          for (int e = 0; e < 4; ++e) mx = fmaxf(mx, sc[qg][kb][e]);
        mx = quad_max(mx);
        // The reference maximum only follows when the row maximum has outgrown it by more than
        // 2^8 in the exponent's units (any reference gives the same sums; this one keeps p <= 256
        // and makes rescaling O rare).  Finite from the first tile on: key 0 is never masked.
        const float m_new = mx * c > m[qg] * c + 8.0f ? mx : m[qg];
        const float mc = EXACT ? product_of(m_new, scale) : m_new * c;
        float rs = 0.0f;
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float p = weight<EXACT>(sc[qg][kb][e], f, mc);
            sc[qg][kb][e] = p;
            rs += p;
          }
        alpha[qg] = EXACT ? exact_exp((m[qg] - m_new) * scale) : fast_exp2((m[qg] - m_new) * c);
        l[qg] = l[qg] * alpha[qg] + rs;
        m[qg] = m_new;
      }
      bool moved = false;
#pragma unroll
      for (int qg = 0; qg < G; ++qg) moved = moved || alpha[qg] != 1.0f;
      if (__builtin_amdgcn_ballot_w64(moved) != 0) {  // a reference maximum moved: rescale O
#pragma unroll
        for (int qg = 0; qg < G; ++qg)
#pragma unroll
          for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int e = 0; e < 4; ++e) o[qg][db][e] *= alpha[qg];
      }
      {  // step i: key half i / (DB / 2), output blocks 2 (i % (DB / 2)) and + 1
        Parts<EXACT ? 3 : 1> pf[2][G];
        bf16x8 vfr[4][2];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
          for (int qg = 0; qg < G; ++qg) pf[ks][qg] = weights<EXACT>(sc[qg][2 * ks], sc[qg][2 * ks + 1]);
        constexpr int HB = DB / 2;
        pipelined<2 * HB, 3>(
            [&](int i) {
#pragma unroll
              for (int h = 0; h < 2; ++h) vfr[i & 3][h] = T::tr(Vt, ln, 2 * (i % HB) + h, i / HB);
            },
            [&](int i) {
#pragma unroll
              for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int qg = 0; qg < G; ++qg)
                  o[qg][2 * (i % HB) + h] = mma_weights(vfr[i & 3][h], pf[i / HB][qg], o[qg][2 * (i % HB) + h]);
            },
            [&](int i) { issue_step(2 * KK + i, nn); });
      }
    }
    kv.advance();
    cur = cur == 2 ? 0 : cur + 1;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the look-ahead tiles, which nobody reads

#pragma unroll
  for (int qg = 0; qg < G; ++qg) {
    const int q = qw + 16 * qg + lr;
    const float lsum = quad_sum(l[qg]);
    bf16 *out = a + ((int64_t)bi * s + q) * ((int64_t)n * d) + (int64_t)j * d;
    float *out_lse = lse + ((int64_t)bi * n + j) * s + q;
    float z = 0.0f;   // EXACT: NaN where a result is not finite
    if (q < s && !rb.idle) {
      const float inv = 1.0f / lsum;
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        if (EXACT && db * 16 + 4 * g >= d) continue;
        bf16x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float x = o[qg][db][e] * (EXACT ? inv * PARTS_UNSCALE : inv);
          if constexpr (EXACT) z = fmaf(x, 0.0f, z);
          v[e] = (bf16)x;
        }
        *reinterpret_cast<bf16x4 *>(out + db * 16 + 4 * g) = v;
      }
      if (g == 0) *out_lse = EXACT ? plus_log(product_of(m[qg], scale), lsum) : (m[qg] * c + log2f(lsum)) * kLn2;
    }
    if constexpr (EXACT) {
      const int first = qw + 16 * qg, last = first + 15 < s ? first + 15 : s - 1;
      if (!all_finite(z)) redo_fwd<bf16, D>(base, ld, s, d, scale, q, last, g, out, out_lse);
    }
  }
}

// Forward with 32 rows per wave on eight waves (256 rows per workgroup): every K / V fragment read from LDS feeds two
// MFMAs, which halves the kernel's LDS traffic -- its bound: each of the eight waves reads the whole K and V tile, the
// V tile through half-rate transposing reads -- but halves the number of workgroups as well.  Taken when that still
// leaves at least one workgroup per compute unit (the MT-NLG slice at micro-batch 1 has 16 heads x 8 = 128: it stays
// with 16 rows per wave) and the head size is 128 or 160 (at 64 the variant measures 17 % slower).  Measured with the
// kernel as it was before the grid ran heads first: 1.3B-shaped layer (4 x 16 heads x 128) 168 with 16 rows, 123 us with 32,
// slice at micro-batch 4 167 and 129 us, whole layer (128 heads) 326 and 250 us.
template <int D, int G, bool EXACT = false>
int fwd_launch_g(int b, int s, int n, int d, float scale, const void *qkv, void *a, float *lse, hipStream_t st) {
  constexpr int smem = 3 * 2 * 64 * D * 2;
  static unsigned long long attr_done = 0;
  int device;
  if (!attr_is_set(attr_done, &device)) {
    if (hipFuncSetAttribute((const void *)attn_fwd_kernel<D, G, EXACT>, hipFuncAttributeMaxDynamicSharedMemorySize, smem) !=
        hipSuccess)
      return MTNLG_HIP_ERROR;
    attr_mark_set(attr_done, device);
  }
  const int count = PairedBlocks<G>::count(s), group = HeadBlock::group(b, n, count, 32, D >= 128 ? 511 : 768);   // (768: 3 a compute unit)
  LaunchScope scope(MTNLG_K_ATTN_FWD, st);
  attn_fwd_kernel<D, G, EXACT><<<HeadBlock::grid(b, n, group, count), 512, smem, st>>>(b, s, n, d, group, scale, (const bf16 *)qkv, (bf16 *)a, lse);
  return check_launch();
}

template <int D>
int fwd_launch(int b, int s, int n, float scale, const void *qkv, void *a, float *lse, hipStream_t st) {
  if (D >= 128 && (int64_t)PairedBlocks<2>::count(s) * n * b >= 256) return fwd_launch_g<D, 2>(b, s, n, D, scale, qkv, a, lse, st);
  return fwd_launch_g<D, 1>(b, s, n, D, scale, qkv, a, lse, st);
}

}  // namespace

bool attention_mfma_supported(int dtype, int d) { return dtype == MTNLG_BF16 && (d == 64 || d == 128 || d == 160); }

bool attention_mfma_takes(int dtype, int b, int s, int n, int d) {
  return attention_mfma_supported(dtype, d) && n <= 65535 && b <= 65535 && fits(s, n, d);
}

size_t attention_bwd_workspace_bytes(int b, int s, int n, int) { return (size_t)b * n * s * sizeof(float); }

int attention_fwd_mfma(int b, int s, int n, int d, float scale, const void *qkv, void *a, float *lse,
                       hipStream_t stream) {
  if (n > 65535 || b > 65535 || !fits(s, n, d)) return MTNLG_UNSUPPORTED_SHAPE;
  switch (d) {
    case 64: return fwd_launch<64>(b, s, n, scale, qkv, a, lse, stream);
    case 128: return fwd_launch<128>(b, s, n, scale, qkv, a, lse, stream);
    case 160: return fwd_launch<160>(b, s, n, scale, qkv, a, lse, stream);
    default: return MTNLG_UNSUPPORTED_SHAPE;
  }
}

// Rows are fetched in pieces of 16 bytes from addresses that have to be aligned to 4, and results leave in pieces of 8.
static bool exact_takes(int dtype, int b, int s, int n, int d) {
  return dtype == MTNLG_BF16 && d % 8 == 0 && d <= 192 && s <= ATTENTION_F32_MAX_SEQ && n <= 65535 && b <= 65535 && fits(s, n, d);
}
static int64_t groups_of_16(int b, int s, int n) { return (int64_t)b * n * ((s + 15) / 16); }

// Against the kernels without LDS (attention_f32.hip), 444 sizes of 1 to 32 heads of 24 to 184, s 16 to 2048, and larger ones: faster
// wherever those give a wave 16 rows of its own (more than 512 groups of 16 rows).  us, those / these, forward, then backward: 2 x 1024 x 16
// heads of 96 103 / 24, 327 / 61; 4 x 2048 x 16 of 32 243 / 68, 641 / 165; 1024 x 16 of 192 104 / 31, 383 / 76; 32 x 64 x 16 of 80
// 12.4 / 7.8, 32.2 / 25.2.  With fewer groups those split the streamed side over four waves, and these win by the longer sequences:
// 512 x 16 of 96 15.4 / 13.2, 43.9 / 29.2, and at head size 24 512 x 4 6.8 / 8.4, 15.9 / 16.9.  The lines were drawn before small weights cost
// the forward kernel 6 to 8 % and before small calls of those went out backward in one launch.  Since then, forward s > 256: head sizes above
// 96 0.98 to 1.7 times as fast here; 72 to 96 up to 320 groups 0.92 to 1.09 (1712 x 2 of 96 29.7 / 31.8), beyond 1.01 to 1.5; 56 at 257 to 320 groups
// 0.86 to 0.95: they stay, with half the error of lse (1.5e-7 against 2.7e-7 rms).  Forward s <= 256, up to 512 groups: 1.04 to 1.33 here from head size
// 72 on.  Backward up to 128 groups: 0.73 to 0.95 (296 x 1 of 40 11.6 / 16.0, 597 x 1 of 96 25.7 / 30.0), as fast as those in two launches.
bool attention_exact_fwd_takes(int dtype, int b, int s, int n, int d, const void *qkv, const void *a) {
  if (!exact_takes(dtype, b, s, n, d) || (((uintptr_t)qkv | (uintptr_t)a) & 7)) return false;
  const int64_t groups = groups_of_16(b, s, n);
  return groups > 512 ? s > 32 : s > 256 && (d > 64 || (d > 32 && groups > 256));
}
bool attention_exact_bwd_takes(int dtype, int b, int s, int n, int d, const void *qkv, const void *a, const void *da, const void *dqkv) {
  if (!exact_takes(dtype, b, s, n, d) || (((uintptr_t)qkv | (uintptr_t)a | (uintptr_t)da | (uintptr_t)dqkv) & 7)) return false;
  return groups_of_16(b, s, n) > 512 ? s > 32 : s > 192 && d > 32;
}

int attention_fwd_exact(int b, int s, int n, int d, float scale, const void *qkv, void *a, float *lse, hipStream_t stream) {
#define FWD(D) fwd_launch_g<D, 1, true>
  BY_HEAD_SIZE(FWD, b, s, n, d, scale, qkv, a, lse, stream)
#undef FWD
}

}  // namespace mtnlg
