// Fused causal softmax attention on the gfx950 matrix cores (bf16 in, fp32 softmax and accumulation): forward, for head sizes 64, 128 and 160; and
// with P in fp32 (EXACT) for the others up to 192.  Some calls, short sequences above all, go to attention_fwd16.hip.  Backward: attention_bwd.hip, attention_bwd64.hip.
//
//   S = scale * q k^T (causal),  P = rowsoftmax(S),  a = P v,  lse = log sum exp(S)
//
// A workgroup owns 64 or 128 queries, 32 to a wave, held in registers as MFMA B operands (one row to a lane column); K and V stream through LDS in tiles of 64 rows, brought in by LDS
// DMA (buffer_load ... lds, no staging registers), one workgroup barrier per tile.  All products are v_mfma_f32_32x32x16_bf16 with the streamed tile as the A operand, so a product
// block comes out as C[tile row 8 (i / 4) + 4 (lane / 32) + i % 4][own row lane % 32], i < 16: S^T = K Q^T, with the softmax statistics of a query in the two lanes that share lane % 32, and P^T packed
// to bf16 is directly the B operand of O^T += V^T P^T.  That product contracts over the tile's rows: its A operand is read from the same natural [row][D] tile with the transposing LDS read
// (ds_read_b64_tr_b16: a 16-lane group reads 4 tile rows x 16 columns, each lane receives the 4 row values of its column), its k slots ordered as the first product leaves the rows, so P never leaves
// the registers and nothing is transposed in software.  No atomics: every output element has one owner, results are run-to-run identical.
//
// What bounds it: in a tile the softmax (some 75 vector instructions and 16 exponentials for 16 MFMAs at head size 128), which hides behind the MFMAs of the other workgroup on the
// unit only (the matrix pipes work 33 to 48 % of the time of a busy unit, LDS 19 to 24 %); in small calls the 3 to 4 us of a launch and the first trips to memory.  us against eight waves of 16 or 32 queries on 16x16x32 MFMAs, one workgroup to a unit: 16 heads, s = 2048, head
// size 64 24.6 -> 22.3, 128 36.0 -> 30.3, 160 38.8 -> 35.6; 20 heads of 128 51.9 -> 33.1; 128 of 128, s = 768 46.8 -> 36.9; 2 of 160, s = 256 9.3 -> 7.5; 64 of 128, s = 1024 32.2 -> 29.8.
//
// EXACT: any head size d that is a multiple of 8, in tiles of D = d rounded up to 32 columns (the DMA brings zeros past d).  P is not rounded to bf16: it goes into the second product as
// three bf16 parts that add up to it (common.h: Parts; scaled, so of any size), three MFMAs where the other kernels have one.  Inputs that are not finite take the slow path of attention_redo.h.
#include "attention_tiles.h"

namespace mtnlg {

namespace {

// Waves of 32 queries; tiles, fragments, blocks and steps as in the dq kernel of attention_bwd.hip (why 32 rows and 32x32x16 is said there).  Four to a workgroup, and two workgroups
// to a compute unit (four at head size 64): they cover each other's softmax, barriers, start and end.  SPLIT 2: a workgroup owns 64 queries, waves 0, 1 take the first 32 keys of every
// tile, waves 2, 3 the last 32, each with a maximum and a sum of its own; the results are merged through LDS at the end.  SPLIT 1: 128 queries.
constexpr int FWD_RING = 2;   // tiles of K and V in LDS: with a third one workgroup less fits a unit
struct ForwardArgs {
  int b, s, n, head_dim, group;
  bool turns;
  float scale;
  const bf16 *qkv;
  bf16 *a;
  float *lse;
};
constexpr int FWD_WAVES = 4;
template <int D, int SPLIT, bool EXACT>
__global__ __launch_bounds__(64 * FWD_WAVES, 2) void attn_fwd_kernel(ForwardArgs w) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  using T = Tile<D, true>;
  constexpr int ROWS = FWD_WAVES / SPLIT, OWNED = 32 * ROWS;   // waves with rows of their own
  constexpr int K1 = D / 16, CB = D / 32, STAGE = 2 * T::BYTES, NP = EXACT ? 3 : 1;
  constexpr int SUBS = SPLIT == 2 ? 1 : 2;                // 32-key parts of a tile that a wave takes
  constexpr int N1 = 2 * K1, NF = D == 160 ? 5 : D == 96 ? 6 : 4, PF = NF - 1;   // steps of a part: K1 for S, K1 for O
  static_assert(D >= 64 && D <= 160 && N1 % NF == 0, "fragment buffers");
  const int s = w.s, n = w.n, d = EXACT ? w.head_dim : D;
  const int count = own_blocks(s, OWNED);
  const HeadBlock hb(w.b, n, w.group, count, blockIdx.x);
  if (hb.none) return;
  const int lane = threadIdx.x & 63, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // a scalar
  const int64_t ld = (int64_t)n * 3 * d;
  const bf16 *base = w.qkv + (int64_t)hb.batch * s * ld + (int64_t)hb.head * 3 * d;
  const int64_t left = (int64_t)s * ld - 3 * (int64_t)hb.head * d;   // elements from base to the end of the sequence
  const int block = count - 1 - (w.turns ? in_turns(hb.order, count, w.b * n) : hb.order);   // falling work
  // From the thread number and not the scalar: with a scalar condition for masked tiles the compiler lays the tile's code out per path and holds more registers.
  const int rows_of = (threadIdx.x >> 6) % ROWS;
  const int block0 = block * OWNED, own0 = block0 + rows_of * 32, mine = own0 + (lane & 31);
  const int part = SPLIT == 2 ? wave / ROWS : 0, other = SPLIT == 2 ? wave ^ ROWS : wave;   // the wave with the same rows
  const float c = w.scale * kLog2e, f = EXACT ? w.scale : c;
  typename T::Lane32 ln(lane);
  const uint32_t smem_addr = lds_address(smem);
  const int ntiles = (block + 1) * (OWNED / 64) < row_blocks(s) ? (block + 1) * (OWNED / 64) : row_blocks(s);

  // waves 0, 1 bring 32 rows each of K (SPLIT 2: and 16 of Q, the own rows, which two waves need, into the last stage), waves 2, 3 of V (Q)
  constexpr int BANDS = 8 / FWD_WAVES, IPW = BANDS * T::NI;   // bands of 16 rows
  const int half = wave / (FWD_WAVES / 2), band = BANDS * (wave % (FWD_WAVES / 2));
  const uint32_t dst0 = smem_addr + half * T::BYTES + band * (T::NI * 1024);
  bf16x8 qf[K1];   // own rows: columns 16 kk + 8 h .. + 7
  if constexpr (SPLIT == 2) {
    const TileStream own(base + block0 * ld, (left - block0 * ld) * 2, OWNED * ld * 2);
#pragma unroll
    for (int i = 0; i < T::NI; ++i)
      dma16<Burst::value>(own.rsrc(), smem_addr + STAGE + (wave * T::NI + i) * 1024, T::dma_offset((uint32_t)(ld * 2), wave, lane, i, d));
  } else {
    const int qc = mine < s ? mine : s - 1;
#pragma unroll
    for (int kk = 0; kk < K1; ++kk) qf[kk] = row_chunk<EXACT>(base + (int64_t)qc * ld, 16 * kk + 8 * h, d);
  }
  TileStream stream(base + (1 + half) * d, (left - (1 + half) * d) * 2, 64 * ld * 2);
  uint32_t dma_off[IPW];
#pragma unroll
  for (int i = 0; i < IPW; ++i) dma_off[i] = T::dma_offset((uint32_t)(ld * 2), band + i / T::NI, lane, i % T::NI, d);
  constexpr int ISSUE_STEPS = IPW / 2;   // (one tile ahead: it is waited for in the same iteration)
  auto issue_step = [&](int step, int st) {
#pragma unroll
    for (int i = 0; i < IPW; ++i)
      if (i >= (step ? dma_by<IPW, ISSUE_STEPS>(step - 1) : 0) && i < dma_by<IPW, ISSUE_STEPS>(step))
        dma16<Spread::value>(stream.rsrc(), dst0 + st * STAGE + i * 1024, dma_off[i]);
  };
#pragma unroll
  for (int i = 0; i < IPW; ++i) dma16<Burst::value>(stream.rsrc(), dst0 + i * 1024, dma_off[i]);
  stream.advance();
  if constexpr (SPLIT == 2) {
    wait_and_barrier<IPW>();
#pragma unroll
    for (int kk = 0; kk < K1; ++kk) qf[kk] = T::nat32(smem + STAGE + rows_of * T::ROWS32, ln, kk);
  }
#pragma unroll
  for (int kk = 0; kk < K1; ++kk) arrive(qf[kk]);
  f32x16 o[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) o[cb] = f32x16{};
  float m = -INFINITY, l = 0.0f;   // l: this lane's share of the row sum
  wait_and_barrier<0>();   // tile 0 landed everywhere, the own rows have been read

  bf16x8 fr[NF];
  f32x16 sc;
  Parts<NP> x[2];
  const char *Kt = smem;   // stage of the tile whose fragments are being read
  auto load = [&](int i) {   // the fragment of step i
    const int sub = i / N1, r = i % N1;
    const char *k = Kt + (part + sub) * T::ROWS32;
    if (r < K1) fr[i % NF] = T::nat32(k, ln, r);
    else fr[i % NF] = T::tr32(k + T::BYTES, ln, (r - K1) / 2, r % 2);
  };
#pragma unroll
  for (int i = 0; i < PF; ++i) load(i);
  __builtin_amdgcn_sched_barrier(0);

  int cur = 0;
  auto tile = [&](auto TAKEN, int it) __attribute__((always_inline)) {   // TAKEN: parts, SUBS or the first only
    constexpr int N = decltype(TAKEN)::value * N1;
    ln.here();
    const int next = cur ^ 1;   // stage of tile it + 1
    auto step = [&](auto I) __attribute__((always_inline)) {
      constexpr int i = decltype(I)::value, sub = i / N1, r = i % N1;
      const int row = it * 64 + 32 * (part + sub);
      if (r == 0) sc = f32x16{};
      if (r == K1) {
        // element e: key row + 8 (e / 4) + 4 h + e % 4, query `mine`
        if (row + 31 > own0) {  // wave-uniform: diagonal (or past-the-end keys) among these keys
#pragma unroll
          for (int e = 0; e < 16; ++e)
            if (row + 8 * (e / 4) + 4 * h + e % 4 > mine) sc[e] = -INFINITY;
        }
        // m tracks the running maximum of the raw scores; exponents are taken in base 2 with the scale folded in: p = 2^(s c - m c).  The reference maximum only
        // follows when the row maximum has outgrown it by more than 2^8 in the exponent's units (any reference gives the same sums; this one keeps p <= 256
        // and makes rescaling O rare).  -inf until a part has seen a key of the row.  A weight of 1, the reference's, is a bf16 value, others round; so a wave that takes whole tiles follows to the
        // maximum of the first one, as SPLIT 2 has one of each half of the keys: with that of the first 32 keys the results are 1.1 % further off (randn inputs, s 512 to 2048, rms 2.04e-3 against 2.01e-3).
        float mx = sc[0];
#pragma unroll
        for (int e = 1; e < 16; ++e) mx = fmaxf(mx, sc[e]);
        mx = pair_max(mx);
        const float m_new = mx * c > m * c + (sub == 1 && it == 0 ? 0.0f : 8.0f) ? mx : m;
        const float ref = m_new == -INFINITY ? 0.0f : m_new;
        const float mc = EXACT ? product_of(ref, w.scale) : ref * c;
        float rs = 0.0f;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          sc[e] = weight<EXACT>(sc[e], f, mc);
          rs += sc[e];
        }
        const float alpha = m == m_new ? 1.0f : EXACT ? exact_exp(product_of(m, w.scale) - mc) : fast_exp2((m - m_new) * c);   // EXACT: by what the weights are relative to, rounded as it is
        l = l * alpha + rs;
        m = m_new;
        if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {   // a reference maximum moved: rescale O
#pragma unroll
          for (int cb = 0; cb < CB; ++cb) o[cb] *= alpha;
        }
        x[0] = weights16<EXACT>(sc, 0);
        x[1] = weights16<EXACT>(sc, 1);
      }
      if (i == N - PF) {   // all of tile `it` has been read; tile it + 1 landed everywhere
        wait_and_barrier<0>();
        Kt = smem + next * STAGE;
      }
      load((i + PF) % N);
      if (i < ISSUE_STEPS) issue_step(i, next);
      const bf16x8 &v = fr[i % NF];
      if constexpr (r < K1) sc = MFMA32(v, qf[r], sc);
      else o[(r - K1) / 2] = mma_weights32(v, x[r % 2], o[(r - K1) / 2]);
      __builtin_amdgcn_sched_barrier(0);
    };
    for_each_step(step, std::make_integer_sequence<int, N>{});
    stream.advance();
    cur = next;
  };
  // How many 32-key parts this wave takes: those with a key that one of its queries sees.  The rest, at the end, it passes over: an infinity or NaN there would reach its rows (0 x inf).
  const int visible = visible_parts(block0 / 32 + wave % ROWS, part, SUBS, ntiles);
  int it = 0;
  // Where the loop lies in 32-byte pieces of code counts for a wave that is alone on its SIMD (2 heads of 64, s = 3749: 31.1 to 33.2 us from place to place; 20 and more workgroups to a unit: nothing).
  asm volatile(".p2align 6");
  for (; it < visible / SUBS; ++it) tile(std::integral_constant<int, SUBS>{}, it);
  if constexpr (SUBS == 2) {
    if (visible % 2) tile(std::integral_constant<int, 1>{}, it++);
  }
  for (; it < ntiles; ++it) {   // passed over: its share of the next tile, and the barrier
#pragma unroll
    for (int i = 0; i < IPW; ++i) dma16<Burst::value>(stream.rsrc(), dst0 + (cur ^ 1) * STAGE + i * 1024, dma_off[i]);
    wait_and_barrier<0>();
    stream.advance();
    cur ^= 1;
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");   // the look-ahead tiles, which nobody uses

  l += __shfl_xor(l, 32, 64);
  f32x4 *slots = reinterpret_cast<f32x4 *>(smem) + lane;
  float *const stat = reinterpret_cast<float *>(smem + 2 * FWD_WAVES * CB * 1024);   // maximum and sum of each wave
  if constexpr (SPLIT == 2) {   // the part's results relative to the larger of the two maxima
    __syncthreads();   // the rings are no longer read
    stat[wave * 128 + lane] = m;
    stat[wave * 128 + 64 + lane] = l;
    __syncthreads();
    const float mo = stat[other * 128 + lane], lo = stat[other * 128 + 64 + lane], both = fmaxf(m, mo);   // finite: key 0 is never masked
    auto relative = [&](float x) { return EXACT ? exact_exp(product_of(x, w.scale) - product_of(both, w.scale)) : fast_exp2((x - both) * c); };
    const float mul = relative(m);
    l = part ? fmaf(l, mul, lo * relative(mo)) : fmaf(lo, relative(mo), l * mul);
    m = both;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) o[cb] *= mul;
    // the two waves with the same rows each hand over half of their column blocks' elements (q 0, 1 or 2, 3) and finish the other half
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int q = 0; q < 2; ++q) slots[((wave * CB + cb) * 2 + q) * 64] = part ? quarter_of(o[cb], q) : quarter_of(o[cb], 2 + q);
    __syncthreads();
  }
  float z = 0.0f;   // EXACT: NaN where a result is not finite
  bf16 *const out = w.a + ((int64_t)hb.batch * s + mine) * ((int64_t)n * d) + (int64_t)hb.head * d;
  float *const out_lse = w.lse + ((int64_t)hb.batch * n + hb.head) * s + mine;
  const float inv = EXACT ? 1.0f / l * PARTS_UNSCALE : 1.0f / l;
  auto put = [&](int cb, int q, f32x4 sum) {   // columns 32 cb + 8 q + 4 h .. + 3
    const int col = 32 * cb + 8 * q + 4 * h;
    if (EXACT && col >= d) return;
    bf16x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float r = sum[e] * inv;
      if constexpr (EXACT) z = fmaf(r, 0.0f, z);
      v[e] = (bf16)r;
    }
    *reinterpret_cast<bf16x4 *>(out + col) = v;
  };
  if (mine < s) {
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      if constexpr (SPLIT == 2) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const f32x4 rest = slots[((other * CB + cb) * 2 + q) * 64];
          if (part) put(cb, 2 + q, quarter_of(o[cb], 2 + q) + rest);
          else put(cb, q, quarter_of(o[cb], q) + rest);
        }
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) put(cb, q, quarter_of(o[cb], q));
      }
    }
    if (h == 0 && part == 0) *out_lse = EXACT ? plus_log(product_of(m, w.scale), l) : (m * c + log2f(l)) * kLn2;
  }
  if constexpr (EXACT) {
    if constexpr (SPLIT == 2) z = either_part(z, smem, wave, other, part, lane);
    if (!all_finite(z)) {
      const int lr = lane & 15, g = lane >> 4;
#pragma unroll 1
      for (int k = 0; k < 2; ++k) {
        const int q = own0 + 16 * k + lr, last = own0 + 16 * k + 15;
        redo_fwd<bf16, D>(base, ld, s, d, w.scale, q, last < s ? last : s - 1, g, w.a + ((int64_t)hb.batch * s + q) * ((int64_t)n * d) + (int64_t)hb.head * d,
                          w.lse + ((int64_t)hb.batch * n + hb.head) * s + q);
      }
    }
  }
}

template <int D, int SPLIT, bool EXACT = false>
int fwd_launch_rows(int b, int s, int n, int d, float scale, const void *qkv, void *a, float *lse, hipStream_t st) {
  constexpr int merge = SPLIT == 2 ? FWD_WAVES * (2 * (D / 32) * 1024 + 512) : 0, ring = FWD_RING * 2 * Tile<D>::BYTES, smem = ring > merge ? ring : merge;
  static unsigned long long attr_done = 0;
  int device;
  if (!attr_is_set(attr_done, &device)) {
    MTNLG_TRY(set_lds(attn_fwd_kernel<D, SPLIT, EXACT>, smem));
    attr_mark_set(attr_done, device);
  }
  constexpr int EACH = D <= 64 ? 4 : 2, ALL = 256 * EACH;   // workgroups to a compute unit, and on the chip at once
  const int count = own_blocks(s, 32 * FWD_WAVES / SPLIT), group = HeadBlock::group(b, n, count, 32, ALL);
  LaunchScope scope(MTNLG_K_ATTN_FWD, st);
  attn_fwd_kernel<D, SPLIT, EXACT><<<HeadBlock::grid(b, n, group, count), 64 * FWD_WAVES, smem, st>>>(
      ForwardArgs{b, s, n, d, group, (int64_t)b * n * count <= ALL, scale, (const bf16 *)qkv, (bf16 *)a, lse});
  return check_launch();
}

// Sequences of one or two blocks of 64 rows: 16 rows to a wave (attention_fwd16.hip) while few workgroups share a unit.  Eight waves to a block and no merge make a shorter chain there.  Times as fast
// as these, one block (up to `few` of them), then two (257 to 512): head size 64 1.01 to 1.15, 1.02 to 1.12; 33 to 64 with P in fp32 1.02 to 1.15, 1.02 to 1.05; 65 to 96 1.00 to
// 1.16, 1.05 to 1.11; 97 to 128 1.1 to 1.18, 1.05 to 1.2; 129 to 160 1.1 to 1.2, 1.1 to 1.28.  (700 and 1800 sizes; d 64 3.3 / 3.7 us, 8 x 80 x 32 4.6 / 5.1.)  Head sizes 128 and 160 only up to 32
// tokens and 255 blocks, 1.02 to 1.1.
bool short_on_rows16(int s, int64_t blocks, int few) { return s <= 64 ? blocks <= few : s <= 128 && blocks > 256 && blocks <= 512; }

// Workgroups of 128 queries halve the tiles' way into LDS and what a workgroup costs besides its tiles; those of 64 even out better, and where all run at once a full
// round of either does better than a part of one.  By workgroups of 128; us with 64 / 128 queries: head size 128: 64 heads, s = 1024 (512) 30.4 / 29.8; 128, 768 (768) 36.9 /
// 42.1; 48, 2048 (768) 70.1 / 70.4; 256, 512 (1024) 39.1 / 37.8; 128, 2048 (2048) 174 / 165; 512, 768 (3072) 155 / 134; 160: 64, 1024 (512) 37.6 / 35.0; 128, 768 (768) 45.0 / 49.8; 64, 2048
// (1024) 108 / 101; 512, 768 (3072) 194 / 166.  Head size 64, four workgroups to a unit: 64, 2048 (1024) 60.4 / 50.6; 128, 1024 (1024) 33.6 / 30.6; 256, 512 (1024) 23.1 / 22.3; but 512, 256
// (1024) 17.8 / 18.7; 48, 2048 (768) 39.0 / 50.1; 512, 768 (3072) 72.4 / 75.8.
// Head sizes 128 and 160, 800 sizes: from 513 workgroups of 128 on they are 1.0 to 1.1 times as fast as those of 64 beyond 1024 tokens, 1.2 to 1.7 if the number of heads is odd and every workgroup's K and V come
// from another XCD's L2 (47 heads, s = 2048 of 128 114 / 73, of 160 148 / 91; 1486 of 160 89 / 60); s 577 to 1024 and odd 0.93 to 1.4 (at 160 from 385 on).
// Head size 64 besides: where 128 queries hold the whole sequence, beyond 896 blocks of 64 (s 65 to 128: 1.02 to 1.2 times as fast), and of sequences up to 384 those whose workgroups of 64 just fill
// the chip (897 to 1024: 384 tokens x 170 heads 15.0 / 13.5).
template <int D>
int fwd_launch(int b, int s, int n, float scale, const void *qkv, void *a, float *lse, hipStream_t st) {
  const int64_t large = (int64_t)b * n * own_blocks(s, 128), blocks = (int64_t)b * n * row_blocks(s);
  const bool odd = (int64_t)b * n % 2 != 0;
  bool rows128 = large >= 1024 || (large > 448 && large <= 512) || (s > 1024 && large > 512) || (odd && s > 576 && large > (D == 128 ? 448 : 384));
  const bool rows16 = D == 64 ? short_on_rows16(s, blocks, 512) : (s <= 32 && blocks < 256) || heads_scattered(b, n, s, D);
  if (rows16) return attention_fwd_mfma16(b, s, n, D, scale, qkv, a, lse, st);
  if constexpr (D == 64) {
    rows128 = (s >= 512 && large > 896 && large <= 1024) || (s > 64 && s <= 384 && blocks > 896 && (s <= 128 || (s > 192 && blocks <= 1024)));
  }
  if (rows128) return fwd_launch_rows<D, 1>(b, s, n, D, scale, qkv, a, lse, st);
  return fwd_launch_rows<D, 2>(b, s, n, D, scale, qkv, a, lse, st);
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
  // 16 rows to a wave where that is as fast or faster: up to head size 32, above 160, short sequences, and from 65 to 96 with many blocks of 64 rows.  us, those / these: 64 heads, s = 1536, of 32
  // 42 / 47; 16, 2048 of 192 62 / 76; of 96 32, 1024 (512 blocks) 24.3 / 22.3; 48, 1024 (768) 32.8 / 31.7; 96, 512 (768) 20.8 / 24.1; 64, 1024 (1024) 34.4 / 38.7; 64, 2048
  // (2048) 108 / 118.  The others: 64, 1024 of 48 29.6 / 26.9; 4, 2048 of 104 42.2 / 36.3; 64, 2048 of 120 161 / 140, of 144 181 / 164.  65 to 96 at s 65 to 96 those 1.01 to 1.2 times as fast throughout, at
  // s 97 to 128 beyond 256 blocks up to 1.18; at s 129 to 192 1.08 from 513 to 768, 0.93 beyond.
  const int64_t blocks = (int64_t)b * n * row_blocks(s);
  bool rows16 = d <= 32 || d > 160 || short_on_rows16(s, blocks, d <= 64 ? 512 : d <= 96 ? 384 : 256);
  if (d > 64 && d <= 96 && s > 64) rows16 = s <= 96 || (s <= 128 ? blocks > 256 : s <= 192 ? blocks > 512 && blocks <= 768 : blocks >= 704);
  if (d > 64 && s > 192 && s <= (d > 128 ? 768 : 384) && heads_scattered(b, n, s, d)) rows16 = true;
  if (rows16) return attention_fwd_exact16(b, s, n, d, scale, qkv, a, lse, stream);
  if (d <= 64) return fwd_launch_rows<64, 2, true>(b, s, n, d, scale, qkv, a, lse, stream);
  if (d <= 96) return fwd_launch_rows<96, 2, true>(b, s, n, d, scale, qkv, a, lse, stream);
  if (d <= 128) return fwd_launch_rows<128, 2, true>(b, s, n, d, scale, qkv, a, lse, stream);
  return fwd_launch_rows<160, 2, true>(b, s, n, d, scale, qkv, a, lse, stream);
}

}  // namespace mtnlg
