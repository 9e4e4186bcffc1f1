// Backward of the fused causal attention (attention_mfma.hip: forward), for bf16 head sizes 128 and 160 and, with P and dS in fp32 (EXACT), for the longer sequences of
// the others up to 192 (the rest: attention_bwd64.hip; attention_bwd_exact says which).
//
//   D_t = da_t . a_t:  dP = da v^T,  dS = P o (dP - D),  dq = scale dS k,  dk = scale dS^T q,  dv = P^T da.
//
// Two kernels (one launch for small calls): dq, which streams K and V past its own queries, and dk / dv, which streams Q and dO past its own keys; tiles come into
// LDS as in the forward kernel.  No atomics: every output element has one owner, results are run-to-run identical.  Both form S and dP: writing dS
// instead would move 2 bytes a score, four times what is read and written otherwise.
//
// What bounds them: the MFMAs and the vector work that does not hide behind them.  The matrix pipes work 44 to 57 % of the time of a busy unit in dq and 42 to 49 % in dk / dv (head sizes 128 and 160, one
// to four sequences of 2048, 16 heads; EXACT 34 to 48 %), LDS 24 to 38 %, without bank conflicts; the rest are exponentials, dS, packing, barriers, and the 3 to 6 us that a workgroup costs at its start and end.  us against the kernels before, 16 own rows a wave on 16x16x32 MFMAs: 1990 tokens
// x 16 heads of 160 112 -> 97, 2048 x 16 of 128 98 -> 81, 4 x 2048 x 16 of 128 325 -> 270, 2048 x 20 of 128 137 -> 102, 384 x 256 of 160 126 -> 105, 256 x 2 of 160 13.8 -> 11.2.
#include "attention_tiles.h"

namespace mtnlg {

namespace {

// On v_mfma_f32_32x32x16_bf16, 32 own rows to a wave: a vector instruction hides behind a matrix instruction only beyond its first 16 cycles, so
// that of the vector work (exponentials, dS, addresses; some 200 instructions a tile and SIMD) hardly any hides behind 16x16x32 MFMAs of 16 cycles, and half of the time of a 32x32x16 has
// room for it (measured with two waves to a SIMD, cycles for an MFMA and n vector instructions: 16x16x32 17 alone, 27 with 4, 40 with 8;
// 32x32x16 32, 34, 42).  Every fragment read from LDS feeds 32 own rows; with 16 own rows a wave, reading fragments (128 to 220 bytes a clock by kind)
// took 1.5 to 1.8 times as long as the MFMAs.
// Blocks are C[streamed row 8 (i / 4) + 4 (lane / 32) + i % 4][own row lane % 32], i < 16; the second product takes them as they are: slot (lane / 32, e) of its
// 16-row step t is row 16 t + 4 (lane / 32) + e for e < 4, 16 t + 8 + 4 (lane / 32) + e - 4 otherwise, elements 8 t .. 8 t + 7 of the lane.
//
// SPLIT 2: a workgroup owns 64 rows; half of the waves take the first 32 rows of every streamed tile, half the last 32, and the partial results are
// merged through LDS at the end.  SPLIT 1: 128 rows, every wave takes whole tiles.  Blocks go out in the order of falling work.
//
// A step is one fragment and its MFMA (EXACT: three in the second product).  Fragments are read PF steps ahead across the end of a tile, and a tile's barrier
// stands PF steps before its end.  A wave passes over the 32-row parts that none of its rows sees: they cost it the barriers and its share of the DMA, and what is in them does not reach its results.
// what both kernels know of the head that a workgroup works on
template <bool EXACT, int D>
struct Head {
  int s, d, lane;
  int64_t ld, pld;
  const bf16 *base, *dab, *ab;
  const float *lse;
  float *Dvec;
  bf16 *out;
  int64_t left, pleft;   // elements from base, dab to the end of the sequence
  __device__ __forceinline__ Head(const BackwardArgs &w, int batch, int head) : s(w.s), d(EXACT ? w.head_dim : D), lane(threadIdx.x & 63) {
    ld = (int64_t)w.n * 3 * d;
    pld = (int64_t)w.n * d;
    base = w.qkv + (int64_t)batch * s * ld + (int64_t)head * 3 * d;
    out = w.dqkv + (base - w.qkv);
    dab = w.da + (int64_t)batch * s * pld + (int64_t)head * d;
    ab = w.a + (dab - w.da);
    const int64_t row = ((int64_t)batch * w.n + head) * s;
    lse = w.lse + row;
    Dvec = w.Dvec + row;
    left = (int64_t)s * ld - 3 * (int64_t)head * d;
    pleft = (int64_t)s * pld - (int64_t)head * d;
  }
  // one of the two matrices of a side (queries: Q and dO, else K and V)
  __device__ __forceinline__ uint32_t pitch_bytes(bool queries, int second) const { return (uint32_t)((queries && second ? pld : ld) * 2); }
  __device__ __forceinline__ TileStream matrix(bool queries, int second, int row0, int rows) const {   // from a row on, in tiles of so many
    const int64_t p = queries && second ? pld : ld;
    const bf16 *first = queries ? (second ? dab : base) : base + (1 + second) * d;
    const int64_t n = queries ? (second ? pleft : left) : left - (1 + second) * d;
    return TileStream(first + row0 * p, (n - row0 * p) * 2, rows * p * 2);
  }
};

// ------------------------------------------------------------------ backward: dq (and D)
// Four waves, and two workgroups to a compute unit where registers and LDS allow: they cover each other's start, end and barriers.
constexpr int DQ_THREADS = 256;
constexpr int dq_ring(int d, bool exact) { return d <= (exact ? 128 : 160) ? 2 : 3; }
template <int D, int SPLIT, bool EXACT>
__device__ __forceinline__ void dq_block(unsigned place, char *smem, const BackwardArgs &w) {
  using T = Tile<D, true>;
  constexpr int OWNED = SPLIT == 2 ? 64 : 128;
  constexpr int K1 = D / 16, STAGE = 2 * T::BYTES, RING = dq_ring(D, EXACT), NP = EXACT ? 3 : 1;
  constexpr int SUBS = SPLIT == 2 ? 1 : 2;                // 32-row parts of a tile that a wave takes
  constexpr int N1 = 3 * K1, NF = D == 160 ? 5 : D == 64 ? 4 : 6, PF = NF - 1;   // steps of a part: K1 for S, K1 for dP, K1 for dq
  static_assert(N1 % NF == 0, "fragment buffers");
  const HeadBlock hb(w.b, w.n, w.group, own_blocks(w.s, OWNED), place);
  if (hb.none) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // a scalar
  const Head<EXACT, D> at(w, hb.batch, hb.head);
  const int half = wave >> 1;   // waves 0, 1 bring 32 rows each of K (of Q, the own rows), waves 2, 3 of V (dO)
  const int s = at.s, d = at.d, lane = at.lane, g = lane >> 4, lr = lane & 15, h = lane >> 5;
  const int heads = w.b * w.n, count = own_blocks(s, OWNED);   // falling work
  const int block = count - 1 - (RING == 2 && heads * count <= 512 ? in_turns(hb.order, count, heads) : hb.order);
  const int rows_of = SPLIT == 2 ? (threadIdx.x >> 6) & 1 : threadIdx.x >> 6;   // (from the thread number: see the forward kernel)
  const int block0 = block * OWNED, own0 = block0 + rows_of * 32, mine = own0 + (lane & 31);
  const int part = SPLIT == 2 ? wave >> 1 : 0;
  const float f = EXACT ? w.scale : w.scale * kLog2e;
  typename T::Lane32 ln(lane);
  const uint32_t smem_addr = lds_address(smem);
  const int ntiles = (block + 1) * (OWNED / 64) < row_blocks(s) ? (block + 1) * (OWNED / 64) : row_blocks(s);
  const int visible = visible_parts(block0 / 32 + (SPLIT == 2 ? wave & 1 : wave), part, SUBS, ntiles);   // the rest of the 32-key parts is passed over (as in the forward kernel)

  constexpr int IPW = 2 * T::NI;
  auto offset = [&](bool queries, int i) {
    return T::dma_offset(at.pitch_bytes(queries, half), 2 * (wave & 1) + i / T::NI, lane, i % T::NI, d);
  };
  const uint32_t dst0 = smem_addr + half * T::BYTES + (wave & 1) * (2 * T::NI * 1024);
  if constexpr (SPLIT == 2) {   // two waves need every own row: through LDS, in the last stage
    const TileStream own = at.matrix(true, half, block0, 64);
#pragma unroll
    for (int i = 0; i < IPW; ++i) dma16<Burst::value>(own.rsrc(), dst0 + (RING - 1) * STAGE + i * 1024, offset(true, i));
  }
  const int qc = mine < s ? mine : s - 1;
  bf16x8 of0[K1], of1[K1], av[K1];   // own rows of Q, dO and a: columns 16 kk + 8 h .. + 7
#pragma unroll
  for (int kk = 0; kk < K1; ++kk) {
    const int col = 16 * kk + 8 * h;
    av[kk] = row_chunk<EXACT>(at.ab + (int64_t)qc * at.pld, col, d);
    if constexpr (SPLIT == 1) {
      of0[kk] = row_chunk<EXACT>(at.base + (int64_t)qc * at.ld, col, d);
      of1[kk] = row_chunk<EXACT>(at.dab + (int64_t)qc * at.pld, col, d);
    }
  }
  float lsf = at.lse[qc], dsum;
  TileStream stream = at.matrix(false, half, 0, 64);
  uint32_t dma_off[IPW];
#pragma unroll
  for (int i = 0; i < IPW; ++i) dma_off[i] = offset(false, i);
  auto issue_step = [&](auto STEPS, int step, int st) {   // over the first STEPS steps of a tile
    constexpr int steps = decltype(STEPS)::value;
#pragma unroll
    for (int i = 0; i < IPW; ++i)
      if (i >= (step ? dma_by<IPW, steps>(step - 1) : 0) && i < dma_by<IPW, steps>(step))
        dma16<Spread::value>(stream.rsrc(), dst0 + st * STAGE + i * 1024, dma_off[i]);
  };
#pragma unroll
  for (int t = 0; t < RING - 1; ++t) {
#pragma unroll
    for (int i = 0; i < IPW; ++i) dma16<Burst::value>(stream.rsrc(), dst0 + t * STAGE + i * 1024, dma_off[i]);
    stream.advance();
  }
  if constexpr (SPLIT == 2) {
    wait_and_barrier<(RING - 1) * IPW>();
    const char *own = smem + (RING - 1) * STAGE + rows_of * T::ROWS32;
#pragma unroll
    for (int kk = 0; kk < K1; ++kk) {
      of0[kk] = T::nat32(own, ln, kk);
      of1[kk] = T::nat32(own + T::BYTES, ln, kk);
    }
  }
  {   // D on the diagonal of a dO^T, by the same MFMAs as dP (EXACT: where a row has one key, a = v, the two cancel exactly)
    f32x16 t = {};
#pragma unroll
    for (int kk = 0; kk < K1; ++kk) t = MFMA32(av[kk], of1[kk], t);
    const int row = lane & 31, i = 4 * (row >> 3) + (row & 3);
    float v = t[0];
#pragma unroll
    for (int e = 1; e < 16; ++e) v = i == e ? t[e] : v;
    dsum = __shfl(EXACT ? v : -v, row + 32 * (row >> 2 & 1), 64);   // D, or -D, as dP's accumulators start
    if constexpr (!EXACT) lsf *= kLog2e;
  }
  if (mine < s && h == 0 && part == 0) at.Dvec[mine] = dsum;
#pragma unroll
  for (int kk = 0; kk < K1; ++kk) {
    arrive(of0[kk]);
    arrive(of1[kk]);
  }
  arrive(lsf);
  arrive(dsum);
  f32x16 acc[D / 32];
#pragma unroll
  for (int cb = 0; cb < D / 32; ++cb) acc[cb] = f32x16{};
  wait_and_barrier<(RING - 2) * IPW>();   // tile 0 landed everywhere, the own rows have been read

  bf16x8 fr[NF];
  f32x16 sc, pc;   // pc accumulates dP - D (EXACT: dP)
  Parts<NP> x[2];
  const char *Kt = smem;   // stage of the tile whose fragments are being read
  auto load = [&](int i) {   // the fragment of step i
    const int sub = i / N1, r = i % N1;
    const char *k = Kt + part * T::ROWS32 + sub * T::ROWS32;
    bf16x8 &v = fr[i % NF];
    if (r < K1) v = T::nat32(k, ln, r);
    else if (r < 2 * K1) v = T::nat32(k + T::BYTES, ln, r - K1);
    else v = T::tr32(k, ln, (r - 2 * K1) / 2, r % 2);
  };
#pragma unroll
  for (int i = 0; i < PF; ++i) load(i);
  __builtin_amdgcn_sched_barrier(0);

  int cur = 0;
  auto next_of = [](int cur) { return cur == RING - 1 ? 0 : cur + 1; };                         // stages of tiles it + 1
  auto ahead_of = [&](int cur) { return RING == 2 ? next_of(cur) : cur == 0 ? 2 : cur - 1; };   // and it + RING - 1
  auto tile = [&](auto TAKEN, int it) __attribute__((always_inline)) {   // TAKEN: parts, SUBS or the first only
    constexpr int N = decltype(TAKEN)::value * N1;
    constexpr int ISSUE_STEPS = RING == 2 ? IPW / 2 : N - PF;   // (one tile ahead: it is waited for in the same iteration)
    ln.here();
    const int next = next_of(cur), nn = ahead_of(cur);
    auto step = [&](auto I) __attribute__((always_inline)) {
      constexpr int i = decltype(I)::value, sub = i / N1, r = i % N1;
      const int row = it * 64 + 32 * (part + sub);
      if (r == 0) {
        const float start = EXACT ? 0.0f : dsum;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          sc[e] = 0.0f;
          pc[e] = start;
        }
      }
      if (r == K1 && row + 31 > own0) {   // wave-uniform: diagonal (or past-the-end keys) among these keys
        const int h4 = (lane_here() >> 5) * 4;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int key = row + 8 * (e / 4) + h4 + e % 4;
          if (key > mine || key >= s) sc[e] = -INFINITY;
        }
      }
      // the vector work: weights over dP, dS^T = P^T o (dP^T - D) behind it
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        if (r == K1 + e * K1 / 16) sc[e] = weight<EXACT>(sc[e], f, lsf);
        if (r == 2 * K1) pc[e] = (EXACT ? pc[e] - dsum : pc[e]) * sc[e];
      }
      if (r == 2 * K1) {
        x[0] = weights16<EXACT>(pc, 0);
        x[1] = weights16<EXACT>(pc, 1);
      }
      if (i == N - PF) {   // all of tile `it` has been read; tile it + 1 landed everywhere
        wait_and_barrier<(RING - 2) * IPW>();
        Kt = smem + next * STAGE;
      }
      load((i + PF) % N);
      if (i < ISSUE_STEPS) issue_step(std::integral_constant<int, ISSUE_STEPS>{}, i, nn);
      const bf16x8 &v = fr[i % NF];
      if constexpr (r < K1) sc = MFMA32(v, of0[r], sc);
      else if constexpr (r < 2 * K1) pc = MFMA32(v, of1[r - K1], pc);
      else acc[(r - 2 * K1) / 2] = mma_weights32(v, x[r % 2], acc[(r - 2 * K1) / 2]);
      __builtin_amdgcn_sched_barrier(0);
    };
    for_each_step(step, std::make_integer_sequence<int, N>{});
    stream.advance();
    cur = next;
  };
  int it = 0;
  for (; it < visible / SUBS; ++it) tile(std::integral_constant<int, SUBS>{}, it);
  if constexpr (SUBS == 2) {
    if (visible % 2) tile(std::integral_constant<int, 1>{}, it++);
  }
  for (; it < ntiles; ++it) {   // passed over: its share of a later tile, and the barrier
    const int nn = ahead_of(cur);
#pragma unroll
    for (int i = 0; i < IPW; ++i) dma16<Burst::value>(stream.rsrc(), dst0 + nn * STAGE + i * 1024, dma_off[i]);
    wait_and_barrier<(RING - 2) * IPW>();
    stream.advance();
    cur = next_of(cur);
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");   // the look-ahead tiles, which nobody uses

  float z = 0.0f;   // EXACT: NaN where a result is not finite
  bf16 *out = at.out + (int64_t)mine * at.ld;
  const int h4 = (lane_here() >> 5) * 4;
  auto put = [&](int cb, int q, f32x4 sum) {   // elements 4 q .. + 3 of column block cb: columns 32 cb + 8 q + 4 h .. + 3
    const int col = 32 * cb + 8 * q + h4;
    if (EXACT && col >= d) return;
    bf16x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float r = (EXACT ? sum[e] * PARTS_UNSCALE : sum[e]) * w.scale;
      if constexpr (EXACT) z = fmaf(r, 0.0f, z);
      o[e] = (bf16)r;
    }
    *reinterpret_cast<bf16x4 *>(out + col) = o;
  };
  // SPLIT 2: the two waves with the same rows each hand over half of their column blocks' elements (q 0, 1 or 2, 3) and finish the other half
  f32x4 *slots = reinterpret_cast<f32x4 *>(smem) + lane;
  if constexpr (SPLIT == 2) {
    __syncthreads();   // the rings are no longer read
#pragma unroll
    for (int cb = 0; cb < D / 32; ++cb)
#pragma unroll
      for (int q = 0; q < 2; ++q) slots[((wave * (D / 32) + cb) * 2 + q) * 64] = part ? quarter_of(acc[cb], q) : quarter_of(acc[cb], 2 + q);
    __syncthreads();
  }
  if (mine < s) {
#pragma unroll
    for (int cb = 0; cb < D / 32; ++cb) {
      if constexpr (SPLIT == 2) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const f32x4 other = slots[(((wave ^ 2) * (D / 32) + cb) * 2 + q) * 64];
          if (part) put(cb, 2 + q, quarter_of(acc[cb], 2 + q) + other);
          else put(cb, q, quarter_of(acc[cb], q) + other);
        }
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) put(cb, q, quarter_of(acc[cb], q));
      }
    }
  }
  if constexpr (EXACT) {
    if constexpr (SPLIT == 2) z = either_part(z, smem, wave, wave ^ 2, part, lane);
    if (!all_finite(z)) {
#pragma unroll 1
      for (int c = 0; c < 2; ++c) {
        const int q = own0 + 16 * c + lr, last = own0 + 16 * c + 15;
        const float ds = __shfl(dsum, 16 * c + lr, 64);
        redo_dq<bf16, D>(at.base, at.ld, at.dab, at.pld, s, d, w.scale, q, last < s ? last : s - 1, at.lse[q < s ? q : s - 1], ds, g, at.out + (int64_t)q * at.ld);
      }
    }
  }
}

// ------------------------------------------------------------------ backward: dk, dv
// Eight waves, two to a SIMD, in pairs (roles 0 and 1) of which each owns 32 keys and takes 32 rows of a tile: role 0 forms S and P and accumulates dv,
// role 1 forms dP and dS and accumulates dk, so that either holds one of K and V and one of the results (both of both would take all 256 registers).  P goes to
// role 1 through LDS in fp32.  LAG: the second product runs one tile behind, so that one barrier a tile serves the exchange as well, and the vector
// work issues between MFMAs that do not wait for it; else, where LDS has no room for a third tile and two sets of P, a second barrier stands
// behind the exchange.
// SPLIT 1: tiles of 32 rows.
constexpr int DKV_THREADS = 512;
constexpr int ONE_LAUNCH_ROWS = 4096;   // whose D a workgroup with OWN_D has room for
template <int D, int OWNED, int ROWS, bool EXACT, bool OWN_D>
struct DkvLds {
  static constexpr int GROUPS = OWNED / 32, PARTS = ROWS / 32, PAIRS = GROUPS * PARTS;
  static constexpr int MATRIX = ROWS * D * 2, STAGE = 2 * MATRIX + 512;   // Q tile, dO tile, 256 bytes each of lse and -D (EXACT: D)
  static constexpr int XCHG = PAIRS * 4096;                               // P of a tile
  static constexpr int ROOM = 160 * 1024 - (OWN_D ? ONE_LAUNCH_ROWS * (int)sizeof(float) : 0);
  static constexpr bool LAG = 3 * STAGE + 2 * XCHG <= ROOM;
  static constexpr int RING = LAG ? (4 * STAGE + 2 * XCHG <= ROOM ? 4 : 3) : (3 * STAGE + XCHG <= ROOM ? 3 : 2);
  static constexpr int AHEAD = RING - (LAG ? 2 : 1);   // tiles that are fetched ahead
  static constexpr int BYTES = RING * STAGE + (LAG ? 2 : 1) * XCHG;
  // the own rows of K and V come into the end of it first, beside them as many of the first tiles as there is room for
  static constexpr int OWN = BYTES - OWNED / 64 * 2 * Tile<D>::BYTES;
  static constexpr int FIRST = OWN / STAGE < AHEAD ? OWN / STAGE : AHEAD;
  static_assert(128 * PAIRS == DKV_THREADS, "");
  static_assert(BYTES <= ROOM && OWN >= 0 && (PARTS == 1 || BYTES >= 8 * (D / 32) * 2 * 1024), "");
};
// OWN_D: D is computed here (a: read then), not taken from the dq workgroups.
template <int D, int OWNED, int ROWS, bool EXACT, bool OWN_D>
__device__ __forceinline__ void dkv_block(unsigned place, char *smem, const BackwardArgs &w) {
  using T = Tile<D, true>;
  using L = DkvLds<D, OWNED, ROWS, EXACT, OWN_D>;
  constexpr int K1 = D / 16, CB = D / 32, STAGE = L::STAGE, RING = L::RING, AHEAD = L::AHEAD, NP = EXACT ? 3 : 1;
  constexpr bool LAG = L::LAG;
  constexpr int N = 2 * K1, NF = D == 128 ? 8 : D == 160 ? 10 : 4, PF = D == 128 ? 5 : D == 160 ? 6 : NF - 1;   // steps of a tile: K1 for the first product, K1 for the second (LAG: of the tile before)
  constexpr int HAND_OVER = LAG ? N - PF : K1;
  static_assert(D >= 64 && D <= 192 && N % NF == 0 && HAND_OVER >= K1, "");
  const HeadBlock hb(w.b, w.n, w.group, own_blocks(w.s, OWNED), place);
  if (hb.none) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // a scalar
  const Head<EXACT, D> at(w, hb.batch, hb.head);
  const int s = at.s, d = at.d, lane = at.lane, g = lane >> 4, lr = lane & 15, h = lane >> 5;
  const int rows_of = (threadIdx.x >> 6) & (L::GROUPS - 1);   // (from the thread number: see the forward kernel)
  const int block0 = hb.order * OWNED, own0 = block0 + rows_of * 32, mine = own0 + (lane & 31);
  const int part = L::PARTS == 2 ? wave >> 1 & 1 : 0, role = wave >> 2;
  const float f = EXACT ? w.scale : w.scale * kLog2e;
  typename T::Lane32 ln(lane);
  const uint32_t smem_addr = lds_address(smem);
  const int ntiles = (s + ROWS - 1) / ROWS - block0 / ROWS;
  // Tiles whose rows, those that this pair takes, none of its keys is seen by: the first ones, passed over (as in the forward kernel).
  const int before_own = ((wave & (L::GROUPS - 1)) - part + ROWS / 32 - 1) / (ROWS / 32), hidden = before_own < ntiles ? before_own : ntiles;

  // Tiles of 64 rows: waves 0-3 bring the Q tile, waves 4-7 the dO tile, 16 rows each; of 32 rows: waves 0, 1 and waves 2, 3.  Every wave that brings any brings the
  // tile's lse values (even waves) or -D values (odd waves) too; those arrive several times over, so that every wave issues the same number of memory
  // operations (or none), which the counted waits rely on.  The own rows come the same way, first: four waves need each of them, and memory requests of
  // the first microseconds are answered slowly (as fragments straight to registers, four times over, they and the first tiles took 10000 cycles; 3200 so).
  constexpr int IPW = T::NI, OPS = IPW + 1;
  const bool brings = ROWS == 64 || wave < 4;
  {
    const int second = wave >> 2;
    TileStream own = at.matrix(false, second, block0, 64);
#pragma unroll
    for (int t = 0; t < OWNED / 64; ++t) {
#pragma unroll
      for (int i = 0; i < IPW; ++i)
        dma16<Burst::value>(own.rsrc(), smem_addr + L::OWN + (2 * t + second) * T::BYTES + ((wave & 3) * IPW + i) * 1024,
                            T::dma_offset(at.pitch_bytes(false, second), wave & 3, lane, i, d));
      own.advance();
    }
  }
  const int half = ROWS == 64 ? wave >> 2 : wave >> 1 & 1, quarter = ROWS == 64 ? wave & 3 : wave & 1;
  TileStream stream = at.matrix(true, half, block0, ROWS);
  TileStream stats(((wave & 1) && !OWN_D ? at.Dvec : at.lse) + block0, (s - block0) * 4, ROWS * 4);
  uint32_t dma_off[IPW];
#pragma unroll
  for (int i = 0; i < IPW; ++i) dma_off[i] = T::dma_offset(at.pitch_bytes(true, half), quarter, lane, i, d);
  auto issue_one = [&](auto tag, int st, int i) {   // i == IPW: the statistics (with tiles of 32 rows those of the next tile as well, unused)
    constexpr int TAG = decltype(tag)::value;
    const uint32_t stage = smem_addr + st * STAGE;
    if (i == IPW) dma4<TAG>(stats.rsrc(), stage + 2 * L::MATRIX + (wave & 1) * 256, lane * 4);
    else dma16<TAG>(stream.rsrc(), stage + half * L::MATRIX + (quarter * IPW + i) * 1024, dma_off[i < IPW ? i : 0]);
  };
  auto advance = [&] {
    stream.advance();
    stats.advance();
  };
  auto issue_tile = [&](int st) {
    if (brings) {
#pragma unroll
      for (int i = 0; i < OPS; ++i) issue_one(Burst{}, st, i);
    }
    advance();
  };
  constexpr int ISSUE_STEPS = AHEAD == 1 ? (OPS + 1) / 2 : N - PF;   // (one tile ahead: it is waited for in the same iteration)
  auto issue_step = [&](int step, int st) {
    if (!brings) return;
#pragma unroll
    for (int i = 0; i < OPS; ++i)
      if (i >= (step ? dma_by<OPS, ISSUE_STEPS>(step - 1) : 0) && i < dma_by<OPS, ISSUE_STEPS>(step)) issue_one(Spread{}, st, i);
  };
#pragma unroll
  for (int t = 0; t < L::FIRST; ++t) issue_tile(t);
  if (!brings) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  wait_and_barrier<L::FIRST * OPS>();   // the own rows landed everywhere
  bf16x8 of[K1];   // own rows of K (role 0) or V
#pragma unroll
  for (int kk = 0; kk < K1; ++kk) of[kk] = T::nat32(smem + L::OWN + 2 * (rows_of >> 1) * T::BYTES + role * T::BYTES + (rows_of & 1) * T::ROWS32, ln, kk);
  float *const rows_d = reinterpret_cast<float *>(smem + L::BYTES);   // OWN_D: -D of the rows from the first tile on
  if constexpr (OWN_D) {
    constexpr int AT_ONCE = 2;   // rows of a thread: one at a time, every row is a trip to memory
    for (int row = (threadIdx.x >> 2); row < ntiles * ROWS; row += AT_ONCE * DKV_THREADS / 4) {   // four lanes to a row
      float t[AT_ONCE];
#pragma unroll
      for (int q = 0; q < AT_ONCE; ++q) {
        const int r = block0 + row + q * (DKV_THREADS / 4);
        const int64_t from = (int64_t)(r < s ? r : s - 1) * at.pld + (threadIdx.x & 3) * 8;
        t[q] = 0.0f;
#pragma unroll
        for (int kk = 0; kk < D / 32; ++kk) {
          const bf16x8 x = *reinterpret_cast<const bf16x8 *>(at.dab + from + 32 * kk), y = *reinterpret_cast<const bf16x8 *>(at.ab + from + 32 * kk);
#pragma unroll
          for (int e = 0; e < 8; ++e) t[q] += (float)x[e] * (float)y[e];
        }
      }
#pragma unroll
      for (int q = 0; q < AT_ONCE; ++q) {
        t[q] += __shfl_xor(t[q], 1, 64);
        t[q] += __shfl_xor(t[q], 2, 64);
        const int r = row + q * (DKV_THREADS / 4);
        if ((threadIdx.x & 3) == 0 && r < ntiles * ROWS) rows_d[r] = -t[q];
      }
    }
  }
#pragma unroll
  for (int kk = 0; kk < K1; ++kk) arrive(of[kk]);
  f32x16 acc[CB];   // dv (role 0) or dk (role 1)
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) acc[cb] = f32x16{};
  if constexpr (L::FIRST < AHEAD) {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // the own rows have been read
#pragma unroll
    for (int t = L::FIRST; t < AHEAD; ++t) issue_tile(t);
  }
  wait_and_barrier<(AHEAD - 1) * OPS>();   // tile 0 landed everywhere

  // the loop, once for each role
  const char *now = smem, *before = smem;   // stages of the tile whose first product, and whose second, are next to be read
  f32x4 *const xchg = reinterpret_cast<f32x4 *>(smem + RING * STAGE) + (wave & 3) * 256 + lane;   // 4 x 64 of the pair
  int cur = 0, odd = 0;
  auto next_of = [](int cur) { return cur == RING - 1 ? 0 : cur + 1; };   // stages of tiles it + 1
  auto ahead_of = [&](int cur) { return AHEAD == 1 ? next_of(cur) : cur + AHEAD >= RING ? cur + AHEAD - RING : cur + AHEAD; };   // and it + AHEAD
  for (int it = 0; it < hidden; ++it) {   // its share of a later tile, and the barriers
    if constexpr (!LAG) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    issue_tile(ahead_of(cur));
    wait_and_barrier<(AHEAD - 1) * OPS>();
    cur = next_of(cur);
    odd ^= 1;
  }
  now = before = smem + cur * STAGE;   // (LAG: the first second product, of zeros, is with rows that the pair takes)
  auto run = [&](auto ROLE) __attribute__((always_inline)) {
    constexpr int me = decltype(ROLE)::value;
    const int part_rows = part * T::ROWS32;
    constexpr int FIRST_AT = me ? L::MATRIX : 0, SECOND_AT = me ? 0 : L::MATRIX;   // S from Q, then dv from dO; dP from dO, then dk from Q
    bf16x8 fr[NF];
    f32x16 sc, prev = {};   // S and P (role 0); dP - D (EXACT: dP) of this tile and of the one before
    Parts<NP> x[2], xn[2];  // the second product's operand: what is in use, and (role 0) the next
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < NP; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) x[t].p[i][e] = (bf16)0.0f;
    auto load = [&](int r) {   // the fragment of step r
      if (r < K1) fr[r % NF] = T::nat32(now + FIRST_AT + part_rows, ln, r);
      else fr[r % NF] = T::tr32((LAG ? before : now) + SECOND_AT + part_rows, ln, (r - K1) / 2, r % 2);
    };
    auto take = [&](int buffer, f32x16 &p) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 v = xchg[buffer * (L::XCHG / 16) + q * 64];
#pragma unroll
        for (int e = 0; e < 4; ++e) p[4 * q + e] = v[e];
      }
    };
    // LAG: the first tile has none before it.  Its products are with zeros, P among them: LDS holds what was there before
    if constexpr (LAG && me == 1) {
#pragma unroll
      for (int q = 0; q < 4; ++q) xchg[(odd ^ 1) * (L::XCHG / 16) + q * 64] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
    f32x16 dn_all;   // EXACT: D of this tile's rows, and of the one before
    f32x16 dn_prev = {};
    auto gradient = [&](float p, float dp, float dd) { return (EXACT ? dp - dd : dp) * p; };
#pragma unroll
    for (int i = 0; i < PF; ++i) load(i);
    __builtin_amdgcn_sched_barrier(0);
    for (int it = hidden; it < ntiles; ++it) {
      ln.here();
      const int next = next_of(cur), nn = ahead_of(cur);
      const float *stat = reinterpret_cast<const float *>(smem + cur * STAGE + 2 * L::MATRIX) + 32 * part + 4 * h;
      const float *dneg = OWN_D ? rows_d + it * ROWS + 32 * part + 4 * h : stat + 64;
      const int row = block0 + it * ROWS + 32 * part;   // element e: row + 8 (e / 4) + 4 h + e % 4
      f32x16 ls, p;
      if constexpr (me == 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x4 v = *reinterpret_cast<const f32x4 *>(stat + 8 * q);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            ls[4 * q + e] = v[e];
            sc[4 * q + e] = 0.0f;
          }
        }
      } else {
        if (LAG) take(odd ^ 1, p);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x4 v = *reinterpret_cast<const f32x4 *>(dneg + 8 * q);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            dn_all[4 * q + e] = v[e];
            sc[4 * q + e] = EXACT ? 0.0f : v[e];
          }
        }
      }
      auto step = [&](auto I) __attribute__((always_inline)) {
        constexpr int r = decltype(I)::value;
        if constexpr (me == 0) {
          if (r == K1 && (row < own0 + 31 || row + 31 >= s)) {   // wave-uniform: diagonal or past-the-end queries
#pragma unroll
            for (int e = 0; e < 16; ++e) {
              const int q = row + 8 * (e / 4) + 4 * h + e % 4;
              if (q < mine || q >= s) sc[e] = -INFINITY;
            }
          }
#pragma unroll
          for (int e = 0; e < 16; ++e)
            if (r == K1 + e * (HAND_OVER - K1) / 16) sc[e] = weight<EXACT>(sc[e], f, EXACT ? ls[e] : ls[e] * kLog2e);
          if (r == HAND_OVER) {
#pragma unroll
            for (int t = 0; t < 2; ++t) xn[t] = weights16<EXACT>(sc, t);
#pragma unroll
            for (int q = 0; q < 4; ++q) xchg[(LAG ? odd : 0) * (L::XCHG / 16) + q * 64] = quarter_of(sc, q);
            if constexpr (!LAG) {
              asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
              x[0] = xn[0];
              x[1] = xn[1];
            }
          }
        } else {
          // dS of the tile before (LAG: over its first product's steps) or of this one
          if (!LAG && r == K1) {
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            take(0, p);
          }
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            if (LAG && r == 2 + e * (K1 - 2) / 16) prev[e] = gradient(p[e], prev[e], dn_prev[e]);
            if (!LAG && r == K1) prev[e] = gradient(p[e], sc[e], dn_all[e]);
          }
          if (r == K1)
#pragma unroll
            for (int t = 0; t < 2; ++t) x[t] = weights16<EXACT>(prev, t);
        }
        if (r == N - PF) {   // all that this iteration reads has been read, and all it hands over is written; tile it + 1 landed everywhere
          wait_and_barrier<(AHEAD - 1) * OPS>();
          before = now;
          now = smem + next * STAGE;
        }
        load((r + PF) % N);
        if (r < ISSUE_STEPS) issue_step(r, nn);
        const bf16x8 &v = fr[r % NF];
        if constexpr (r < K1) sc = MFMA32(v, of[r], sc);
        else acc[(r - K1) / 2] = mma_weights32(v, x[r % 2], acc[(r - K1) / 2]);
        __builtin_amdgcn_sched_barrier(0);
      };
      for_each_step(step, std::make_integer_sequence<int, N>{});
      if constexpr (LAG) {
        if constexpr (me == 0) {
          x[0] = xn[0];
          x[1] = xn[1];
        } else {
          prev = sc;
          if constexpr (EXACT) dn_prev = dn_all;
        }
      }
      advance();
      cur = next;
      odd ^= 1;
    }
    if (!LAG || hidden == ntiles) return;
    // the second product of the last tile
    if constexpr (me == 1) {
      f32x16 p;
      take(odd ^ 1, p);
#pragma unroll
      for (int e = 0; e < 16; ++e) prev[e] = gradient(p[e], prev[e], dn_prev[e]);
#pragma unroll
      for (int t = 0; t < 2; ++t) x[t] = weights16<EXACT>(prev, t);
    }
    bf16x8 v[4];
    pipelined<K1, 3>([&](int i) { v[i & 3] = T::tr32(before + SECOND_AT + part_rows, ln, i / 2, i % 2); },
                     [&](int i) { acc[i / 2] = mma_weights32(v[i & 3], x[i % 2], acc[i / 2]); }, [](int) {});
  };
  if (role == 0) run(std::integral_constant<int, 0>{});
  else run(std::integral_constant<int, 1>{});
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");   // the look-ahead tiles, which nobody uses

  float z = 0.0f;   // EXACT: NaN where a result is not finite
  bf16 *const head = at.out + (int64_t)mine * at.ld, *const out = head + (role ? d : 2 * d);
  const float mul = role ? w.scale : 1.0f;
  auto put = [&](int cb, int q, f32x4 sum) {   // columns 32 cb + 8 q + 4 h .. + 3
    const int col = 32 * cb + 8 * q + 4 * h;
    if (EXACT && col >= d) return;
    bf16x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float r = (EXACT ? sum[e] * PARTS_UNSCALE : sum[e]) * mul;
      if constexpr (EXACT) z = fmaf(r, 0.0f, z);
      o[e] = (bf16)r;
    }
    *reinterpret_cast<bf16x4 *>(out + col) = o;
  };
  // Two parts: of the two waves with the same rows and role each hands over half of its columns and finishes the other half
  f32x4 *slots = reinterpret_cast<f32x4 *>(smem) + lane;
  if constexpr (L::PARTS == 2) {
    __syncthreads();   // the rings are no longer read
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int q = 0; q < 2; ++q) slots[((wave * CB + cb) * 2 + q) * 64] = part ? quarter_of(acc[cb], q) : quarter_of(acc[cb], 2 + q);
    __syncthreads();
  }
  if (mine < s) {
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      if constexpr (L::PARTS == 2) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const f32x4 other = slots[(((wave ^ 2) * CB + cb) * 2 + q) * 64];
          if (part) put(cb, 2 + q, quarter_of(acc[cb], 2 + q) + other);
          else put(cb, q, quarter_of(acc[cb], q) + other);
        }
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) put(cb, q, quarter_of(acc[cb], q));
      }
    }
  }
  if constexpr (EXACT) {
    if constexpr (L::PARTS == 2) z = either_part(z, smem, wave, wave ^ 2, part, lane);
    if (!all_finite(z)) {
      auto d_of = [&](int t) { return at.Dvec[t]; };
#pragma unroll 1
      for (int c = 0; c < 2; ++c) {
        const int first = own0 + 16 * c, key = first + lr;
        bf16 *const o = at.out + (int64_t)key * at.ld;
        if (role) redo_dk<bf16, D>(at.base, at.ld, at.dab, at.pld, s, d, w.scale, first, key, at.lse, d_of, g, o);
        else redo_dv<bf16, D>(at.base, at.ld, at.dab, at.pld, s, d, w.scale, first, key, at.lse, g, o);
      }
    }
  }
}

template <int D, int SPLIT, bool EXACT>
__global__ __launch_bounds__(DQ_THREADS, dq_ring(D, EXACT) == 2 ? 2 : 1) void attn_bwd_dq_kernel(BackwardArgs w) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  dq_block<D, SPLIT, EXACT>(blockIdx.x, smem, w);
}
// How dk / dv are shared out: own rows of a workgroup and rows of a tile
constexpr int dkv_owned(int split) { return split == 1 ? 128 : 64; }
constexpr int dkv_rows(int split) { return split == 1 ? 32 : 64; }
template <int D, int SPLIT, bool EXACT>
__global__ __launch_bounds__(DKV_THREADS) void attn_bwd_dkv_kernel(BackwardArgs w) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  dkv_block<D, dkv_owned(SPLIT), dkv_rows(SPLIT), EXACT, false>(blockIdx.x, smem, w);
}
// Both in one launch (bwd_one_launch says when): the first half of a grid row's workgroups (dk / dv, the longer ones) compute D for themselves.
template <int D>
__global__ __launch_bounds__(DKV_THREADS) void attn_bwd_kernel(BackwardArgs w) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const unsigned half = gridDim.x / 2;
  if (blockIdx.x < half) dkv_block<D, 64, 64, false, true>(blockIdx.x, smem, w);
  else if (threadIdx.x < DQ_THREADS) dq_block<D, 2, false>(blockIdx.x - half, smem, w);
}

template <int D, int SPLIT, bool EXACT = false>
int bwd_launch_p(int b, int s, int n, int d, float scale, const void *qkv, const void *a, const float *lse, const void *da,
                 void *dqkv, void *ws, hipStream_t st) {
  constexpr int smem_dq = dq_ring(D, EXACT) * 2 * Tile<D>::BYTES, smem_dkv = DkvLds<D, dkv_owned(SPLIT), dkv_rows(SPLIT), EXACT, false>::BYTES;
  static unsigned long long attr_done = 0;
  int device;
  if (!attr_is_set(attr_done, &device)) {
    MTNLG_TRY(set_lds(attn_bwd_dq_kernel<D, SPLIT, EXACT>, smem_dq));
    MTNLG_TRY(set_lds(attn_bwd_dkv_kernel<D, SPLIT, EXACT>, smem_dkv));
    attr_mark_set(attr_done, device);
  }
  float *Dvec = (float *)ws;
  const int count = own_blocks(s, SPLIT == 2 ? 64 : 128), group = HeadBlock::group(b, n, count, SPLIT == 1 || D >= 128 ? 32 : 128, SPLIT == 1 ? 511 : 2047);
  const dim3 grid = HeadBlock::grid(b, n, group, count);
  LaunchScope scope(MTNLG_K_ATTN_BWD, st);
  const BackwardArgs w{b, s, n, d, group, scale, (const bf16 *)qkv, (const bf16 *)a, lse, (const bf16 *)da, (bf16 *)dqkv, Dvec};
  attn_bwd_dq_kernel<D, SPLIT, EXACT><<<grid, DQ_THREADS, smem_dq, st>>>(w);
  MTNLG_TRY(check_launch());
  attn_bwd_dkv_kernel<D, SPLIT, EXACT><<<grid, DKV_THREADS, smem_dkv, st>>>(w);
  return check_launch();
}

template <int D>
int bwd_launch_one(int b, int s, int n, float scale, const void *qkv, const void *a, const float *lse, const void *da, void *dqkv, void *ws,
                   hipStream_t st) {
  const int count = row_blocks(s), group = HeadBlock::group(b, n, count, 32, 2047);
  constexpr int rings = DkvLds<D, 64, 64, false, true>::BYTES;
  const int with_d = rings + count * 64 * (int)sizeof(float), dq = dq_ring(D, false) * 2 * Tile<D>::BYTES, smem = with_d > dq ? with_d : dq;
  static unsigned long long attr_done = 0;
  int device;
  if (!attr_is_set(attr_done, &device)) {
    MTNLG_TRY(set_lds(attn_bwd_kernel<D>, rings + ONE_LAUNCH_ROWS * (int)sizeof(float)));
    attr_mark_set(attr_done, device);
  }
  dim3 grid = HeadBlock::grid(b, n, group, count);
  grid.x *= 2;
  LaunchScope scope(MTNLG_K_ATTN_BWD, st);
  attn_bwd_kernel<D><<<grid, DKV_THREADS, smem, st>>>(
      BackwardArgs{b, s, n, D, group, scale, (const bf16 *)qkv, (const bf16 *)a, lse, (const bf16 *)da, (bf16 *)dqkv, (float *)ws});
  return check_launch();
}

// By blocks of 64 rows of all heads together.  One launch where (nearly) all workgroups of either kernel run at once, so that both kernels' would leave units idle
// one after the other: a second D for every tile costs less than that and the launch.  us, two launches / one, head size 128: 2 heads, s = 256 (8
// blocks) 17.1 / 10.5; 16, 1024 (256) 38.9 / 32.9; 75, 256 (300) 27.4 / 26.4; 40, 512 (320) 29.2 / 28.1; 20, 1024 (320) 40.4 / 41.7; 24, 1024 (384) 45.7 / 51.6; at 160 the same.  Over 27 sizes of
// 257 to 320 blocks one is 0.96 to 1.21 times as fast, 1.05 on average (s 65 to 96 from 297 blocks on 0.94 to 0.99, against 128 rows), over 25 of 321 to 384 0.81 to 1.18, 0.97.
// Workgroups of 128 rows where there are enough of them to even out: half of what a workgroup costs besides its tiles, and of the tiles' way into LDS.
// us, 64 / 128 rows, head size 128, then 160: 20 heads, s = 2048 (640 blocks) 102 / 115, 118 / 129; 80, 512 (640) 49.2 / 49.6, 61.1 / 58.8; 24, 2048 (768) 114 / 116, 136 / 134; 48,
// 1024 (768) 74.2 / 72.9, 91.5 / 86.1; 200, 256 (800) 52.7 / 48.1, 67.0 / 58.8; 28, 2048 (896) 133 / 129, 162 / 151; 64, 2048 (2048) 291 / 275, 358 / 321; 512, 768 542 / 466, 634 / 541.
// Shorter sequences (1600 sizes, times as fast with 128 rows): s 65 to 128, one round of 128 rows (257 to 512 blocks) 1.0 to 1.24 (80 x 200 heads of 128 21.4 / 18.8), 513 to 767 0.93 to 1.02; s 129 to
// 512, 513 blocks and more 0.98 to 1.18, to 1024, 577 and more 0.99 to 1.27; s 33 to 64, of whose 128 rows half are empty, 0.92 to 1.0; scattered heads (s 129 to 384, at head size 128 from 385 blocks on) 1.0 to 1.17.
template <int D>
int bwd_launch(int b, int s, int n, float scale, const void *qkv, const void *a, const float *lse, const void *da,
               void *dqkv, void *ws, hipStream_t st) {
  const int64_t blocks = (int64_t)b * n * row_blocks(s);
  const bool two_blocks = s > 64 && s <= 128;
  if (s <= ONE_LAUNCH_ROWS && blocks <= (two_blocks && s <= 96 ? 296 : 320)) return bwd_launch_one<D>(b, s, n, scale, qkv, a, lse, da, dqkv, ws, st);
  bool rows128 = blocks >= 768 && (s <= 32 || s > 64);
  if (two_blocks) rows128 = blocks <= 512 || blocks >= 768;
  else if (s > 128 && s <= 1024) rows128 = blocks > (s <= 512 ? 512 : 576) || (s <= 384 && blocks > (D == 128 ? 384 : 320) && heads_scattered(b, n, s, D));
  if (rows128) return bwd_launch_p<D, 1>(b, s, n, D, scale, qkv, a, lse, da, dqkv, ws, st);
  return bwd_launch_p<D, 2>(b, s, n, D, scale, qkv, a, lse, da, dqkv, ws, st);
}

// EXACT: 128 own rows to a workgroup from 2048 blocks of 64 rows on, and for shorter sequences before.  us, 64 / 128 rows: of 96 64 heads, s = 1024 (1024) 109 / 123, 64, 2048 (2048) 359 / 350, 512, 512
// 309 / 270; of 144 48, 2048 (1536) 411 / 401, 96, 1024 (1536) 249 / 257, 64, 2048 (2048) 561 / 526; of 104 1024, 256 279 / 265.  s 65 to 128, more than 256 blocks: 128 rows 1.05 to 1.4 times as
// fast; s 129 to 512, more than 768: 1.0 to 1.25.
template <int D>
int exact_launch(int b, int s, int n, int d, float scale, const void *qkv, const void *a, const float *lse, const void *da, void *dqkv, void *ws,
                 hipStream_t st) {
  const int64_t blocks = (int64_t)b * n * row_blocks(s);
  if (s > 64 && blocks > (s <= 128 ? 256 : s <= 512 ? 768 : 2047)) return bwd_launch_p<D, 1, true>(b, s, n, d, scale, qkv, a, lse, da, dqkv, ws, st);
  return bwd_launch_p<D, 2, true>(b, s, n, d, scale, qkv, a, lse, da, dqkv, ws, st);
}

}  // namespace

int attention_bwd_mfma(int b, int s, int n, int d, float scale, const void *qkv, const void *a, const float *lse,
                       const void *da, void *dqkv, void *ws, hipStream_t stream) {
  if (n > 65535 || b > 65535 || !fits(s, n, d)) return MTNLG_UNSUPPORTED_SHAPE;
  switch (d) {
    case 64: return attention_bwd64(b, s, n, scale, qkv, a, lse, da, dqkv, ws, stream);
    case 128: return bwd_launch<128>(b, s, n, scale, qkv, a, lse, da, dqkv, ws, stream);
    case 160: return bwd_launch<160>(b, s, n, scale, qkv, a, lse, da, dqkv, ws, stream);
    default: return MTNLG_UNSUPPORTED_SHAPE;
  }
}

int attention_bwd_exact(int b, int s, int n, int d, float scale, const void *qkv, const void *a, const float *lse, const void *da,
                        void *dqkv, void *ws, hipStream_t stream) {
  // 16 rows to a wave (attention_bwd64.hip) up to head size 32, to 64 but for few blocks of long sequences, and for short sequences of the others: there the chain of these kernels' prologue, exchange
  // and merge is most of the time.  Times as fast as these (2300 sizes): 33 to 64, s up to 128 1.1 to 1.45, 385 to 768 1.0 to 1.05 (more than 512 blocks 1.1 to 1.25), beyond 0.95 to 1.0 (1.1 to
  // 1.2); 65 to 96, s up to 64 1.06 to 1.25, 129 to 192 1.05 to 1.1, 193 to 384 1.02 to 1.1, 385 and more 0.93 to 1.0; 97 to 128, s up to 64 1.05 to 1.1 up to 256 blocks, else 0.96 to 1.0; 129 to
  // 160, s up to 64 1.03 to 1.16; 161 to 192, s up to 96 1.02 to 1.13 beyond 384 blocks.  us: 2 x 87 tokens x 169 heads of 48 22.6 / 27.6, 80 x 774 of 144 114 / 124.
  const int64_t blocks = (int64_t)b * n * row_blocks(s);
  bool rows16;
  if (d <= 32) rows16 = true;
  else if (d <= 64) rows16 = s <= 768 || blocks > 512;
  else if (d <= 96) rows16 = s <= 64 || (s <= 96 ? blocks <= 256 : s <= 192 || (s <= 384 && blocks <= 768));
  else if (d <= 128) rows16 = s <= 64 && blocks <= 256;
  else if (d <= 160) rows16 = s <= 64;
  else rows16 = s <= 96 && blocks > 384;
  if (rows16) return attention_bwd_exact64(b, s, n, d, scale, qkv, a, lse, da, dqkv, ws, stream);
  if (d <= 64) return bwd_launch_p<64, 2, true>(b, s, n, d, scale, qkv, a, lse, da, dqkv, ws, stream);
  if (d <= 96) return exact_launch<96>(b, s, n, d, scale, qkv, a, lse, da, dqkv, ws, stream);
  if (d <= 128) return exact_launch<128>(b, s, n, d, scale, qkv, a, lse, da, dqkv, ws, stream);
  if (d <= 160) return exact_launch<160>(b, s, n, d, scale, qkv, a, lse, da, dqkv, ws, stream);
  return bwd_launch_p<192, 2, true>(b, s, n, d, scale, qkv, a, lse, da, dqkv, ws, stream);
}

}  // namespace mtnlg
