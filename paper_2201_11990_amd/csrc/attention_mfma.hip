// Fused causal softmax attention on the gfx950 matrix cores (bf16 in, fp32 softmax
// and accumulation), forward and backward, for head sizes 64, 128 and 160; and with P and dS in fp32 (EXACT) for the others up to 192.
//
//   S = scale * q k^T (causal),  P = rowsoftmax(S),  a = P v,  lse = log sum exp(S)
//   backward with D_t = da_t . a_t :  dP = da v^T,  dS = P o (dP - D),
//   dq = scale dS k,  dk = scale dS^T q,  dv = P^T da.
//
// Three kernels of eight waves.  A workgroup owns rows of one side (forward: 128 or 256 queries, 16 or 32 per wave;
// dq and dk/dv: 64 queries or keys, 16 per wave, each half of the workgroup on one half of every tile, or 128 with a block
// to each half), held in registers as MFMA B operands (groups of 16, one row per lane column); the other side streams through
// LDS in tiles of 64 rows, brought in by LDS DMA (buffer_load ... lds, no staging
// registers) three tiles deep, one workgroup barrier per tile.  What bounds them: no single unit.  Between two barriers a
// wave runs LDS reads, MFMAs, the softmax and the DMA issue in one chain, and the waves of a workgroup run it in step, so
// the times of the four add up; taking any one out shortened a tile by no more than that one's own time.
//
// All products are v_mfma_f32_16x16x32_bf16 with the streamed tile as the A operand, so a
// product block comes out as C[tile row 4 (lane/16) + i][own row lane%16], i = 0..3:
//   forward : S^T = K Q^T; the softmax statistics of a query live in the four lanes that
//             share lane%16; P^T packed to bf16 is directly the B operand of O^T += V^T P^T.
//   dq      : S^T and dP^T = V dO^T the same way, dQ^T += K^T dS^T.
//   dk / dv : S = Q K^T, dP = dO V^T with the key on the lane column,
//             dV^T += dO^T P, dK^T += Q^T dS.
// The second product of each chain contracts over the tile's rows.  Its A operand is read
// from the same natural [row][D] tile with the transposing LDS read (ds_read_b64_tr_b16: a
// 16-lane group reads 4 tile rows x 16 columns, each lane receives the 4 row values of its
// column); the k slots of that MFMA are ordered to match the accumulator layout of the
// first product (slot (g, e) of a 32-row step = tile row 4g + e for e < 4, 16 + 4g + e - 4
// otherwise), so P and dS never leave the registers and nothing is transposed in software.
// No atomics: every output element has one owner, results are run-to-run identical.
//
// EXACT: any head size d that is a multiple of 8, in tiles of D = d rounded up to 32 columns (the DMA brings zeros past d).  P and dS are
// not rounded to bf16: each goes into the second product as three bf16 parts that add up to it (common.h: Parts; scaled, so of any size), three MFMAs
// where the other kernels have one; 17 against 9 a tile in all, but the chain between barriers stays the bound.  2 x 1024 tokens, 16 heads of
// 96, forward / backward: 103 / 327 us on the fp32 instructions without LDS (attention_f32.hip), 24 / 61 here.  Inputs that are not finite
// take the slow path of attention_redo.h.
#include <math.h>

#include "attention_redo.h"
#include "common.h"

namespace mtnlg {

namespace {

typedef __attribute__((ext_vector_type(8))) short i16x8;
typedef __attribute__((ext_vector_type(4))) short i16x4;
typedef __attribute__((address_space(3))) i16x4 *lds_i16x4_ptr;

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

#define MFMA16(a, b, c) __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0)

// 2^x on the transcendental unit (v_exp_f32): no denormal fix-up, 2^-inf = 0.
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
// e^x down to the least weight that fp32 has.  The instruction takes results below 2^-126 for 0, so it is given half the exponent: one
// multiplication more (2 x 1024 x 16 heads of 96, forward and backward: 81.4 us without, 82.1 so; 83.8 with a branch for such weights).
__device__ __forceinline__ float exact_exp(float x) {
  const float half = fast_exp2(x * (0.5f * kLog2e));
  return half * half;
}
// e^(s f - shift).  EXACT: f is the scale, whose rounding after a multiplication by log2 e would move every exponent the same way; else
// f and shift have the factor log2 e.
template <bool EXACT>
__device__ __forceinline__ float weight(float s, float f, float shift) {
  const float x = fmaf(s, f, -shift);
  return EXACT ? exact_exp(x) : fast_exp2(x);
}
// m + log(l), rounded about once, with log 2 in two parts (Cody and Waite): the reference maximum may lie up to 2^8 below the largest weight, and log(l) of such a sum is large
// enough for its own rounding to show (2048 keys, 4 heads of 96: log-sum-exp 3.4e-7 off, rms, with m + logf(l), 1.8e-7 so; 3.0e-7 with a maximum that always follows).
__device__ __forceinline__ float plus_log(float m, float l) {
  int k;
  const float f = frexpf(l, &k), t = k * 0x1.62e4p-1f;   // log l = k log 2 + log f, log 2 = 0x1.62e4p-1 + 1.4286068e-6; t is exact
  const float sum = m + t, b = sum - m, rest = (m - (sum - b)) + (t - b);
  return sum + (rest + fmaf((float)k, 1.4286068e-6f, logf(f)));
}
// rounded to fp32, never fused into an addition
__device__ __forceinline__ float product_of(float x, float y) {
  float p = x * y;
  asm("" : "+v"(p));
  return p;
}

// A 64-row x D-column bf16 tile in LDS, rows as in memory, the 16-byte units of a row
// permuted by an XOR that depends on the row.  The masks are the ones a micro-benchmark of the
// two fragment read patterns found fastest (cycles per wave instruction, two waves per SIMD):
// head size 160: 4.5-4.9 for the 16-byte reads and 3.0 for the transposing reads (no conflicts; so 32 and 96, whose rows are an odd
// number of 64-byte pieces too, and 192 as 64);
// 64: the same; 128: 4.5 and 4.0 (no mask of this form is conflict-free for both at a row of
// exactly 256 bytes).  The masks look at the low four bits of the row only.
template <int D>
struct Tile {
  static constexpr bool ODD = D / 32 % 2 == 1;   // 32, 96, 160
  static constexpr int UPR = D / 8;        // 16-byte units per row
  static constexpr int BYTES = 64 * D * 2;
  static constexpr int NI = D / 32;        // DMA instructions per wave and tile (16 rows)
  static __device__ __forceinline__ int mask(int row) {
    if constexpr (ODD) return (row >> 1) & 3;
    else if constexpr (D == 128) return row & 15;
    else return row & 7;
  }
  static __device__ __forceinline__ int off(int row, int u) { return (row * UPR + (u ^ mask(row))) * 16; }

  // Byte offset, from the tile's first row in memory (row pitch ld_bytes), of what lane `lane` moves in DMA instruction i of
  // the wave that brings rows 16 quarter .. + 15: instruction i fills 1024 consecutive LDS bytes, lane l the 16 at 16 l.
  // (units past column d: outside any descriptor, they arrive as zeros)
  static __device__ __forceinline__ uint32_t dma_offset(uint32_t ld_bytes, int quarter, int lane, int i, int d) {
    const int p = i * 64 + lane, r = 16 * quarter + p / UPR, u = (p % UPR) ^ mask(r);
    return u * 8 < d ? r * ld_bytes + u * 16 : 0xFFFFFFF0u;
  }
  // Byte offsets of a lane's fragment reads inside a tile.  mask() looks at the low four bits of a
  // row only, so a block of 16 rows further down is a constant distance away; and the offsets of the k-steps and
  // column blocks differ by an XOR of bits that the row part leaves empty (ODD, whose mask touches the low two
  // bits of a unit only: by a constant, and one bit for odd column blocks; 192, the low three: one or two bits and a constant).  One register each instead of one per step.
  struct Lane {
    uint32_t n0;   // row lane%16, 16-byte unit lane/16
    uint32_t t0;   // as address supplier of a transposing read: row 4 (lane/16) + L/4, columns 4 (L%4) .. + 3, L = lane%16
    __device__ __forceinline__ explicit Lane(int lane) {
      const int g = lane >> 4, L = lane & 15, col = 4 * (L & 3);
      n0 = (uint32_t)off(L, g);
      t0 = (uint32_t)(off(4 * g + (L >> 2), col >> 3) + (col & 7) * 2);
    }
    // once per tile: keeps the compiler from holding every offset in a register of its own across tiles
    __device__ __forceinline__ void here() { asm volatile("" : "+v"(n0), "+v"(t0)); }
    __device__ __forceinline__ uint32_t nat(int kk) const {
      if constexpr (ODD) return n0 + kk * 64;
      else if constexpr (D == 192) return (n0 ^ ((kk & 1) * 64)) + (kk >> 1) * 128;
      else return n0 ^ (kk * 64);
    }
    __device__ __forceinline__ uint32_t tr(int cblk) const {
      if constexpr (ODD) return (t0 ^ ((cblk & 1) * 32)) + (cblk >> 1) * 64;
      else if constexpr (D == 192) return (t0 ^ ((cblk & 3) * 32)) + (cblk >> 2) * 128;
      else return t0 ^ (cblk * 32);
    }
  };
  static constexpr int ROWS16 = 16 * UPR * 16;   // bytes of 16 tile rows
  // A operand contracting over columns: lane l holds row 16 blk + l%16, columns 32 kk + 8 (l/16) .. + 7
  static __device__ __forceinline__ bf16x8 nat(const char *t, const Lane &ln, int blk, int kk) {
    return *reinterpret_cast<const bf16x8 *>(t + ln.nat(kk) + blk * ROWS16);
  }
  // A operand contracting over tile rows 32 ks .. 32 ks + 31: lane l holds column 16 cblk + l%16 and,
  // with g = l/16, tile rows 32 ks + 4 g .. + 3 (elements 0-3) and 32 ks + 16 + 4 g .. + 3 (4-7).
  static __device__ __forceinline__ bf16x8 tr(const char *t, const Lane &ln, int cblk, int ks) {
    const char *p = t + ln.tr(cblk) + 2 * ks * ROWS16;
    const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_ptr)p);
    const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_ptr)(p + ROWS16));
    const i16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
  }
};

// The stream of a matrix's 64-row tiles into LDS: the descriptor of the next tile to fetch.  Its base moves by a tile and
// its size shrinks by one in scalar registers; a lane's offsets never change, and rows past the end of the matrix lie
// outside the descriptor and arrive as zeros.  (Offsets computed per instruction took a multiplication and five more
// vector instructions each, on kernels bound by vector issue.)
struct TileStream {
  uint64_t base;
  int left;   // bytes from base to the end of the matrix
  int tile_bytes;
  __device__ __forceinline__ TileStream(const void *first, int64_t bytes, int64_t tile) {
    const uint64_t a = (uint64_t)first;
    base = ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(a >> 32)) << 32) | (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)a);
    left = __builtin_amdgcn_readfirstlane(bytes > 0 ? (int)bytes : 0);
    tile_bytes = __builtin_amdgcn_readfirstlane(tile < 0x7FFFFFFF ? (int)tile : 0x7FFFFFFF);   // a tile beyond that is the only one
  }
  __device__ __forceinline__ dma_rsrc_t rsrc() const { return dma_rsrc((const void *)base, (uint32_t)left); }
  __device__ __forceinline__ void advance() {
    base += (uint32_t)tile_bytes;
    left = left > tile_bytes ? left - tile_bytes : 0;
  }
};

// call-site tags of the DMA helpers
struct Burst { static constexpr int value = 0; };
struct Spread { static constexpr int value = 1; };

// two accumulator blocks (tile rows 32 ks + 4g + i and 32 ks + 16 + 4g + i) as the bf16 B operand
__device__ __forceinline__ bf16x8 pack2(const f32x4 &lo, const f32x4 &hi) {
  bf16x8 o;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    o[i] = (bf16)lo[i];
    o[4 + i] = (bf16)hi[i];
  }
  return o;
}

// the same with fp32 values kept: three parts
template <bool EXACT>
__device__ __forceinline__ Parts<EXACT ? 3 : 1> weights(const f32x4 &lo, const f32x4 &hi) {
  Parts<EXACT ? 3 : 1> w;
  if constexpr (EXACT) w.of({lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
  else w.p[0] = pack2(lo, hi);
  return w;
}
template <int N>
__device__ __forceinline__ f32x4 mma_weights(const bf16x8 &x, const Parts<N> &w, f32x4 acc) {
#pragma unroll
  for (int i = N - 1; i >= 0; --i) acc = MFMA16(x, w.p[i], acc);
  return acc;
}

// columns 32 kk + 8 g .. + 7 of a row
template <bool EXACT>
__device__ __forceinline__ bf16x8 row_chunk(const bf16 *row, int col, int d) {
  if constexpr (!EXACT) {
    return *reinterpret_cast<const bf16x8 *>(row + col);
  } else {   // rows are aligned to 8 bytes; columns past d are 0
    typedef __attribute__((ext_vector_type(8), aligned(8))) bf16 bf16x8_8;
    const bf16x8 t = *reinterpret_cast<const bf16x8_8 *>(row + (col < d ? col : 0));
    bf16x8 o;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = col < d ? t[e] : (bf16)0.0f;
    return o;
  }
}

// Steps 0 .. N-1 of a run of MFMAs whose A operands come from LDS: load(i) fetches the fragments
// of step i, mma(i) multiplies with them, extra(i) is whatever else should issue during step i.
// The loads run P steps ahead of the MFMAs, and nothing may be scheduled across a step boundary:
// left alone, the compiler issues each LDS read right in front of its MFMA and the wave (one per
// SIMD in these kernels) sits out the LDS latency each time.
template <int N, int P, typename L>
__device__ __forceinline__ void pipelined_start(L &&load) {
#pragma unroll
  for (int i = 0; i < P && i < N; ++i) load(i);
  __builtin_amdgcn_sched_barrier(0);
}
template <int N, int P, typename L, typename M, typename X>
__device__ __forceinline__ void pipelined_run(L &&load, M &&mma, X &&extra) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if (i + P < N) load(i + P);
    extra(i);
    mma(i);
    __builtin_amdgcn_sched_barrier(0);
  }
}
template <int N, int P, typename L, typename M, typename X>
__device__ __forceinline__ void pipelined(L &&load, M &&mma, X &&extra) {
  pipelined_start<N, P>(load);
  pipelined_run<N, P>(load, mma, extra);
}

// wait until at most N of this wave's memory operations are outstanding, then the workgroup barrier
template <int N>
__device__ __forceinline__ void wait_and_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// The value is needed "now": makes the compiler wait for the global load behind v here, before the
// main loop, rather than at the first use inside it -- a wait for ordinary loads inside the loop
// would also drain the DMAs in flight, which the compiler does not know about.
template <typename V>
__device__ __forceinline__ void arrive(V &v) {
  asm volatile("" : "+v"(v));
}
// maximum over the four lanes that share lane % 16:
// v_permlane{16,32}_swap of a value with itself leaves the two halves of every pair side by side; unlike a shuffle
// through LDS it costs a vector instruction's latency, which the forward kernel pays twice in every tile's chain.
// The results are taken into scalars before they are reinterpreted: __builtin_bit_cast of an element of a vector reads
// element 0 whichever is named (ROCm 7.2's clang), and the maximum of element 0 with itself folds away.
__device__ __forceinline__ float quad_max(float v) {
  typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
  const unsigned a = __builtin_bit_cast(unsigned, v);
  const u32x2 p = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane16_swap(a, a, false, false));
  const unsigned p0 = p[0], p1 = p[1];
  v = fmaxf(__builtin_bit_cast(float, p0), __builtin_bit_cast(float, p1));
  const unsigned b = __builtin_bit_cast(unsigned, v);
  const u32x2 q = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(b, b, false, false));
  const unsigned q0 = q[0], q1 = q[1];
  return fmaxf(__builtin_bit_cast(float, q0), __builtin_bit_cast(float, q1));
}

// Number of a wave's IPW DMA instructions that go out by step `step` of the STEPS MFMA steps of a tile (both runs counted):
// spread evenly, because the texture path takes 16 cycles for each and a wave that meets a full queue waits.
template <int IPW, int STEPS>
constexpr int dma_by(int step) { return ((step + 1) * IPW + STEPS - 1) / STEPS; }

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

// The backward kernels: a workgroup owns one 64-row block (queries for dq, keys for dk / dv), 16 rows to each of waves 0-3
// and again to waves 4-7: the two halves of the workgroup take the first and the last 32 rows of every streamed
// tile, and their partial results are merged through LDS at the end.  Half the tile per wave halves the registers
// of its scores and its chain per tile, and no wave idles while the mask leaves work to the other half only.  Blocks are
// handed out in the order of falling work, so a compute unit that got a long block gets a short one after it.  Measured with
// paired blocks and whole tiles before, dq + dk/dv at 2048 tokens x 16 heads: head size 64 75 us, 128 107, 160 121;
// now 56, 92, 101.  (In the forward kernel, which has fewer registers to save, the merge costs more than it gives.)
__host__ __device__ inline int row_blocks(int s) { return (s + 63) / 64; }

// Over many sequences the work evens out by itself, and what a workgroup costs besides its tiles (its own rows, the first
// tiles, the merge, the results: 12-17 us at head sizes 128 and 160) counts instead.  PAIRED has half the workgroups: waves 0-3
// and 4-7 own blocks p and nb - 1 - p and take whole tiles, as in the forward kernel, with nothing to merge.  32 x 16 heads of 160,
// us: s 80 halves 64, paired 52; 128 88, 70; 256 175, 149; 768 699, 652.  16 heads, s = 1990: 103, 113.  bwd_paired() chooses.
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

// Which head a workgroup works on, and at which place of the head's order of blocks.  The heads of all sequences are numbered
// through and a grid row takes `group` of them, heads fastest: with a multiple of 8 all workgroups of a head run on one XCD (they
// are dealt out in turn) and its L2 serves every tile after the first reading.  Measured with the blocks running fastest, forward
// at 4 x 2048 x 16 heads: head size 64 61-64 us, 128 113-116, 160 122; with the heads fastest 55, 102, 105.
// Rows of about 32 heads, 4 to an XCD, because with all heads in one row the L2 holds too little of each to serve it: forward
// at 32 x 16 heads, s = 768, head size 64 97 us in one row, 71 in rows; 160 207, 168; backward of 64 at s = 1024 473, 418.
// One row where (nearly) all workgroups are in flight at once or few wait, and the order by length matters more: forward at
// 256 heads of 64, s = 320 (768 workgroups) 13.2 us in one row, 14.8 in rows; the backward by halves, of head size 64, does
// better with 128 heads to a row.  The rows are evened out, and the last is as short as it has to be: places without work at
// the end of every row unbalance the chip (128 x 100 heads, s = 1990, in rows of 32 places: backward 682 us instead of 577).
struct HeadBlock {
  int head, batch, order;
  bool none;   // nothing left at this place of the last row
  __device__ HeadBlock(int b, int n, int group, int count, unsigned place) {   // count: blocks of a head; place: in the grid row
    const unsigned heads = (unsigned)b * (unsigned)n, first = blockIdx.y * (unsigned)group;
    const unsigned here = heads - first < (unsigned)group ? heads - first : (unsigned)group;
    const unsigned hb = first + place % here;
    order = place / here;
    head = hb % (unsigned)n;
    batch = hb / (unsigned)n;
    none = order >= count;
  }
  static int group(int b, int n, int count, int want, int few) {   // few: up to how many workgroups one row takes all
    const int64_t heads = (int64_t)b * n;
    int64_t rows = heads * count <= few || heads < want ? 1 : heads / want;
    if (rows > 65535) rows = 65535;   // the grid's limit
    const int64_t even = ((heads + rows - 1) / rows + 7) / 8 * 8;
    return (int)(even < heads ? even : heads);
  }
  static dim3 grid(int b, int n, int group, int count) {
    return dim3((unsigned)group * count, (unsigned)(((int64_t)b * n + group - 1) / group));
  }
};

// Partial accumulators of waves 4-7 to waves 0-3 through LDS: 16-byte slots per lane, conflict-free.
__device__ __forceinline__ f32x4 *merge_slots(char *smem, int wave, int lane, int blocks) {
  return reinterpret_cast<f32x4 *>(smem) + (wave & 3) * (blocks * 64) + lane;
}

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

// ------------------------------------------------------------------ backward: dq (and D)
struct BackwardArgs {
  int b, s, n, head_dim, group;
  float scale;
  const bf16 *qkv, *a;
  const float *lse;
  const bf16 *da;
  bf16 *dqkv;
  float *Dvec;
};

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
  const bf16 *dah = da + (int64_t)bi * s * pld + (int64_t)j * d;
  {
    const bf16 *ar = a + ((int64_t)bi * s + qc) * pld + (int64_t)j * d;
    f32x4 t = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const int col = 32 * kk + 8 * g;
      qf[kk] = row_chunk<EXACT>(base + (int64_t)qc * ld, col, d);
      dof[kk] = row_chunk<EXACT>(dah + (int64_t)qc * pld, col, d);
      const bf16x8 av = row_chunk<EXACT>(ar, col, d);
      if constexpr (EXACT) {   // D on the diagonal of a dO^T, by the same MFMAs as dP: where a row has one key (a = v) the two cancel exactly
        t = MFMA16(av, dof[kk], t);
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) dsum += (float)dof[kk][i] * (float)av[i];
      }
    }
    if constexpr (EXACT) {
      const float mine = (lr & 2) ? ((lr & 1) ? t[3] : t[2]) : ((lr & 1) ? t[1] : t[0]);
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
  constexpr bool LATE = PAIRED && D == 160;   // fewer fragments read ahead: no room in the registers
  const HeadBlock hb(b, n, group, BackwardBlocks<PAIRED>::count(s), place);
  const int j = hb.head, bi = hb.batch;
  if (hb.none) return;
  const BackwardBlocks<PAIRED> bb(s, hb.order, threadIdx.x >> 6);   // (from the thread number; head size 160: 194 registers instead of 230)
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
        constexpr int P = LATE ? 1 : 2;
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
      constexpr int PT = LATE ? 2 : 3;
      bf16x8 otr[PT + 1], qtr[PT + 1];
      auto load = [&](int i) {   // step i: query slot i / DB, output block i % DB
        otr[i % (PT + 1)] = T::tr(Ot, ln, i % DB, i / DB);
        qtr[i % (PT + 1)] = T::tr(Qt, ln, i % DB, i / DB);
      };
      if constexpr (!LATE) pipelined_start<NS * DB, PT>(load);
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
        const f32x4 ls = *reinterpret_cast<const f32x4 *>(stat + 16 * qb + 4 * g);
        if constexpr (EXACT) pc[qb] -= *reinterpret_cast<const f32x4 *>(stat + 64 + 16 * qb + 4 * g);
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
      if constexpr (LATE) pipelined_start<NS * DB, PT>(load);
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
    const int64_t st = ((int64_t)bi * n + j) * s;
    if (wave < 4 && !all_finite(z)) redo_dkv<bf16, D>(base, ld, dab, pld, s, d, scale, kw, key, lse + st, [&](int t) { return Dvec[st + t]; }, g, out);
  }
}

template <int D, bool PAIRED, bool EXACT>
__global__ __launch_bounds__(512) void attn_bwd_dq_kernel(BackwardArgs w) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  dq_block<D, PAIRED, EXACT>(blockIdx.x, smem, w.b, w.s, w.n, w.head_dim, w.group, w.scale, w.qkv, w.a, w.lse, w.da, w.dqkv, w.Dvec);
}
template <int D, bool PAIRED, bool EXACT>
__global__ __launch_bounds__(512) void attn_bwd_dkv_kernel(BackwardArgs w) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  dkv_block<D, PAIRED, EXACT, false>(blockIdx.x, smem, w.b, w.s, w.n, w.head_dim, w.group, w.scale, w.qkv, w.a, w.lse, w.Dvec, w.da, w.dqkv);
}
// Both in one launch (bwd_one_launch says when): the first half of a grid row's workgroups (dk / dv, the longer ones) compute D for themselves.
template <int D>
__global__ __launch_bounds__(512) void attn_bwd_kernel(BackwardArgs w) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const unsigned half = gridDim.x / 2;
  if (blockIdx.x < half)
    dkv_block<D, false, false, true>(blockIdx.x, smem, w.b, w.s, w.n, w.head_dim, w.group, w.scale, w.qkv, w.a, w.lse, nullptr, w.da, w.dqkv);
  else
    dq_block<D, false, false>(blockIdx.x - half, smem, w.b, w.s, w.n, w.head_dim, w.group, w.scale, w.qkv, w.a, w.lse, w.da, w.dqkv, w.Dvec);
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

// 16 rows per wave in both backward kernels: 32 do not fit the 256 registers a wave has at eight waves.
template <int D, bool PAIRED, bool EXACT = false>
int bwd_launch_p(int b, int s, int n, int d, float scale, const void *qkv, const void *a, const float *lse, const void *da,
                 void *dqkv, void *ws, hipStream_t st) {
  constexpr int smem_dq = 3 * 2 * 64 * D * 2, smem_dkv = 3 * (2 * 64 * D * 2 + 512);
  static_assert(smem_dkv >= 4 * 2 * (D / 16) * 1024, "the merge of the two halves fits the rings");
  static unsigned long long attr_done = 0;
  int device;
  if (!attr_is_set(attr_done, &device)) {
    if (hipFuncSetAttribute((const void *)attn_bwd_dq_kernel<D, PAIRED, EXACT>, hipFuncAttributeMaxDynamicSharedMemorySize, smem_dq) != hipSuccess ||
        hipFuncSetAttribute((const void *)attn_bwd_dkv_kernel<D, PAIRED, EXACT>, hipFuncAttributeMaxDynamicSharedMemorySize, smem_dkv) != hipSuccess)
      return MTNLG_HIP_ERROR;
    attr_mark_set(attr_done, device);
  }
  float *Dvec = (float *)ws;
  const int count = BackwardBlocks<PAIRED>::count(s), group = HeadBlock::group(b, n, count, PAIRED || D >= 128 ? 32 : 128, PAIRED ? 511 : 2047);
  const dim3 grid = HeadBlock::grid(b, n, group, count);
  LaunchScope scope(MTNLG_K_ATTN_BWD, st);
  const BackwardArgs w{b, s, n, d, group, scale, (const bf16 *)qkv, (const bf16 *)a, lse, (const bf16 *)da, (bf16 *)dqkv, Dvec};
  attn_bwd_dq_kernel<D, PAIRED, EXACT><<<grid, 512, smem_dq, st>>>(w);
  MTNLG_TRY(check_launch());
  attn_bwd_dkv_kernel<D, PAIRED, EXACT><<<grid, 512, smem_dkv, st>>>(w);
  return check_launch();
}

// What either backward kernel takes for `heads` heads of nb blocks in `count` workgroups each, of nb tiles and fewer: the longest
// workgroup where all run at once, else the work spread over the compute units and a part of a last, shortest workgroup.
struct BackwardCost {
  double tile, fixed, tail;   // us for each tile, for each workgroup; the part of the last workgroup
  double time(int64_t heads, int nb, int count) const {
    const double longest = nb * tile + fixed, shortest = (nb - count + 1) * tile + fixed;
    if (heads * count <= 256) return longest;
    const double spread = heads * count * ((2 * nb - count + 1) / 2.0 * tile + fixed) / 256 + tail * shortest;
    return spread > longest ? spread : longest;
  }
};

// Two blocks of a head in each workgroup?  At head size 128 and 160, where one workgroup at a time runs on a compute unit, whichever
// the estimate says; its constants were fitted to 207 and 201 measured sizes (8 to 1024 heads, s 80 to 4096, both kernels), for
// which the choice costs 0.4 % on average against the better of the two (10 % at most: 160, 96 heads, s = 384).  At head size 64, with three workgroups on a compute unit to
// cover each other, only for sequences of two blocks, of which those that come here have more than 384 heads (bwd_one_launch takes the others):
// 512 heads, s = 80 26.0 us by halves, 23.3 paired; but 300, s = 192 31.2, 36.7.
template <int D>
bool bwd_paired(int b, int s, int n) {
  const int64_t heads = (int64_t)b * n;
  const int nb = row_blocks(s);
  if (D < 128) return nb == 2;
  constexpr BackwardCost halves = D == 128 ? BackwardCost{1.95, 12.0, 0.5} : BackwardCost{2.1, 14.5, 0.63};
  constexpr BackwardCost pairs = D == 128 ? BackwardCost{2.6, 13.0, 0.75} : BackwardCost{3.2, 16.5, 0.67};
  return pairs.time(heads, nb, (nb + 1) / 2) < halves.time(heads, nb, nb);
}

constexpr int ONE_LAUNCH_ROWS = 4096;   // what their D has room for in LDS
template <int D>
int bwd_launch_one(int b, int s, int n, float scale, const void *qkv, const void *a, const float *lse, const void *da, void *dqkv, void *ws,
                   hipStream_t st) {
  const int count = row_blocks(s), group = HeadBlock::group(b, n, count, 32, 2047);
  const int smem = 3 * (2 * 64 * D * 2 + 512) + count * 64 * (int)sizeof(float);
  static unsigned long long attr_done = 0;
  int device;
  if (!attr_is_set(attr_done, &device)) {
    if (hipFuncSetAttribute((const void *)attn_bwd_kernel<D>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            3 * (2 * 64 * D * 2 + 512) + ONE_LAUNCH_ROWS * (int)sizeof(float)) != hipSuccess)
      return MTNLG_HIP_ERROR;
    attr_mark_set(attr_done, device);
  }
  dim3 grid = HeadBlock::grid(b, n, group, count);
  grid.x *= 2;
  LaunchScope scope(MTNLG_K_ATTN_BWD, st);
  attn_bwd_kernel<D><<<grid, 512, smem, st>>>(
      BackwardArgs{b, s, n, D, group, scale, (const bf16 *)qkv, (const bf16 *)a, lse, (const bf16 *)da, (bf16 *)dqkv, (float *)ws});
  return check_launch();
}

// One launch where all workgroups of either kernel run at once, so that both kernels' would leave units idle one after the other: a second
// D for every tile costs less than that and the launch.  us, two launches / one: 1 x 256 x 2 heads of 160 21.9 / 13.7, 2 x 300 x 2 of 128
// 20.8 / 13.4, 2 x 257 of 64 13.3 / 8.7; by blocks of all heads together (s 192 to 1024): up to 128 1.5 times as fast, 256 1.1 to 1.3; 384 1.0 to
// 1.05 and 512 0.85 to 0.93 at head sizes 128 and 160, where one workgroup runs on a unit; at 64, where three do, 512 1.16 to 1.19, 768 1.11,
// 1024 0.96 (two blocks of 70 to 128 rows: 256 1.22 to 1.35, 384 0.92 to 1.10, 512 0.92 to 1.01, 768 1.13 to 1.20).  At 64 beyond s 960 D takes
// the LDS of the third workgroup: up to 256 blocks 1.19 to 1.44 times as fast from s 1030 to 4096, 384 1.11 to
// 1.33, 512 0.92 to 1.17, 768 0.94 to 1.06.
template <int D>
bool bwd_one_launch(int b, int s, int n) {
  return s <= ONE_LAUNCH_ROWS && (int64_t)b * n * row_blocks(s) <= (D >= 128 || s > 1024 ? 256 : 768);
}

template <int D>
int bwd_launch(int b, int s, int n, float scale, const void *qkv, const void *a, const float *lse, const void *da,
               void *dqkv, void *ws, hipStream_t st) {
  if (bwd_one_launch<D>(b, s, n)) return bwd_launch_one<D>(b, s, n, scale, qkv, a, lse, da, dqkv, ws, st);
  if (bwd_paired<D>(b, s, n)) return bwd_launch_p<D, true>(b, s, n, D, scale, qkv, a, lse, da, dqkv, ws, st);
  return bwd_launch_p<D, false>(b, s, n, D, scale, qkv, a, lse, da, dqkv, ws, st);
}

// The DMA addresses a sequence's rows with 32-bit byte offsets from its first row.
bool fits(int s, int n, int d) { return (int64_t)s * n * 3 * d * 2 < ((int64_t)1 << 31); }

// fn<D>, D: the head size rounded up to a multiple of 32
#define BY_HEAD_SIZE(fn, ...)                                  \
  switch ((d + 31) / 32) {                                     \
    case 1: return fn(32)(__VA_ARGS__);                        \
    case 2: return fn(64)(__VA_ARGS__);                        \
    case 3: return fn(96)(__VA_ARGS__);                        \
    case 4: return fn(128)(__VA_ARGS__);                       \
    case 5: return fn(160)(__VA_ARGS__);                       \
    case 6: return fn(192)(__VA_ARGS__);                       \
    default: return MTNLG_UNSUPPORTED_SHAPE;                   \
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

int attention_bwd_mfma(int b, int s, int n, int d, float scale, const void *qkv, const void *a, const float *lse,
                       const void *da, void *dqkv, void *ws, hipStream_t stream) {
  if (n > 65535 || b > 65535 || !fits(s, n, d)) return MTNLG_UNSUPPORTED_SHAPE;
  switch (d) {
    case 64: return bwd_launch<64>(b, s, n, scale, qkv, a, lse, da, dqkv, ws, stream);
    case 128: return bwd_launch<128>(b, s, n, scale, qkv, a, lse, da, dqkv, ws, stream);
    case 160: return bwd_launch<160>(b, s, n, scale, qkv, a, lse, da, dqkv, ws, stream);
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

int attention_bwd_exact(int b, int s, int n, int d, float scale, const void *qkv, const void *a, const float *lse, const void *da,
                        void *dqkv, void *ws, hipStream_t stream) {
#define BWD(D) bwd_launch_p<D, false, true>
  BY_HEAD_SIZE(BWD, b, s, n, d, scale, qkv, a, lse, da, dqkv, ws, stream)
#undef BWD
}

}  // namespace mtnlg
