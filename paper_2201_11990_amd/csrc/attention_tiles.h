// What the tiled attention kernels share (attention_mfma.hip, attention_fwd16.hip: forward; attention_bwd.hip, attention_bwd64.hip: backward): tiles in LDS and the
// streams that fill them, fragments, weights, the order of the grid.
#pragma once
#include <math.h>

#include <type_traits>
#include <utility>

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
#define MFMA32(a, b, c) __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0)
typedef __attribute__((ext_vector_type(16))) float f32x16;

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
// WIDE: for the fragments of 32x32x16 MFMAs.  16-byte reads are served 16 lanes at a time (0-3, 12-15, 20-27; 4-11, 16-19, 28-31; the same from 32 on), here
// 16 rows that differ in their low four bits; transposing reads 32 lanes at a time, 64 bytes each of rows 4 h .. 4 h + 3.  So the mask takes all bits
// of the row that its units do not place already, the lowest ones to the highest bits: no conflicts at any head size (128 with the other mask: four rows of a
// transposing read on the same banks, a fifth of the kernel's time).
template <int D, bool WIDE = false>
struct Tile {
  static constexpr bool ODD = D / 32 % 2 == 1;   // 32, 96, 160
  static constexpr int UPR = D / 8;        // 16-byte units per row
  static constexpr int BYTES = 64 * D * 2;
  static constexpr int NI = D / 32;        // DMA instructions per wave and tile (16 rows)
  static __device__ __forceinline__ int mask(int row) {
    if constexpr (ODD) return WIDE ? row >> 2 & 3 : row >> 1 & 3;
    else if constexpr (WIDE && D == 128) return (row & 3) << 2 | (row >> 2 & 3);
    else if constexpr (WIDE) return (row >> 1 & 1) << 2 | (row >> 2 & 3);
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
  static constexpr int ROWS16 = 16 * UPR * 16, ROWS32 = 2 * ROWS16;   // bytes of 16, 32 tile rows
  // The same for the fragments of 32x32x16 MFMAs: lane l holds row l%32, columns 16 kk + 8 (l/32) .. + 7, or column 32 cb + l%32 and, with
  // h = l/32, rows 16 t + 4 h .. + 3 (elements 0-3) and 16 t + 8 + 4 h .. + 3 (4-7).
  struct Lane32 {
    uint32_t n0, t0;
    __device__ __forceinline__ explicit Lane32(int lane) {
      const int L = lane & 15;
      n0 = (uint32_t)off(lane & 31, lane >> 5);
      const int col = 16 * (lane >> 4 & 1) + 4 * (L & 3);
      t0 = (uint32_t)(off(4 * (lane >> 5) + (L >> 2), col >> 3) + (col & 7) * 2);
    }
    __device__ __forceinline__ void here() { asm volatile("" : "+v"(n0), "+v"(t0)); }
    __device__ __forceinline__ uint32_t nat(int kk) const {
      if constexpr (ODD) return (n0 ^ ((kk & 1) * 32)) + (kk >> 1) * 64;
      else if constexpr (D == 192) return (n0 ^ ((kk & 3) * 32)) + (kk >> 2) * 128;
      else return n0 ^ (kk * 32);
    }
    __device__ __forceinline__ uint32_t tr(int cb, int low8) const {   // low8: rows + 8
      static_assert(WIDE, "");
      if constexpr (ODD) return (t0 ^ (low8 * 32)) + cb * 64 + low8 * (ROWS16 / 2);
      else if constexpr (D == 192) return (t0 ^ ((cb & 1) * 64) ^ (low8 * 32)) + (cb >> 1) * 128 + low8 * (ROWS16 / 2);
      else return (t0 ^ (cb * 64) ^ (low8 * 32)) + low8 * (ROWS16 / 2);
    }
  };
  static __device__ __forceinline__ bf16x8 nat32(const char *t, const Lane32 &ln, int kk) { return *reinterpret_cast<const bf16x8 *>(t + ln.nat(kk)); }
  static __device__ __forceinline__ bf16x8 tr32(const char *t, const Lane32 &ln, int cb, int t16) {
    const char *p = t + t16 * ROWS16;
    const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_ptr)(p + ln.tr(cb, 0)));
    const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_ptr)(p + ln.tr(cb, 1)));
    const i16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
  }
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
    // left = max(left - tile_bytes, 0) in scalar registers: left to itself the compiler makes a saturating subtraction of it, which only the vector unit has,
    // and a descriptor in vector registers
    asm("s_sub_i32 %0, %0, %1\n\ts_max_i32 %0, %0, 0" : "+s"(left) : "s"(tile_bytes) : "scc");
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

// the same of elements 8 t .. 8 t + 7 of a 32x32 block
template <bool EXACT>
__device__ __forceinline__ Parts<EXACT ? 3 : 1> weights16(const f32x16 &v, int t) {
  Parts<EXACT ? 3 : 1> w;
  if constexpr (EXACT) {
    w.of({v[8 * t], v[8 * t + 1], v[8 * t + 2], v[8 * t + 3], v[8 * t + 4], v[8 * t + 5], v[8 * t + 6], v[8 * t + 7]});
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) w.p[0][e] = (bf16)v[8 * t + e];
  }
  return w;
}
template <int N>
__device__ __forceinline__ f32x16 mma_weights32(const bf16x8 &x, const Parts<N> &w, f32x16 acc) {
#pragma unroll
  for (int i = N - 1; i >= 0; --i) acc = MFMA32(x, w.p[i], acc);
  return acc;
}
__device__ __forceinline__ f32x4 quarter_of(const f32x16 &v, int q) { return f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]}; }

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

// fn(0) .. fn(N - 1) with the number known at compile time (loops of this size are not unrolled on request, and arrays indexed by a loop's
// counter would live in memory)
template <typename F, int... I>
__device__ __forceinline__ void for_each_step(F &&fn, std::integer_sequence<int, I...>) {
  (fn(std::integral_constant<int, I>{}), ...);
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
// The lane's number, worked out where it stands: a register less across a loop that needs them all.
__device__ __forceinline__ int lane_here() {
  int lane;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
  return lane;
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

// what the backward kernels take
struct BackwardArgs {
  int b, s, n, head_dim, group;
  float scale;
  const bf16 *qkv, *a;
  const float *lse;
  const bf16 *da;
  bf16 *dqkv;
  float *Dvec;
};

// maximum over the two lanes that share lane % 32
__device__ __forceinline__ float pair_max(float v) {
  typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
  const unsigned a = __builtin_bit_cast(unsigned, v);
  const u32x2 p = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(a, a, false, false));
  const unsigned p0 = p[0], p1 = p[1];
  return fmaxf(__builtin_bit_cast(float, p0), __builtin_bit_cast(float, p1));
}

// EXACT with SPLIT 2, where waves `wave` and `other` have stored half of a result's columns each: the slow path computes whole rows, so the wave of part 0
// takes it if either has found a result that is not finite (z: NaN), after what both have stored.
__device__ __forceinline__ float either_part(float z, char *smem, int wave, int other, int part, int lane) {
  __syncthreads();   // LDS is free
  int *bad = reinterpret_cast<int *>(smem);
  const bool any = __builtin_amdgcn_ballot_w64(z != 0.0f) != 0;
  if (lane == 0) bad[wave] = any;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  return part == 0 && (bad[wave] | bad[other]) ? NAN : 0.0f;
}

// Number of a wave's IPW DMA instructions that go out by step `step` of the STEPS MFMA steps of a tile (both runs counted):
// spread evenly, because the texture path takes 16 cycles for each and a wave that meets a full queue waits.
template <int IPW, int STEPS>
constexpr int dma_by(int step) { return ((step + 1) * IPW + STEPS - 1) / STEPS; }

__host__ __device__ inline int row_blocks(int s) { return (s + 63) / 64; }
// How many of the 32-row parts of a workgroup's ntiles tiles hold a row that the own rows 32 own .. + 31 see under the causal mask, from the first on: by a wave that takes part `part` of every
// tile (subs 1) or both (2).
__device__ __forceinline__ int visible_parts(int own, int part, int subs, int ntiles) {
  const int seen = subs == 1 ? (own + 2 - part) / 2 : own + 1;
  return seen < subs * ntiles ? seen : subs * ntiles;
}
__host__ __device__ inline int own_blocks(int s, int owned) { return (s + owned - 1) / owned; }   // workgroups to a head

// Where all workgroups run at once, several to a compute unit, places i, 256 + i, 512 + i share one: every other 256 go out in the opposite order, so that
// the units' work comes out even.
__device__ __forceinline__ int in_turns(int order, int count, int heads) {
  const int each = (255 + heads) / heads, turn = order / each, first = turn * each, end = first + each < count ? first + each : count;
  return turn & 1 ? end - 1 - (order - first) : order;
}

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

// Calls of more workgroups of 64 rows than there are units, and no more of 128, whose heads are scattered: with heads running fastest the workgroups of a head lie on one XCD if the number of heads is a
// multiple of 8, else on 2, 4 or 8, and what it streams comes into as many L2s.  The fewer and larger workgroups (pairs of blocks with 16 rows to a wave, attention_fwd16.hip, or 128 rows) do better, on
// more XCDs up to longer sequences.  Times as fast as workgroups of 64 rows with 32 to a wave, forward at head size 160 by number of heads (900 sizes): multiples of 8 0.83 to 1.04; of 4 s 65 to 128 1.04 to 1.18, then 0.9
// to 1.03; of 2 up to 384 1.03 to 1.27, 385 to 512 0.99 to 1.02, then 0.9 to 0.99; odd 1.05 to 1.37 up to 768; at 128 0.95 to 1.13, 1.02 to 1.2, 1.03 to 1.28.  us: 384 tokens x 85 heads of 160 21.3 / 17.6, 123 x 225
// 12.2 / 9.2, 197 x 102 14.0 / 11.6; but 350 x 68 12.9 / 13.6.  At 128 only from 321 blocks on, and not from s 129 to 192 (142 x 120 7.1 / 7.6); an odd number of heads of more than 256 tokens from 64 blocks
// less on (358 x 51 of 128 12.5 / 10.9, 251 x 63 of 160 10.8 / 10.0).
inline bool heads_scattered(int b, int n, int s, int d) {
  const int64_t heads = (int64_t)b * n;
  const int longest = heads % 8 == 0 ? 0 : heads % 4 == 0 ? 128 : heads % 2 == 0 ? 384 : 768;
  if (d <= 128 && s > 128 && s <= 192) return false;
  const int fewest = (d <= 128 ? 320 : 256) - (heads % 2 && s > 256 ? 64 : 0);
  return s <= longest && heads * row_blocks(s) > fewest && heads * own_blocks(s, 128) <= 256;
}

// The DMA addresses a sequence's rows with 32-bit byte offsets from its first row.
inline bool fits(int s, int n, int d) { return (int64_t)s * n * 3 * d * 2 < ((int64_t)1 << 31); }

template <typename K>
int set_lds(K kernel, int bytes) {
  return hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess ? MTNLG_OK : MTNLG_HIP_ERROR;
}

}  // namespace

}  // namespace mtnlg
