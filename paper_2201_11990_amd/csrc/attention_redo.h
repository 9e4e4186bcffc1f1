// What the attention kernels that keep P and dS in fp32 share (attention_f32.hip; the EXACT ones of attention_mfma.hip, attention_fwd16.hip, attention_bwd.hip, attention_bwd64.hip): the slow path
// for inputs that are not finite.
#pragma once
#include "common.h"

namespace mtnlg {

namespace {

// sum over the four lanes that share lane % 16
__device__ __forceinline__ float quad_sum(float v) {
  v += __shfl_xor(v, 16, 64);
  return v + __shfl_xor(v, 32, 64);
}

// The slow path of the kernels that keep scores in fp32.  Their loops multiply masked elements (P or dS = 0) with rows that the mask
// hides, in the blocks of 16 or 32 rows that the diagonal crosses and in a last block that hangs over the end.  With finite inputs
// that adds zero; an infinity or NaN in such a row would spread to rows that do not depend on it (0 x inf).  A wave whose result is
// not finite therefore computes its 16 rows once more, on the vector ALU and one streamed row at a time, reading only what each
// row depends on.  Four lanes share a row; lane g of them holds columns 16 c + 4 g .. + 3.  Operands are read from memory at every
// use: held in registers they would cost the loop above its occupancy.  (A NaN in token 0, so that every wave comes here: 8.0 ms forward
// and backward at 2 x 1024 x 16 heads of 96, 0.43 ms with finite inputs.  Checking the crossed blocks inside the loops instead: up to
// 90 registers more in them.)
template <typename E, int DP>
struct Quarter {
  static constexpr int NC = DP / 16;
  f32x4 v[NC];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int c = 0; c < NC; ++c) v[c] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  }
  __device__ __forceinline__ void add(float w, const E *row, int d, int g) {   // columns past d: anything, not stored
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int col = 16 * c + 4 * g;
      const f32x4 t = load4(row + (col < d ? col : 0));
#pragma unroll
      for (int e = 0; e < 4; ++e) v[c][e] = fmaf(w, t[e], v[c][e]);
    }
  }
  __device__ __forceinline__ void store(E *row, int d, float mul, int g) const {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int col = 16 * c + 4 * g;
      if (col >= d) continue;
      const f32x4 x = v[c] * mul;
      if constexpr (sizeof(E) == 4) *reinterpret_cast<f32x4 *>(row + col) = x;
      else *reinterpret_cast<bf16x4 *>(row + col) = bf16x4{(bf16)x[0], (bf16)x[1], (bf16)x[2], (bf16)x[3]};
    }
  }
};
// Whether no lane of the wave has stored a non-finite value (z: 0 or NaN).  If one has, the stores are waited for: other lanes write
// the same places next.
__device__ __forceinline__ bool all_finite(float z) {
  if (__builtin_amdgcn_ballot_w64(z != 0.0f) == 0) return true;
  __threadfence_block();
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  return false;
}
template <typename E>   // the dot product of two rows, in all four lanes
__device__ __forceinline__ float dot(const E *x, const E *y, int d, int g) {
  float t = 0.0f;
#pragma unroll 1
  for (int col = 4 * g; col < d; col += 16) {
    const f32x4 p = load4(x + col), q = load4(y + col);
#pragma unroll
    for (int e = 0; e < 4; ++e) t = fmaf(p[e], q[e], t);
  }
  return quad_sum(t);
}

// 16 rows of the result, row q = first row + lane % 16 (rows q >= s: computed as row s - 1, not stored).  base, da, lse, out: of
// the batch's sequence and the head, row 0; last: the last key any of the rows sees.
template <typename E, int DP>
__device__ __forceinline__ void redo_fwd(const E *base, int64_t ld, int s, int d, float scale, int q, int last, int g, E *out, float *out_lse) {
  const E *qrow = base + (q < s ? q : s - 1) * ld;
  Quarter<E, DP> sum;
  sum.clear();
  float m = -INFINITY;
#pragma unroll 1
  for (int u = 0; u <= last; ++u) {
    const float sc = dot(qrow, base + d + u * ld, d, g) * scale;
    if (u <= q) m = fmaxf(m, sc);
  }
  float l = 0.0f;
#pragma unroll 1
  for (int u = 0; u <= last; ++u) {
    const float p = expf(dot(qrow, base + d + u * ld, d, g) * scale - m);
    if (u <= q) {
      l += p;
      sum.add(p, base + 2 * d + u * ld, d, g);
    }
  }
  if (q >= s) return;
  sum.store(out, d, 1.0f / l, g);
  if (g == 0) *out_lse = m + logf(l);
}
template <typename E, int DP>
__device__ __forceinline__ void redo_dq(const E *base, int64_t ld, const E *da, int64_t pld, int s, int d, float scale, int q, int last,
                                        float lse, float dsum, int g, E *out) {
  const int qc = q < s ? q : s - 1;
  Quarter<E, DP> sum;
  sum.clear();
#pragma unroll 1
  for (int u = 0; u <= last; ++u) {
    const E *krow = base + d + u * ld;
    const float dp = dot(da + qc * pld, krow + d, d, g);
    const float p = expf(dot(base + qc * ld, krow, d, g) * scale - lse);
    if (u <= q) sum.add(p * (dp - dsum), krow, d, g);
  }
  if (q < s) sum.store(out, d, scale, g);
}
template <typename E, int DP>
__device__ __forceinline__ void redo_dv(const E *base, int64_t ld, const E *da, int64_t pld, int s, int d, float scale, int row0, int key,
                                        const float *lse, int g, E *out) {
  const E *krow = base + d + (key < s ? key : s - 1) * ld;
  Quarter<E, DP> sum;
  sum.clear();
#pragma unroll 1
  for (int t = row0; t < s; ++t) {
    const float p = expf(dot(krow, base + t * ld, d, g) * scale - lse[t]);
    if (t >= key) sum.add(p, da + t * pld, d, g);
  }
  if (key < s) sum.store(out + 2 * d, d, 1.0f, g);
}
template <typename E, int DP, typename DOf>   // d_of(t): D of row t
__device__ __forceinline__ void redo_dk(const E *base, int64_t ld, const E *da, int64_t pld, int s, int d, float scale, int row0, int key,
                                        const float *lse, DOf &&d_of, int g, E *out) {
  const E *krow = base + d + (key < s ? key : s - 1) * ld;
  Quarter<E, DP> sum;
  sum.clear();
#pragma unroll 1
  for (int t = row0; t < s; ++t) {
    const float p = expf(dot(krow, base + t * ld, d, g) * scale - lse[t]), dp = dot(krow + d, da + t * pld, d, g), dt = d_of(t);
    if (t >= key) sum.add(p * (dp - dt), base + t * ld, d, g);
  }
  if (key < s) sum.store(out + d, d, scale, g);
}

}  // namespace

}  // namespace mtnlg
