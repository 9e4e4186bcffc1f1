// Causal softmax attention, forward and backward, on the fp32 matrix instructions (v_mfma_f32_16x16x4_f32): scores,
// probabilities and sums stay in fp32.  This is the attention of the fp32 path, and of bf16 head sizes other than 64, 128 and 160 in
// small calls and above 192 (the rest: the EXACT kernels of the four files of bf16 attention).  Head sizes: multiples of 8 up to 256; sequences up to 4096.
//
//   S[t,u] = scale * q_t . k_u  (u <= t),  P = rowsoftmax(S),  a_t = sum_u P[t,u] v_u
//   lse[t] = log sum_u exp(S[t,u])
// backward, with D_t = da_t . a_t = sum_u P[t,u] dP[t,u]:
//   dP[t,u] = da_t . v_u,  dS = P o (dP - D),  dq_t = scale sum_u dS[t,u] k_u,
//   dk_u = scale sum_t dS[t,u] q_t,  dv_u = sum_t P[t,u] da_t
//
// Bound by the fp32 matrix rate where there are enough rows, else by each wave's chain of loads, MFMAs and exponentials.
// bf16 inputs need not be widened for the products of two inputs (q k^T, da v^T, D): those run on the bf16 matrix
// instructions with fp32 sums.  2 x 1024 tokens, 16 heads of 96, forward / backward: 162 / 540 us with all products on the
// fp32 instructions, 104 / 327 us so.  (P and dS cut into three bf16 parts that add up to them exactly, for the other products:
// slower here, 237 us forward: the waves wait for loads by then.  With tiles in LDS that is the better form.)
// A wave owns 16 rows of one side (queries forward and for dq, keys for dk / dv) and walks the other side 16 or 32 rows
// at a time; fragments are loaded from global memory straight into the registers the MFMAs read (at this matrix rate a
// wave asks the caches for 8 bytes a cycle), so there is no LDS, no barrier, and a wave stops at its own diagonal.  The four
// waves of a workgroup own neighbouring rows and share what they load in the L1, or, in small calls, the same rows, with
// the other side split between them; a head's workgroups go to one XCD where the number of heads allows it; workgroups with
// the most work start first.
//
// Lane l = 16 g + r.  Two fragment forms of a 16-row block X:
//   Rows: element (c, e) = X[r][16 c + 4 g + e]; an MFMA per (c, e) contracts over columns.  With Rows of both sides a
//         lane holds S[streamed row 4 g + i][own row r], i = 0..3.
//   (bf16: element (c, e) = X[r][32 c + 8 g + e], one MFMA per c.)
//   Cols: element (block, e) = X[4 g + e][column], NB consecutive columns per lane and group of 16 NB; an MFMA per
//         (block, e) contracts over the rows, and its other operand for e is exactly that accumulator element: P
//         and dS are used where they were computed.
#include "attention_redo.h"

namespace mtnlg {

namespace {

typedef __attribute__((ext_vector_type(2))) float f32x2;

#define MFMA4(a, b, c) __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0)

template <typename E, int DP>
struct Rows {
  static constexpr int NC = DP / 16;
  f32x4 v[NC];
  // rows first .. first + 15 of the matrix at base (pitch ld); rows past the end repeat the last one; columns past d are 0
  __device__ __forceinline__ void load(const E *base, int64_t ld, int first, int rows, int d, int g, int r) {
    const int row = first + r < rows ? first + r : rows - 1;
    const E *p = base + row * ld;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int col = 16 * c + 4 * g;
      if (16 * c + 16 > DP - 32) {   // d lies in (DP - 32, DP]
        const f32x4 t = load4(p + (col < d ? col : 0));
#pragma unroll
        for (int e = 0; e < 4; ++e) v[c][e] = col < d ? t[e] : 0.0f;
      } else {
        v[c] = load4(p + col);
      }
    }
  }
};

// bf16 rows stay bf16: lane l holds X[r][32 c + 8 g .. + 7], one v_mfma_f32_16x16x32_bf16 per c contracts over columns.
// Products of bf16 elements are exact in fp32 and the sums are fp32, as after widening, at 16 times the rate.
template <int DP>
struct Rows<bf16, DP> {
  static constexpr int NC = DP / 32;
  typedef __attribute__((ext_vector_type(8), aligned(8))) bf16 bf16x8_8;   // rows need not be aligned to more
  bf16x8 v[NC];
  __device__ __forceinline__ void load(const bf16 *base, int64_t ld, int first, int rows, int d, int g, int r) {
    const int row = first + r < rows ? first + r : rows - 1;
    const bf16 *p = base + row * ld;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int col = 32 * c + 8 * g;
      if (c == NC - 1) {   // d lies in (DP - 32, DP]
        const bf16x8 t = *reinterpret_cast<const bf16x8_8 *>(p + (col < d ? col : 0));
#pragma unroll
        for (int e = 0; e < 8; ++e) v[c][e] = col < d ? t[e] : (bf16)0.0f;
      } else {
        v[c] = *reinterpret_cast<const bf16x8_8 *>(p + col);
      }
    }
  }
};

// Rows that a wave sums in one chain.  (64 where the waves share the streamed side: with 128 dk and dv of some shapes came out up
// to 5 % less exact than with whole chains in one wave, with 64 nowhere, at 0.7 % of the time.)
constexpr int sum_rows(bool split) { return split ? 64 : 128; }

template <int DP>
struct Blocks {   // DP / 16 accumulator blocks over columns, in the order of Cols
  static constexpr int N4 = DP / 64, N2 = DP % 64 / 32, N = DP / 16;
  f32x4 b[N];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int i = 0; i < N; ++i) b[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  }
  // fp32 results: sums over rows are taken sum_rows() at a time and added up here, because the error of one chain grows with its
  // length (s = 2048, head size 64, dk against 64 bits: 1.08e-6 in one chain, 4.1e-7 so, at the same time up to head size 160).
  // A bf16 result does not show it.
  __device__ __forceinline__ void flush(Blocks &part) {
#pragma unroll
    for (int i = 0; i < N; ++i) b[i] += part.b[i];
    part.clear();
  }
  // row r of the result times mul: a lane holds 16 (or 8) consecutive columns per group.  Returns 0, or NaN where a stored value is not
  // finite.
  template <typename E>
  __device__ __forceinline__ float store(E *row, int d, float mul, int g) const {
    float z = 0.0f;
    auto put = [&](int col, f32x4 x) {
      if (col >= d) return;
      x *= mul;
#pragma unroll
      for (int e = 0; e < 4; ++e) z = fmaf(x[e], 0.0f, z);
      if constexpr (sizeof(E) == 4) *reinterpret_cast<f32x4 *>(row + col) = x;
      else *reinterpret_cast<bf16x4 *>(row + col) = bf16x4{(bf16)x[0], (bf16)x[1], (bf16)x[2], (bf16)x[3]};
    };
#pragma unroll
    for (int q = 0; q < N4; ++q)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        put(64 * q + 16 * g + 4 * i, f32x4{b[4 * q][i], b[4 * q + 1][i], b[4 * q + 2][i], b[4 * q + 3][i]});
    if constexpr (N2 > 0) {
#pragma unroll
      for (int v = 0; v < 2; ++v)
        put(64 * N4 + 8 * g + 4 * v, f32x4{b[4 * N4][2 * v], b[4 * N4 + 1][2 * v], b[4 * N4][2 * v + 1], b[4 * N4 + 1][2 * v + 1]});
    }
    return z;
  }
};

template <typename E, int DP>
struct Cols {
  static constexpr int N4 = Blocks<DP>::N4, N2 = Blocks<DP>::N2;
  f32x4 v4[N4 > 0 ? N4 : 1][4];
  f32x2 v2[4];
  // columns past d repeat valid ones: what they produce is not stored
  __device__ __forceinline__ void load(const E *base, int64_t ld, int first, int rows, int d, int g, int r) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int row = first + 4 * g + e < rows ? first + 4 * g + e : rows - 1;
      const E *p = base + row * ld;
#pragma unroll
      for (int q = 0; q < N4; ++q) {
        const int col = 64 * q + 4 * r;
        v4[q][e] = load4(p + (64 * q + 64 <= DP - 32 || col < d ? col : 0));
      }
      if constexpr (N2 > 0) {
        const int col = 64 * N4 + 2 * r;
        const E *pp = p + (col < d ? col : 0);
        if constexpr (sizeof(E) == 4) {
          v2[e] = *reinterpret_cast<const f32x2 *>(pp);
        } else {
          typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
          const bf16x2 t = *reinterpret_cast<const bf16x2 *>(pp);
          v2[e] = f32x2{(float)t[0], (float)t[1]};
        }
      }
    }
  }
  // acc += this^T x, x: element e belongs to row 4 g + e of the block
  __device__ __forceinline__ void accumulate(Blocks<DP> &acc, const f32x4 &x) const {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
#pragma unroll
      for (int q = 0; q < N4; ++q)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc.b[4 * q + b] = MFMA4(v4[q][e][b], x[e], acc.b[4 * q + b]);
      if constexpr (N2 > 0) {
#pragma unroll
        for (int b = 0; b < 2; ++b) acc.b[4 * N4 + b] = MFMA4(v2[e][b], x[e], acc.b[4 * N4 + b]);
      }
    }
  }
};

template <typename E, int DP>
__device__ __forceinline__ f32x4 product(const Rows<E, DP> &streamed, const Rows<E, DP> &own) {
  f32x4 lo = {0.0f, 0.0f, 0.0f, 0.0f}, hi = {0.0f, 0.0f, 0.0f, 0.0f};   // two chains: an MFMA waits for its accumulator
#pragma unroll
  for (int c = 0; c < Rows<E, DP>::NC; ++c) {
    if constexpr (sizeof(E) == 2) {
      lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(streamed.v[c], own.v[c], lo, 0, 0, 0);
    } else {
#pragma unroll
      for (int e = 0; e < 4; e += 2) {
        lo = MFMA4(streamed.v[c][e], own.v[c][e], lo);
        hi = MFMA4(streamed.v[c][e + 1], own.v[c][e + 1], hi);
      }
    }
  }
  return lo + hi;
}

__device__ __forceinline__ float quad_max(float v) {
  v = fmaxf(v, __shfl_xor(v, 16, 64));
  return fmaxf(v, __shfl_xor(v, 32, 64));
}

// Grid: (heads, blocks of rows, batch).  A wave owns rows row0 .. row0 + 15 and takes part `part` of the other side's steps.
// A workgroup owns 64 rows, 16 to a wave, or (SPLIT) 16, of which every wave takes a quarter of the steps (every fourth one); the
// partial results meet in LDS.
template <bool SPLIT>
struct Where {
  int lane, g, r, row0, part, head, batch;
  __device__ __forceinline__ Where(int blk) {   // blk: of the head's blocks of rows
    lane = threadIdx.x & 63;
    g = lane >> 4;
    r = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    row0 = SPLIT ? blk * 16 : blk * 64 + 16 * wave;
    part = SPLIT ? wave : 0;
    head = blockIdx.x;
    batch = blockIdx.z;
  }
};
template <int DP>
struct Meeting {
  f32x4 slot[3][Blocks<DP>::N][64];
  __device__ __forceinline__ void add(Blocks<DP> &x, int part, int lane) {   // the sum of all parts, in part 0
    if (part > 0) {
#pragma unroll
      for (int i = 0; i < Blocks<DP>::N; ++i) slot[part - 1][i][lane] = x.b[i];
    }
    __syncthreads();
    if (part > 0) return;
#pragma unroll
    for (int i = 0; i < Blocks<DP>::N; ++i) x.b[i] = (x.b[i] + slot[0][i][lane]) + (slot[1][i][lane] + slot[2][i][lane]);
  }
};

template <typename E, int DP, bool SPLIT>
__global__ __launch_bounds__(256) void attn_fwd_f32_kernel(int s, int n, int d, float scale, const E *__restrict__ qkv,
                                                           E *__restrict__ a, float *__restrict__ lse) {
  const Where<SPLIT> w(gridDim.y - 1 - blockIdx.y);
  constexpr int STRIDE = SPLIT ? 128 : 32;
  const int first = 32 * w.part;
  if (w.row0 >= s) return;
  const int64_t ld = (int64_t)n * 3 * d;
  const E *base = qkv + (int64_t)w.batch * s * ld + (int64_t)w.head * 3 * d;
  const int q = w.row0 + w.r;
  Rows<E, DP> qf, kf[2];
  qf.load(base, ld, w.row0, s, d, w.g, w.r);
  const int last = w.row0 + 15 < s ? w.row0 + 15 : s - 1;   // last key any row of the wave sees
#pragma unroll
  for (int kb = 0; kb < 2; ++kb) kf[kb].load(base + d, ld, first + 16 * kb, s, d, w.g, w.r);
  constexpr bool PARTS = sizeof(E) == 4;
  Blocks<DP> o, total;
  o.clear();
  if constexpr (PARTS) total.clear();
  float m = -INFINITY, l = 0.0f;   // l: this lane's share of the row sum
  for (int k0 = first; k0 <= last; k0 += STRIDE) {
    Cols<E, DP> vf[2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) vf[kb].load(base + 2 * d, ld, k0 + 16 * kb, s, d, w.g, w.r);
    f32x4 p[2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) p[kb] = product(kf[kb], qf) * scale;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) kf[kb].load(base + d, ld, k0 + STRIDE + 16 * kb, s, d, w.g, w.r);   // of the next step
    float mx = -INFINITY;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (k0 + 16 * kb + 4 * w.g + i > q) p[kb][i] = -INFINITY;
        mx = fmaxf(mx, p[kb][i]);
      }
    const float m_new = fmaxf(m, quad_max(mx));   // finite: key 0 is never masked, but for a part that has seen none of a row's keys
    const float shift = SPLIT && m_new == -INFINITY ? 0.0f : m_new;
    const float alpha = expf(m - shift);
    float sum = 0.0f;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        p[kb][i] = expf(p[kb][i] - shift);
        sum += p[kb][i];
      }
    l = l * alpha + sum;
    m = m_new;
    if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
      for (int i = 0; i < Blocks<DP>::N; ++i) {
        o.b[i] *= alpha;
        if constexpr (PARTS) total.b[i] *= alpha;
      }
    }
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) vf[kb].accumulate(o, p[kb]);
    if constexpr (PARTS)
      if ((k0 / STRIDE + 1) % (sum_rows(SPLIT) / 32) == 0) total.flush(o);
  }
  if constexpr (PARTS) o.flush(total);
  l = quad_sum(l);
  if constexpr (SPLIT) {   // every part's sums relative to the maximum of all
    __shared__ float stat[2][4][16];
    __shared__ Meeting<DP> meet;
    if (w.g == 0) {
      stat[0][w.part][w.r] = m;
      stat[1][w.part][w.r] = l;
    }
    __syncthreads();
    float top = -INFINITY;
#pragma unroll
    for (int i = 0; i < 4; ++i) top = fmaxf(top, stat[0][i][w.r]);
    l = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i) l = fmaf(stat[1][i][w.r], expf(stat[0][i][w.r] - top), l);
    const float mul = expf(m - top);
    m = top;
#pragma unroll
    for (int i = 0; i < Blocks<DP>::N; ++i) o.b[i] *= mul;
    meet.add(o, w.part, w.lane);
    if (w.part > 0) return;
  }
  E *out = a + ((int64_t)w.batch * s + q) * ((int64_t)n * d) + (int64_t)w.head * d;
  float *out_lse = lse + ((int64_t)w.batch * n + w.head) * s + q;
  float z = 0.0f;
  if (q < s) {
    z = o.store(out, d, 1.0f / l, w.g);
    if (w.g == 0) *out_lse = m + logf(l);
  }
  if (all_finite(z)) return;
  redo_fwd<E, DP>(base, ld, s, d, scale, q, last, w.g, out, out_lse);
}

// dq, and D for the kernel below.  meet: SPLIT only, like everywhere
template <typename E, int DP, bool SPLIT>
__device__ __forceinline__ void dq_rows(int blk, Meeting<DP> *meet, int s, int n, int d, float scale, const E *__restrict__ qkv,
                                        const E *__restrict__ a, const float *__restrict__ lse, const E *__restrict__ da,
                                        E *__restrict__ dqkv, float *__restrict__ D) {
  const Where<SPLIT> w(blk);
  constexpr int STRIDE = SPLIT ? 64 : 16;
  const int first = 16 * w.part;
  if (w.row0 >= s) return;
  const int64_t ld = (int64_t)n * 3 * d, pld = (int64_t)n * d;
  const E *base = qkv + (int64_t)w.batch * s * ld + (int64_t)w.head * 3 * d;
  const int64_t po = (int64_t)w.batch * s * pld + (int64_t)w.head * d, st = ((int64_t)w.batch * n + w.head) * s;
  const int q = w.row0 + w.r, qc = q < s ? q : s - 1;
  Rows<E, DP> qf, dof, kf, vf;
  float dsum;
  {  // D on the diagonal of dO a^T, by the same MFMAs as dP: where a row has one key (a = v) the two cancel exactly
    Rows<E, DP> af;
    af.load(a + po, pld, w.row0, s, d, w.g, w.r);
    dof.load(da + po, pld, w.row0, s, d, w.g, w.r);
    const f32x4 t = product(af, dof);
    const float mine = (w.r & 2) ? ((w.r & 1) ? t[3] : t[2]) : ((w.r & 1) ? t[1] : t[0]);
    dsum = __shfl(mine, 16 * (w.r >> 2) + w.r, 64);
  }
  if (q < s && w.g == 0 && w.part == 0) D[st + q] = dsum;
  qf.load(base, ld, w.row0, s, d, w.g, w.r);
  const float ls = lse[st + qc];
  const int last = w.row0 + 15 < s ? w.row0 + 15 : s - 1;
  kf.load(base + d, ld, first, s, d, w.g, w.r);
  vf.load(base + 2 * d, ld, first, s, d, w.g, w.r);
  constexpr bool PARTS = sizeof(E) == 4;
  Blocks<DP> dq, total;
  dq.clear();
  if constexpr (PARTS) total.clear();
  for (int k0 = first; k0 <= last; k0 += STRIDE) {
    Cols<E, DP> kc;
    kc.load(base + d, ld, k0, s, d, w.g, w.r);
    const f32x4 sc = product(kf, qf) * scale, dp = product(vf, dof);
    kf.load(base + d, ld, k0 + STRIDE, s, d, w.g, w.r);   // of the next step
    vf.load(base + 2 * d, ld, k0 + STRIDE, s, d, w.g, w.r);
    f32x4 ds;
#pragma unroll
    for (int i = 0; i < 4; ++i) ds[i] = k0 + 4 * w.g + i > q ? 0.0f : expf(sc[i] - ls) * (dp[i] - dsum);
    kc.accumulate(dq, ds);
    if constexpr (PARTS)
      if ((k0 / STRIDE + 1) % (sum_rows(SPLIT) / 16) == 0) total.flush(dq);
  }
  if constexpr (PARTS) dq.flush(total);
  if constexpr (SPLIT) {
    meet->add(dq, w.part, w.lane);
    if (w.part > 0) return;
  }
  E *out = dqkv + ((int64_t)w.batch * s + q) * ld + (int64_t)w.head * 3 * d;
  float z = 0.0f;
  if (q < s) z = dq.store(out, d, scale, w.g);
  if (all_finite(z)) return;
  redo_dq<E, DP>(base, ld, da + po, pld, s, d, scale, q, last, ls, dsum, w.g, out);
}

// What the compiler is told about waves per SIMD, so that it uses registers as the loop needs them: bf16, head sizes up to 32: 3-4,
// accumulators in ordinary registers (16 heads of 24, s = 1024: dq + dk/dv 97 us, 90 so); up to 64: no more than 2, else 20 more values
// go to and fro between the two kinds of register (16 heads of 56, s = 1024: 137 us, 134 so).
template <typename E, int DP>
constexpr int dkv_waves(int most) {
  if (sizeof(E) == 2 && DP == 32) return most ? 4 : 3;
  if (sizeof(E) == 2 && DP == 64) return most ? 2 : 1;
  return most ? 8 : 1;
}
// OWN_D: D is not read; it is the diagonal of dO a^T by the MFMAs that give dP, as in the dq kernel.
template <typename E, int DP, bool SPLIT, bool OWN_D>
__device__ __forceinline__ void dkv_rows(int blk, Meeting<DP> *meet, int s, int n, int d, float scale, const E *__restrict__ qkv,
                                         const E *__restrict__ a, const float *__restrict__ lse, const float *__restrict__ D,
                                         const E *__restrict__ da, E *__restrict__ dqkv) {
  const Where<SPLIT> w(blk);
  constexpr int STRIDE = SPLIT ? 64 : 16;
  const int first = w.row0 + 16 * w.part;
  if (w.row0 >= s) return;
  const int64_t ld = (int64_t)n * 3 * d, pld = (int64_t)n * d;
  const E *base = qkv + (int64_t)w.batch * s * ld + (int64_t)w.head * 3 * d;
  const E *dab = da + (int64_t)w.batch * s * pld + (int64_t)w.head * d, *ab = a + (int64_t)w.batch * s * pld + (int64_t)w.head * d;
  const int64_t st = ((int64_t)w.batch * n + w.head) * s;
  const int key = w.row0 + w.r;
  Rows<E, DP> kf, vf, qf, of, af;
  kf.load(base + d, ld, w.row0, s, d, w.g, w.r);
  vf.load(base + 2 * d, ld, w.row0, s, d, w.g, w.r);
  constexpr bool PARTS = sizeof(E) == 4;
  Blocks<DP> dk, dv, tk, tv;
  dk.clear();
  dv.clear();
  if constexpr (PARTS) {
    tk.clear();
    tv.clear();
  }
  qf.load(base, ld, first, s, d, w.g, w.r);
  of.load(dab, pld, first, s, d, w.g, w.r);
  if constexpr (OWN_D) af.load(ab, pld, first, s, d, w.g, w.r);
  for (int q0 = first; q0 < s; q0 += STRIDE) {
    Cols<E, DP> oc, qcol;
    oc.load(dab, pld, q0, s, d, w.g, w.r);
    qcol.load(base, ld, q0, s, d, w.g, w.r);
    float ls[4], dd[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int q = q0 + 4 * w.g + i < s ? q0 + 4 * w.g + i : s - 1;
      ls[i] = lse[st + q];
      if constexpr (!OWN_D) dd[i] = D[st + q];
    }
    if constexpr (OWN_D) {
      const f32x4 t = product(of, af);
#pragma unroll
      for (int i = 0; i < 4; ++i) dd[i] = __shfl(t[i], 20 * w.g + i, 64);
      af.load(ab, pld, q0 + STRIDE, s, d, w.g, w.r);
    }
    const f32x4 sc = product(qf, kf) * scale, dp = product(of, vf);
    qf.load(base, ld, q0 + STRIDE, s, d, w.g, w.r);   // of the next step
    of.load(dab, pld, q0 + STRIDE, s, d, w.g, w.r);
    f32x4 p, ds;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int q = q0 + 4 * w.g + i;
      p[i] = q < key || q >= s ? 0.0f : expf(sc[i] - ls[i]);
      ds[i] = p[i] * (dp[i] - dd[i]);
    }
    oc.accumulate(dv, p);
    qcol.accumulate(dk, ds);
    if constexpr (PARTS)
      if ((q0 / STRIDE + 1) % (sum_rows(SPLIT) / 16) == 0) {
        tk.flush(dk);
        tv.flush(dv);
      }
  }
  if constexpr (PARTS) {
    dk.flush(tk);
    dv.flush(tv);
  }
  if constexpr (SPLIT) {
    meet->add(dk, w.part, w.lane);
    __syncthreads();
    meet->add(dv, w.part, w.lane);
    if (w.part > 0) return;
  }
  E *out = dqkv + ((int64_t)w.batch * s + key) * ld + (int64_t)w.head * 3 * d;
  float z = 0.0f;
  if (key < s) z = dk.store(out + d, d, scale, w.g) + dv.store(out + 2 * d, d, 1.0f, w.g);
  if (all_finite(z)) return;
  redo_dv<E, DP>(base, ld, dab, pld, s, d, scale, w.row0, key, lse + st, w.g, out);
  if constexpr (OWN_D) redo_dk<E, DP>(base, ld, dab, pld, s, d, scale, w.row0, key, lse + st, [&](int t) { return dot(dab + t * pld, ab + t * pld, d, w.g); }, w.g, out);
  else redo_dk<E, DP>(base, ld, dab, pld, s, d, scale, w.row0, key, lse + st, [&](int t) { return D[st + t]; }, w.g, out);
}

template <typename E>
struct BackwardArgs {
  int s, n, d;
  float scale;
  const E *qkv, *a;
  const float *lse;
  const E *da;
  E *dqkv;
  float *D;
};
template <int DP, bool SPLIT>
__device__ __forceinline__ Meeting<DP> *meeting_place() {
  if constexpr (SPLIT) {
    __shared__ Meeting<DP> meet;
    return &meet;
  }
  return nullptr;
}
// (fp32, small head sizes: two waves per SIMD are asked for, with which the compiler keeps the accumulators in ordinary registers
// instead of copying them at every step; 2 x 512 x 16 heads of 64, dq: 3 us less, 1 x 1990 x 16 of 32: 9 us less.)
template <typename E, int DP, bool SPLIT>
__global__ __launch_bounds__(256, sizeof(E) == 4 && DP <= 64 ? 2 : 1) void attn_bwd_dq_f32_kernel(BackwardArgs<E> x) {
  dq_rows<E, DP, SPLIT>(gridDim.y - 1 - blockIdx.y, meeting_place<DP, SPLIT>(), x.s, x.n, x.d, x.scale, x.qkv, x.a, x.lse, x.da, x.dqkv, x.D);
}
template <typename E, int DP, bool SPLIT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(dkv_waves<E, DP>(0), dkv_waves<E, DP>(1)))) void attn_bwd_dkv_f32_kernel(BackwardArgs<E> x) {
  dkv_rows<E, DP, SPLIT, false>(blockIdx.y, meeting_place<DP, SPLIT>(), x.s, x.n, x.d, x.scale, x.qkv, x.a, x.lse, x.D, x.da, x.dqkv);
}
// Both in one launch, for calls that split the streamed side (one_launch_groups says which): the first half of the blocks are dk / dv, with a D of
// their own.
template <typename E, int DP>
__global__ __launch_bounds__(256, DP <= (sizeof(E) == 4 ? 96 : 128) ? 2 : 1) void attn_bwd_f32_kernel(BackwardArgs<E> x) {
  Meeting<DP> *meet = meeting_place<DP, true>();
  const int half = gridDim.y / 2, blk = blockIdx.y;
  if (blk < half) dkv_rows<E, DP, true, true>(blk, meet, x.s, x.n, x.d, x.scale, x.qkv, x.a, x.lse, nullptr, x.da, x.dqkv);
  else dq_rows<E, DP, true>(2 * half - 1 - blk, meet, x.s, x.n, x.d, x.scale, x.qkv, x.a, x.lse, x.da, x.dqkv, x.D);
}

// Up to how many groups of 16 rows the backward kernels of a call that splits the streamed side go out in one launch.  us, two launches / one, fp32:
// 1 x 257 x 2 heads of 64 22.0 / 15.3, 2 x 300 x 2 of 128 43.8 / 28.9; by groups: up to 128 1.2 to 1.8 times as fast, 256 1.06 to 1.3, and 512 1.07
// to 1.19 up to head size 96, 0.91 at 128; at 160 1.0 for 256, 0.82 for 512; above 192 the registers run out (0.5 to 1.1).
// bf16: 128 x 32 of 96 15.3 / 11.6, 128 x 16 of 184 24.9 / 16.4, 256 x 8 of 256 46 / 31; 512 x 16 of 232 (512 groups) 97.8 / 103.9.
template <typename E, int DP>
constexpr int one_launch_groups() {
  if (sizeof(E) == 2) return DP <= 96 ? 256 : 128;
  return DP <= 96 ? 512 : DP == 128 ? 256 : DP == 160 ? 128 : 0;
}

// Up to how many groups of 16 rows a call splits the streamed side over the waves of a workgroup.  With 64 rows to a workgroup, 16 to a wave, the
// time is the longest wave's chain of steps until there are several waves to a SIMD, and it grows with s; with 16 rows to a workgroup a chain is a quarter of that, but
// the waves no longer share what they load, and the time grows with the work.  So the line lies higher for longer sequences and smaller head sizes; and lower for one
// sequence, whose workgroups start in the order of falling work (of several, the last one's longest wait for all of the others), least of all with a number of heads that is
// no multiple of 8.  Lines by 3789 sizes (head size 16 to 256, s 48 to 4096, 512 to 4600 groups, 1 to 4 sequences, even and odd numbers of heads).  fp32, times as
// fast with 16 rows to a workgroup, before a line and beyond it, one sequence: forward, head size 32, s = 768, 2560 groups 1.13, 4080 0.85; 64, s = 320, 760 1.33, 1020 0.97 to
// 1.07; s = 1024, 1536 1.39, 2496 0.84; 128, s = 512, 768 1.33, 1024 0.92 to 1.08; 256, s = 2048, 1280 1.12, 1536 0.94 to 0.98; backward, 64, s = 512, 2048 1.12, 4064 0.87;
// 256, s = 553, 720 1.5, 1015 0.95.  Several: 4 x 728 tokens, 20 heads of 32 (3680) 1.60, backward 1.53; 2 x 1336, 14 of 64 (2352) 1.36; 4 x 1309, 11 of 48 (3608) backward
// 1.39.  Up to 512 groups at any s above 32 (1 head of 256, s = 256 81.9 -> 28.1 us, 247 -> 87); at s <= 32 there is nothing to share.  bf16 comes here with more groups
// only above head size 192 and in calls that the tiled kernels refuse.  2 x 512 tokens, 16 heads of 64, fp32: 35.5 -> 29.4 us, 118 -> 85.
template <typename E, int DP, bool BACKWARD>
constexpr int64_t most_split_groups(int b, int s) {
  if (s <= 32) return 0;
  if (sizeof(E) == 2) return 512;
  const bool one = b == 1;
  if (!BACKWARD) {
    if (DP == 32) return s >= (one ? 2048 : 512) ? 4096 : s >= 768 ? 3584 : s >= 512 ? 3072 : s >= 192 ? 1024 : 512;
    if (DP <= 96) return s >= (one ? 1536 : 1024) ? 2560 : s >= 1024 ? 2048 : s >= 512 ? 1536 : s >= (one ? 384 : 256) ? 1024 : s >= 256 ? 960 : s >= 192 ? 768 : 512;
    return s >= 2048 ? (one && DP > 224 ? 1280 : 1536) : s >= (one ? 768 : 512) ? 1024 : s >= 512 ? 960 : s >= 256 ? 768 : 512;
  }
  if (DP == 32) return s >= (one ? 768 : 512) ? 4096 : s >= 512 ? 3584 : s >= 128 ? 1024 : 512;
  if (DP == 64) return s >= (one ? 1536 : 512) ? 4096 : s >= 1024 ? 3584 : s >= 768 ? 3072 : s >= 512 ? 2560 : s >= 128 ? 1024 : 512;
  if (DP == 96) return s >= 1024 ? 2048 : s >= 512 ? 1536 : s >= 192 ? 1024 : 512;
  if (DP <= 160) return s >= 1024 ? 1536 : s >= 256 ? 1024 : s >= 192 ? 768 : 512;
  return s >= (one ? 768 : 512) ? 1024 : s >= 512 ? 960 : s >= 256 ? 768 : 512;
}
template <typename E, int DP, bool BACKWARD>
bool splits(int b, int s, int n) { return (int64_t)b * n * ((s + 15) / 16) <= most_split_groups<E, DP, BACKWARD>(b, s); }

template <typename E, int DP, bool SPLIT>
int fwd_launch_s(int b, int s, int n, int d, float scale, const void *qkv, void *a, float *lse, hipStream_t st) {
  const dim3 grid(n, SPLIT ? (s + 15) / 16 : (s + 63) / 64, b);
  LaunchScope scope(MTNLG_K_ATTN_FWD, st);
  attn_fwd_f32_kernel<E, DP, SPLIT><<<grid, 256, 0, st>>>(s, n, d, scale, (const E *)qkv, (E *)a, lse);
  return check_launch();
}
template <typename E, int DP>
int fwd_launch(int b, int s, int n, int d, float scale, const void *qkv, void *a, float *lse, hipStream_t st) {
  if (splits<E, DP, false>(b, s, n)) return fwd_launch_s<E, DP, true>(b, s, n, d, scale, qkv, a, lse, st);
  return fwd_launch_s<E, DP, false>(b, s, n, d, scale, qkv, a, lse, st);
}

template <typename E, int DP, bool SPLIT>
int bwd_launch_s(int b, int s, int n, int d, float scale, const void *qkv, const void *a, const float *lse, const void *da,
                 void *dqkv, void *ws, hipStream_t st) {
  const BackwardArgs<E> x{s, n, d, scale, (const E *)qkv, (const E *)a, lse, (const E *)da, (E *)dqkv, (float *)ws};
  dim3 grid(n, SPLIT ? (s + 15) / 16 : (s + 63) / 64, b);
  LaunchScope scope(MTNLG_K_ATTN_BWD, st);
  if constexpr (SPLIT && one_launch_groups<E, DP>() > 0) {
    if ((int64_t)b * n * ((s + 15) / 16) <= one_launch_groups<E, DP>()) {
      grid.y *= 2;
      attn_bwd_f32_kernel<E, DP><<<grid, 256, 0, st>>>(x);
      return check_launch();
    }
  }
  attn_bwd_dq_f32_kernel<E, DP, SPLIT><<<grid, 256, 0, st>>>(x);
  MTNLG_TRY(check_launch());
  attn_bwd_dkv_f32_kernel<E, DP, SPLIT><<<grid, 256, 0, st>>>(x);
  return check_launch();
}
template <typename E, int DP>
int bwd_launch(int b, int s, int n, int d, float scale, const void *qkv, const void *a, const float *lse, const void *da,
               void *dqkv, void *ws, hipStream_t st) {
  if (splits<E, DP, true>(b, s, n)) return bwd_launch_s<E, DP, true>(b, s, n, d, scale, qkv, a, lse, da, dqkv, ws, st);
  return bwd_launch_s<E, DP, false>(b, s, n, d, scale, qkv, a, lse, da, dqkv, ws, st);
}

// fn<E, DP>, DP: the head size rounded up to a multiple of 32
#define BY_HEAD_SIZE(fn, E, ...)                       \
  switch ((d + 31) / 32) {                             \
    case 1: return fn<E, 32>(__VA_ARGS__);             \
    case 2: return fn<E, 64>(__VA_ARGS__);             \
    case 3: return fn<E, 96>(__VA_ARGS__);             \
    case 4: return fn<E, 128>(__VA_ARGS__);            \
    case 5: return fn<E, 160>(__VA_ARGS__);            \
    case 6: return fn<E, 192>(__VA_ARGS__);            \
    case 7: return fn<E, 224>(__VA_ARGS__);            \
    case 8: return fn<E, 256>(__VA_ARGS__);            \
    default: return MTNLG_UNSUPPORTED_SHAPE;           \
  }

}  // namespace

int attention_fwd_f32(int dtype, int b, int s, int n, int d, float scale, const void *qkv, void *a,
                      float *lse, hipStream_t stream) {
  if (d % 8 || d > 256 || s > ATTENTION_F32_MAX_SEQ || n > 65535 || b > 65535)
    return MTNLG_UNSUPPORTED_SHAPE;
  if (dtype == MTNLG_F32) BY_HEAD_SIZE(fwd_launch, float, b, s, n, d, scale, qkv, a, lse, stream)
  if (dtype == MTNLG_BF16) BY_HEAD_SIZE(fwd_launch, bf16, b, s, n, d, scale, qkv, a, lse, stream)
  return MTNLG_INVALID_ARG;
}

int attention_bwd_f32(int dtype, int b, int s, int n, int d, float scale, const void *qkv,
                      const void *a, const float *lse, const void *da, void *dqkv, void *ws,
                      hipStream_t stream) {
  if (d % 8 || d > 256 || s > ATTENTION_F32_MAX_SEQ || n > 65535 || b > 65535)
    return MTNLG_UNSUPPORTED_SHAPE;
  if (dtype == MTNLG_F32) BY_HEAD_SIZE(bwd_launch, float, b, s, n, d, scale, qkv, a, lse, da, dqkv, ws, stream)
  if (dtype == MTNLG_BF16) BY_HEAD_SIZE(bwd_launch, bf16, b, s, n, d, scale, qkv, a, lse, da, dqkv, ws, stream)
  return MTNLG_INVALID_ARG;
}

}  // namespace mtnlg
