// GEMM on the fp32 matrix instructions (v_mfma_f32_16x16x4_f32): the fp32 path of the library, and the bf16 problems
// whose row lengths the bf16 kernels do not take (their elements are widened on load, which is exact).  Any M, N, K, any layout.
//
// What bounds it: the fp32 matrix rate (256 FLOP per clock and compute unit, a sixteenth of bf16), as long as there are
// enough waves; below that the chain global memory -> registers -> MFMA of one wave.  At that rate an LDS tile buys
// nothing: a 64 x 64 wave tile needs 8 KB of operands per 2048 cycles of MFMA, which the caches deliver, so the
// fragments are loaded straight into the registers the MFMAs read, DEPTH chunks of 16 k ahead, with no barrier in
// the loop.  The K axis of a workgroup's tile may be split over its waves (WGK); their partial tiles are added
// through LDS in a fixed order, so a small M x N still fills the chip and a long K is a short chain.
//   Chunk of 16 KH k: lane l = 16 g + r supplies k = 16 h + 4 g + e in MFMA 4 h + e (the k order inside a chunk is free as
//   long as both operands agree).  KH = 2 takes both 64-byte halves of a K-contiguous line together: taken one chunk
//   apart, the second half had often left the L1 cache (NT 1024 x 3072 x 1024 one chunk in flight: 96 -> 88 us).
//   K-contiguous operand: lane loads 4 consecutive k of row r of each 16-row block.
//   Row-contiguous operand ([k][row]): lane loads NB consecutive rows NB r .. + NB - 1 at each of its 4 k; block b of
//   the wave tile is then rows NB r + b, and the epilogue undoes that.
// The MFMA takes the B fragment first, so a lane holds 4 NB consecutive columns (or NB runs of 4) of one row.
#include "common.h"

namespace mtnlg {

namespace {

struct F32GemmArgs {
  int64_t M, N, K, lda, ldb;
  const void *A, *B;
  void *C;
  EpiArgs ea;
  int tiles_m, tiles_n;
};

template <typename E, int NB>
__device__ __forceinline__ void load_rows(const E *p, float (&out)[NB]) {
  if constexpr (NB == 4) {
    const f32x4 t = load4(p);
#pragma unroll
    for (int b = 0; b < 4; ++b) out[b] = t[b];
  } else {
    static_assert(NB == 2, "wave tiles of 2 or 4 blocks a side");
    if constexpr (sizeof(E) == 4) {
      typedef __attribute__((ext_vector_type(2))) float f32x2;
      const f32x2 t = *reinterpret_cast<const f32x2 *>(p);
      out[0] = t[0];
      out[1] = t[1];
    } else {
      typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
      const bf16x2 t = *reinterpret_cast<const bf16x2 *>(p);
      out[0] = (float)t[0];
      out[1] = (float)t[1];
    }
  }
}

// One operand's fragments of a chunk: v[block][e].  first: this wave's first row; rows: rows of the whole operand.
// Rows past the end repeat the last one (their results are not stored); k past the end repeats K - 1 and is zeroed by
// clear_tail before use.
template <typename E, int NB, int KH, bool ROWC, bool VEC>
struct Frag {
  float v[NB][4 * KH];
  __device__ __forceinline__ void fetch(const E *base, int64_t ld, int64_t first, int64_t rows, int64_t k0, int64_t K,
                                        int g, int r) {
    if constexpr (!ROWC) {
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        int64_t row = first + 16 * b + r;
        if (row >= rows) row = rows - 1;
        const E *p = base + row * ld;
#pragma unroll
        for (int h = 0; h < KH; ++h) {
          const int64_t k = k0 + 16 * h + 4 * g;
          if constexpr (VEC) {   // K is a multiple of 4
            const f32x4 t = load4(p + (k < K ? k : K - 4));
#pragma unroll
            for (int e = 0; e < 4; ++e) v[b][4 * h + e] = t[e];
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[b][4 * h + e] = to_f32(p[k + e < K ? k + e : K - 1]);
          }
        }
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4 * KH; ++e) {
        const int64_t k = k0 + 16 * (e >> 2) + 4 * g + (e & 3);
        const E *p = base + (k < K ? k : K - 1) * ld;
        int64_t row = first + NB * r;
        if constexpr (VEC) {   // rows is a multiple of 4
          if (row >= rows) row = rows - NB;
          float t[NB];
          load_rows<E, NB>(p + row, t);
#pragma unroll
          for (int b = 0; b < NB; ++b) v[b][e] = t[b];
        } else {
#pragma unroll
          for (int b = 0; b < NB; ++b) v[b][e] = to_f32(p[row + b < rows ? row + b : rows - 1]);
        }
      }
    }
  }
  __device__ __forceinline__ void clear_tail(int64_t k0, int64_t K, int g) {
#pragma unroll
    for (int e = 0; e < 4 * KH; ++e)
      if (k0 + 16 * (e >> 2) + 4 * g + (e & 3) >= K) {
#pragma unroll
        for (int b = 0; b < NB; ++b) v[b][e] = 0.0f;
      }
  }
};

// 4 consecutive outputs of row m at column n (n + 3 < N and everything aligned for 4-element accesses)
template <typename E>
__device__ __forceinline__ void epilogue4(const EpiArgs &ea, void *C, int64_t N, int64_t m, int64_t n, f32x4 v) {
  const int64_t off = m * N + n;
  if (ea.flags & MTNLG_EPI_BIAS) v += load4(static_cast<const E *>(ea.bias) + n);
  auto put = [&](E *p, f32x4 x) {
    if constexpr (sizeof(E) == 4) *reinterpret_cast<f32x4 *>(p) = x;
    else *reinterpret_cast<bf16x4 *>(p) = bf16x4{(bf16)x[0], (bf16)x[1], (bf16)x[2], (bf16)x[3]};
  };
  if (ea.flags & MTNLG_EPI_GELU) {
    put(static_cast<E *>(ea.aux) + off, v);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = gelu_f(v[e], (ea.flags & MTNLG_EPI_GELU_ERF) != 0);
  }
  if (ea.flags & (MTNLG_EPI_RESIDUAL | MTNLG_EPI_GELU_GRAD)) {
    const f32x4 t = load4(static_cast<const E *>(ea.aux) + off);
    if (ea.flags & MTNLG_EPI_RESIDUAL) {
      v += t;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] *= gelu_grad_f(t[e], (ea.flags & MTNLG_EPI_GELU_ERF) != 0);
    }
  }
  if (ea.flags & MTNLG_EPI_OUT_F32) {
    float *c = static_cast<float *>(C) + off;
    if (ea.flags & MTNLG_EPI_ACCUMULATE) v += load4(c);
    *reinterpret_cast<f32x4 *>(c) = v;
  } else {
    E *c = static_cast<E *>(C) + off;
    if (ea.flags & MTNLG_EPI_ACCUMULATE) v += load4(c);
    put(c, v);
  }
}

// Workgroup of WGM x WGN x WGK waves, wave tile 16 TMB x 16 TNB.  VEC: every row length is a multiple of 4 elements and
// every pointer aligned to 4 elements.
template <typename E, int TMB, int TNB, int WGM, int WGN, int WGK, int KH, int DEPTH, bool AT, bool BT, bool VEC>
__global__ __launch_bounds__(64 * WGM * WGN * WGK) void gemm_f32_kernel(F32GemmArgs a) {
  constexpr int NV = TMB * TNB;   // vectors of 4 columns a lane holds
  __shared__ f32x4 red[WGK > 1 ? WGK * WGM * WGN * NV * 64 : 1];
  const int lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wk = wave % WGK, wt = wave / WGK, wm = wt / WGN, wn = wt % WGN;

  // XCD x (workgroup id mod 8) takes a contiguous run of tiles, ordered in blocks of 8 row tiles
  const int tiles = a.tiles_m * a.tiles_n, per_xcd = (tiles + 7) / 8;
  const int pid = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per_xcd || pid >= tiles) return;
  const int per_group = 8 * a.tiles_n, grp = pid / per_group, first_m = grp * 8;
  const int gsz = a.tiles_m - first_m < 8 ? a.tiles_m - first_m : 8;
  const int tm = first_m + (pid % per_group) % gsz, tn = (pid % per_group) / gsz;
  const int64_t m0 = ((int64_t)tm * WGM + wm) * (16 * TMB), n0 = ((int64_t)tn * WGN + wn) * (16 * TNB);

  const E *A = static_cast<const E *>(a.A), *B = static_cast<const E *>(a.B);
  const int nc_all = (int)((a.K + 16 * KH - 1) / (16 * KH)), per = (nc_all + WGK - 1) / WGK;
  const int c0 = wk * per, c1 = c0 + per < nc_all ? c0 + per : nc_all;   // this wave's chunks

  f32x4 acc[TMB][TNB];
#pragma unroll
  for (int i = 0; i < TMB; ++i)
#pragma unroll
    for (int j = 0; j < TNB; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  Frag<E, TMB, KH, AT, VEC> af[DEPTH];
  Frag<E, TNB, KH, BT, VEC> bf[DEPTH];
  // Every condition in the loop is the same for the whole wave and held in a scalar register, and the first fetches are
  // unconditional (clamped): fragments that are fetched on some paths only, under a condition the compiler takes for
  // divergent, were miscompiled (accumulators placed over live fragments).
  auto fetch = [&](int d, int c) {
    const int64_t k0 = (int64_t)(c < nc_all ? c : nc_all - 1) * (16 * KH);
    af[d].fetch(A, a.lda, m0, a.M, k0, a.K, g, r);
    bf[d].fetch(B, a.ldb, n0, a.N, k0, a.K, g, r);
  };
#pragma unroll
  for (int d = 0; d < DEPTH; ++d) fetch(d, c0 + d);
  for (int c = c0; c < c1; c += DEPTH) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
      if (c + d < c1) {
        const int64_t k0 = (int64_t)(c + d) * (16 * KH);
        if (k0 + 16 * KH > a.K) {   // uniform: the last chunk of a K that is no multiple of the chunk
          af[d].clear_tail(k0, a.K, g);
          bf[d].clear_tail(k0, a.K, g);
        }
#pragma unroll
        for (int e = 0; e < 4 * KH; ++e)
#pragma unroll
          for (int i = 0; i < TMB; ++i)
#pragma unroll
            for (int j = 0; j < TNB; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(bf[d].v[j][e], af[d].v[i][e], acc[i][j], 0, 0, 0);
        // the 64 x 64 tiles take a superfluous (clamped) last fetch rather than the branch, which costs them 10 %
        if (TMB * TNB == 16 || c + d + DEPTH < c1) fetch(d, c + d + DEPTH);
      }
    }
  }

  // vector v of row block i: columns 4 v .. 4 v + 3 of the lane's 4 TNB (BT), or the 4 of its column block v
  auto vector_of = [&](int i, int v) -> f32x4 {
    if constexpr (!BT) return acc[i][v];
    f32x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = acc[i][(4 * v + e) % TNB][(4 * v + e) / TNB];
    return o;
  };
  auto store = [&](int i, int v, f32x4 x) {
    const int64_t m = m0 + (AT ? TMB * r + i : 16 * i + r);
    const int64_t n = n0 + (BT ? 4 * TNB * g + 4 * v : 16 * v + 4 * g);
    if (m >= a.M) return;
    if constexpr (VEC) {
      if (n < a.N) epilogue4<E>(a.ea, a.C, a.N, m, n, x);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (n + e < a.N) epilogue_store<E>(a.ea, a.C, a.N, m, n + e, x[e]);
    }
  };
  if constexpr (WGK == 1) {
#pragma unroll
    for (int i = 0; i < TMB; ++i)
#pragma unroll
      for (int v = 0; v < TNB; ++v) store(i, v, vector_of(i, v));
  } else {
    // partial tiles through LDS, [tile wave][k wave][vector][lane]; k wave w adds vectors w, w + WGK, ... in order of k
    f32x4 *mine = red + (wt * WGK + wk) * (NV * 64) + lane;
#pragma unroll
    for (int i = 0; i < TMB; ++i)
#pragma unroll
      for (int v = 0; v < TNB; ++v) mine[(i * TNB + v) * 64] = vector_of(i, v);
    __syncthreads();
    for (int t = wk; t < NV; t += WGK) {
      f32x4 s = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int w = 0; w < WGK; ++w) s += red[(wt * WGK + w) * (NV * 64) + t * 64 + lane];
      store(t / TNB, t % TNB, s);
    }
  }
}

template <typename E, int TMB, int TNB, int WGM, int WGN, int WGK, int KH, int DEPTH, bool VEC>
int launch_f32(int layout, F32GemmArgs a, hipStream_t st) {
  const int64_t tm = (a.M + 16 * TMB * WGM - 1) / (16 * TMB * WGM), tn = (a.N + 16 * TNB * WGN - 1) / (16 * TNB * WGN);
  if (tm * tn > (1 << 28)) return MTNLG_UNSUPPORTED_SHAPE;
  a.tiles_m = (int)tm;
  a.tiles_n = (int)tn;
  const dim3 grid((unsigned)((tm * tn + 7) / 8 * 8));
  constexpr int threads = 64 * WGM * WGN * WGK;
  if (layout == MTNLG_GEMM_NT)
    gemm_f32_kernel<E, TMB, TNB, WGM, WGN, WGK, KH, DEPTH, false, false, VEC><<<grid, threads, 0, st>>>(a);
  else if (layout == MTNLG_GEMM_NN)
    gemm_f32_kernel<E, TMB, TNB, WGM, WGN, WGK, KH, DEPTH, false, true, VEC><<<grid, threads, 0, st>>>(a);
  else
    gemm_f32_kernel<E, TMB, TNB, WGM, WGN, WGK, KH, DEPTH, true, true, VEC><<<grid, threads, 0, st>>>(a);
  return check_launch();
}

template <typename E>
int gemm_generic_of(int layout, const F32GemmArgs &a, bool vec, bool small, hipStream_t st) {
  if (!vec) return launch_f32<E, 2, 2, 1, 1, 4, 1, 2, false>(layout, a, st);
  if (small) return launch_f32<E, 2, 2, 1, 1, 8, 1, 2, true>(layout, a, st);
  return launch_f32<E, 4, 4, 1, 1, 4, 2, 1, true>(layout, a, st);
}

}  // namespace

// 32 x 32 tiles (K split over eight waves) or 64 x 64 tiles (over four): rounds of 256 workgroups times the time of a
// round at equal K.  Measured (us, K = 1024, 64 / 32): 256 x 256 23 / 10, 1024 x 1024 26 / 33, 1024 x 3072 NT 88 / 95,
// TN 64 / 100; 256 x 1024 x 256 10 / 5; 2048^3 NT 187 / 228, TN 150 / 236 (115 TFLOP/s; nominal 157).  A round of the 64 x 64
// tiles costs least where both operands are row-contiguous, whose loads cover whole lines.
bool gemm_generic_small_tile(int layout, int64_t M, int64_t N) {
  const double round64 = layout == MTNLG_GEMM_NT ? 25 : layout == MTNLG_GEMM_NN ? 22 : 20, round32 = 8.5;
  auto rounds = [&](int64_t t) { return (double)((((M + t - 1) / t) * ((N + t - 1) / t) + 255) / 256); };
  return rounds(32) * round32 < rounds(64) * round64;
}

int gemm_generic(int dtype, int layout, int64_t M, int64_t N, int64_t K, const void *A,
                 const void *B, void *C, const void *bias, void *aux, uint32_t epi,
                 hipStream_t stream) {
  if (layout < 0 || layout > 2) return MTNLG_INVALID_ARG;
  if ((M + 63) / 64 > 65535) return MTNLG_UNSUPPORTED_SHAPE;
  F32GemmArgs a{M, N, K, layout == MTNLG_GEMM_TN ? M : K, layout == MTNLG_GEMM_NT ? K : N, A, B, C, EpiArgs{bias, aux, epi}, 0, 0};
  const size_t es = dtype == MTNLG_F32 ? 4 : 2;
  const uintptr_t unit = 4 * es - 1, c_unit = (epi & MTNLG_EPI_OUT_F32) ? 15 : unit;
  const bool vec = a.lda % 4 == 0 && a.ldb % 4 == 0 && N % 4 == 0 &&
                   !(((uintptr_t)A | (uintptr_t)B | (uintptr_t)bias | (uintptr_t)aux) & unit) && !((uintptr_t)C & c_unit);
  LaunchScope scope(MTNLG_K_GEMM_NT + layout, stream);
  if (dtype == MTNLG_F32) return gemm_generic_of<float>(layout, a, vec, gemm_generic_small_tile(layout, M, N), stream);
  return gemm_generic_of<bf16>(layout, a, vec, gemm_generic_small_tile(layout, M, N), stream);
}

}  // namespace mtnlg
