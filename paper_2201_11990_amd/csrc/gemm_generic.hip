// GEMM with operands loaded straight into registers: fp32 problems between a few tiles and many, and every problem whose row lengths the kernels that move
// tiles by DMA do not take (bf16 elements are widened on load and go to the bf16 instructions as the one part that they are).  Any M, N, K,
// any layout.
//
// Longer sums of fp32 values: they are cut into three bf16 parts that add up to them exactly, and the six largest of the nine products of parts run
// on v_mfma_f32_16x16x32_bf16 (common.h: Parts): sums in fp32, an error below that of the fp32 instructions (1024 x 1024 x 4096 against
// 64 bits: 5.7e-7 with those, 2.2e-7 so).  What bounds it: per 64 x 64 wave tile and 32 k 96 MFMAs (1600 cycles) and 310 vector
// instructions for the parts (1300 cycles), which the two waves of a SIMD overlap little, and the 16 KB of operands that come
// from L2 for them (9 TB/s over the chip).  On v_mfma_f32_16x16x4_f32 before: 1024 x 4096 x 1024 109 / 96 / 91 us (NT / NN / TN), now 71 / 61 /
// 58; 2048^3 199 / 174 / 157, now 129 / 112 / 110.
// The K axis of a workgroup's tile is split over its waves (WGK); their partial tiles are added through LDS in a fixed
// order, so a small M x N still fills the chip and a long K is a short chain.
//   Chunk of 32 k: lane l = 16 g + r supplies k = 16 h + 4 g + e as element 4 h + e of its operand (the k order inside a chunk is
//   free as long as both operands agree), so both 64-byte halves of a K-contiguous line are taken together.
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

// Workgroup of WGM x WGN x WGK waves, wave tile 16 TMB x 16 TNB.  VEC: every row length is a multiple of 4 elements and
// every pointer aligned to 4 elements.  DIRECT: chunks of 16 k on the fp32 instructions, two in flight (gemm_direct_time says when).
template <typename E, int TMB, int TNB, int WGM, int WGN, int WGK, bool AT, bool BT, bool VEC, bool DIRECT>
__global__ __launch_bounds__(64 * WGM * WGN * WGK, DIRECT && TMB == 2 ? 8 : 2) void gemm_f32_kernel(F32GemmArgs a) {
  constexpr int KH = DIRECT ? 1 : 2, CHUNK = 16 * KH;
  constexpr int NP = sizeof(E) == 2 || DIRECT ? 1 : 3;
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
  const int nc_all = (int)((a.K + CHUNK - 1) / CHUNK), per = (nc_all + WGK - 1) / WGK;
  const int c0 = wk * per, c1 = c0 + per < nc_all ? c0 + per : nc_all;   // this wave's chunks

  f32x4 acc[TMB][TNB];
#pragma unroll
  for (int i = 0; i < TMB; ++i)
#pragma unroll
    for (int j = 0; j < TNB; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  Frag<E, TMB, KH, AT, VEC> af;
  Frag<E, TNB, KH, BT, VEC> bf;
  // Every condition in the loop is the same for the whole wave and held in a scalar register, and the fetches are
  // unconditional (clamped): fragments that are fetched on some paths only, under a condition the compiler takes for
  // divergent, were miscompiled (accumulators placed over live fragments).
  auto start = [&](int c) { return (int64_t)(c < nc_all ? c : nc_all - 1) * CHUNK; };
  if constexpr (DIRECT) {
    Frag<E, TMB, KH, AT, VEC> ad[2];
    Frag<E, TNB, KH, BT, VEC> bd[2];
    auto fetch = [&](int d, int c) {
      ad[d].fetch(A, a.lda, m0, a.M, start(c), a.K, g, r);
      bd[d].fetch(B, a.ldb, n0, a.N, start(c), a.K, g, r);
    };
    fetch(0, c0);
    fetch(1, c0 + 1);
    for (int c = c0; c < c1; c += 2) {
#pragma unroll
      for (int d = 0; d < 2; ++d) {
        if (c + d < c1) {
          const int64_t k0 = (int64_t)(c + d) * CHUNK;
          if (k0 + CHUNK > a.K) {
            ad[d].clear_tail(k0, a.K, g);
            bd[d].clear_tail(k0, a.K, g);
          }
#pragma unroll
          for (int e = 0; e < 4 * KH; ++e)
#pragma unroll
            for (int i = 0; i < TMB; ++i)
#pragma unroll
              for (int j = 0; j < TNB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(bd[d].v[j][e], ad[d].v[i][e], acc[i][j], 0, 0, 0);
          if (c + d + 2 < c1) fetch(d, c + d + 2);
        }
      }
    }
  } else {
    af.fetch(A, a.lda, m0, a.M, start(c0), a.K, g, r);
    bf.fetch(B, a.ldb, n0, a.N, start(c0), a.K, g, r);
    for (int c = c0; c < c1; ++c) {
      const int64_t k0 = (int64_t)c * CHUNK;
      if (k0 + CHUNK > a.K) {   // uniform: the last chunk of a K that is no multiple of the chunk
        af.clear_tail(k0, a.K, g);
        bf.clear_tail(k0, a.K, g);
      }
      Parts<NP> ap[TMB], bp[TNB];
#pragma unroll
      for (int i = 0; i < TMB; ++i) ap[i].of(af.v[i]);
      af.fetch(A, a.lda, m0, a.M, start(c + 1), a.K, g, r);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < TNB; ++j) bp[j].of(bf.v[j]);
      bf.fetch(B, a.ldb, n0, a.N, start(c + 1), a.K, g, r);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < TNB; ++j) {
#pragma unroll
        for (int i = 0; i < TMB; ++i) acc[i][j] = mma_parts(bp[j], ap[i], acc[i][j], 0);
        if constexpr (NP > 1) {   // the smaller products in sums of their own (for one chunk: there are no registers to keep them)
          f32x4 low[TMB];
#pragma unroll
          for (int i = 0; i < TMB; ++i) low[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
          for (int step = 1; step < 6; ++step)
#pragma unroll
            for (int i = 0; i < TMB; ++i) low[i] = mma_parts(bp[j], ap[i], low[i], step);
#pragma unroll
          for (int i = 0; i < TMB; ++i) acc[i][j] += low[i];
        }
      }
    }
  }
  if constexpr (NP > 1) {
    // Where the parts cannot say a value (parts_hold), the wave takes its chunks once more on the fp32 instructions.
    bool odd = false;
#pragma unroll
    for (int i = 0; i < TMB; ++i)
#pragma unroll
      for (int j = 0; j < TNB; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) odd = odd || !parts_hold(acc[i][j][e]);
    if (__builtin_amdgcn_ballot_w64(odd) != 0) {
#pragma unroll
      for (int i = 0; i < TMB; ++i)
#pragma unroll
        for (int j = 0; j < TNB; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
      for (int c = c0; c < c1; ++c) {
        const int64_t k0 = (int64_t)c * CHUNK;
        af.fetch(A, a.lda, m0, a.M, k0, a.K, g, r);
        bf.fetch(B, a.ldb, n0, a.N, k0, a.K, g, r);
        af.clear_tail(k0, a.K, g);
        bf.clear_tail(k0, a.K, g);
#pragma unroll
        for (int e = 0; e < 4 * KH; ++e)
#pragma unroll
          for (int i = 0; i < TMB; ++i)
#pragma unroll
            for (int j = 0; j < TNB; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(bf.v[j][e], af.v[i][e], acc[i][j], 0, 0, 0);
      }
    } else {
#pragma unroll
      for (int i = 0; i < TMB; ++i)
#pragma unroll
        for (int j = 0; j < TNB; ++j) acc[i][j] = parts_sum(acc[i][j]);
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
      if (n < a.N) epilogue4<E, false>(a.ea, a.C, a.N, m, n, x);
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

template <typename E, int TMB, int TNB, int WGM, int WGN, int WGK, bool VEC, bool DIRECT = false>
int launch_f32(int layout, F32GemmArgs a, hipStream_t st) {
  const int64_t tm = (a.M + 16 * TMB * WGM - 1) / (16 * TMB * WGM), tn = (a.N + 16 * TNB * WGN - 1) / (16 * TNB * WGN);
  if (tm * tn > (1 << 28)) return MTNLG_UNSUPPORTED_SHAPE;
  a.tiles_m = (int)tm;
  a.tiles_n = (int)tn;
  const dim3 grid((unsigned)((tm * tn + 7) / 8 * 8));
  constexpr int threads = 64 * WGM * WGN * WGK;
  if (layout == MTNLG_GEMM_NT)
    gemm_f32_kernel<E, TMB, TNB, WGM, WGN, WGK, false, false, VEC, DIRECT><<<grid, threads, 0, st>>>(a);
  else if (layout == MTNLG_GEMM_NN)
    gemm_f32_kernel<E, TMB, TNB, WGM, WGN, WGK, false, true, VEC, DIRECT><<<grid, threads, 0, st>>>(a);
  else
    gemm_f32_kernel<E, TMB, TNB, WGM, WGN, WGK, true, true, VEC, DIRECT><<<grid, threads, 0, st>>>(a);
  return check_launch();
}

template <typename E>
int gemm_generic_of(int layout, const F32GemmArgs &a, bool vec, bool small, bool direct, hipStream_t st) {
  if (!vec) return launch_f32<E, 2, 2, 1, 1, 4, false>(layout, a, st);
  if constexpr (sizeof(E) == 4) {
    if (direct) return small ? launch_f32<E, 2, 2, 1, 1, 8, true, true>(layout, a, st) : launch_f32<E, 4, 4, 1, 1, 4, true, true>(layout, a, st);
  } else {   // (small fp32 problems: gemm_wave)
    if (small) return launch_f32<E, 2, 2, 1, 1, 8, true>(layout, a, st);
  }
  return launch_f32<E, 4, 4, 1, 1, 4, true>(layout, a, st);
}

}  // namespace

// 32 x 32 tiles (K split over eight waves) or 64 x 64 tiles (over four): rounds of 256 workgroups times the time of a round at equal K.
static bool small_tile(int64_t M, int64_t N, double round64, double round32) {
  auto rounds = [&](int64_t t) { return (double)((((M + t - 1) / t) * ((N + t - 1) / t) + 255) / 256); };
  return rounds(32) * round32 < rounds(64) * round64;
}
// fp32 problems on the fp32 instructions: measured (us, K = 1024, 64 / 32) 256 x 256 23 / 10, 1024 x 1024 26 / 33, 1024 x 3072 NT 88 / 95,
// TN 64 / 100.
bool gemm_generic_small_tile(int layout, int64_t M, int64_t N) {
  return small_tile(M, N, layout == MTNLG_GEMM_NT ? 25 : layout == MTNLG_GEMM_NN ? 22 : 20, 8.5);
}
// bf16 problems, one part on the bf16 instructions: 228 sizes (60 to 4100 rows and columns, K 132 to 4100), 0.2 % off the better tile on
// average, 7 % at most; by the line above 1.3 % and 29 %.  us, 64 / 32: 252 x 1020 x 1020 NT 12.3 / 7.8; 508 x 516 x 1028 NT 12.8 / 12.0,
// TN 9.8 / 10.4; 1020 x 1028 x 1028 NT 20.8 / 24.8; 2044 x 2052 x 1028 NT 44 / 78.
bool gemm_generic_small_tile_bf16(int layout, int64_t M, int64_t N) {
  return small_tile(M, N, layout == MTNLG_GEMM_NT ? 11 : layout == MTNLG_GEMM_NN ? 9.5 : 7.7, 4.5);
}

// fp32, 64 x 64 tiles: fitted to 270 measured problems (K 128 to 4096, 4 to 4000 tiles).
double gemm_generic_time(int layout, int64_t M, int64_t N, int64_t K) {
  const double rounds = (double)(((M + 63) / 64) * ((N + 63) / 64)) / 256;
  const double per_k = layout == MTNLG_GEMM_NT ? 0.0137 : layout == MTNLG_GEMM_NN ? 0.0120 : 0.0118;
  if (rounds <= 1) return 7.5 + 1.17 * per_k * (double)K;   // one wave on a SIMD
  return 4.2 + (rounds < 2 ? 2 : rounds) * (3.7 + per_k * (double)K);
}

// fp32 on the fp32 instructions (32 x 32 or 64 x 64 tiles by the rule above): short sums, for which the way through LDS and the parts take longer than the products.
// us here / in gemm_wave.hip, NT, NN, TN: 256 x 1024 x 192 4.6 / 4.7, 4.4 / 4.8, 4.3 / 4.7; 1024 x 1024 x 128 7.9 / 8.8, 7.7 / 9.5, 7.1 / 10.7;
// 1024 x 2048 x 64 9.1 / 11.3, 10.7 / 11.5, 9.9 / 11.3; at K = 320 256 x 1024 5.3 / 5.3, 512 x 1024 7.9 / 6.8.
double gemm_direct_time(int64_t M, int64_t N, int64_t K) {
  if (K > 256) return INFINITY;
  const double rounds = (double)(((M + 31) / 32) * ((N + 31) / 32)) / 256;
  return 3.0 + (rounds < 1 ? 1 : rounds) * (0.45 + 0.0055 * (double)K);
}

int gemm_generic(int dtype, int layout, int64_t M, int64_t N, int64_t K, const void *A,
                 const void *B, void *C, const void *bias, void *aux, uint32_t epi,
                 hipStream_t stream) {
  if (layout < 0 || layout > 2) return MTNLG_INVALID_ARG;
  if (M > GEMM_GENERIC_MAX_ROWS) return MTNLG_UNSUPPORTED_SHAPE;
  F32GemmArgs a{M, N, K, layout == MTNLG_GEMM_TN ? M : K, layout == MTNLG_GEMM_NT ? K : N, A, B, C, EpiArgs{bias, aux, epi}, 0, 0};
  const size_t es = dtype == MTNLG_F32 ? 4 : 2;
  const uintptr_t unit = 4 * es - 1, c_unit = (epi & MTNLG_EPI_OUT_F32) ? 15 : unit;
  const bool vec = a.lda % 4 == 0 && a.ldb % 4 == 0 && N % 4 == 0 &&
                   !(((uintptr_t)A | (uintptr_t)B | (uintptr_t)bias | (uintptr_t)aux) & unit) && !((uintptr_t)C & c_unit);
  LaunchScope scope(MTNLG_K_GEMM_NT + layout, stream);
  if (dtype == MTNLG_F32)
    return gemm_generic_of<float>(layout, a, vec, gemm_generic_small_tile(layout, M, N), gemm_direct_time(M, N, K) < gemm_generic_time(layout, M, N, K), stream);
  return gemm_generic_of<bf16>(layout, a, vec, gemm_generic_small_tile_bf16(layout, M, N), false, stream);
}

}  // namespace mtnlg
