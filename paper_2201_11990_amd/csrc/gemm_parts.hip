// fp32 GEMM for problems with many output tiles: values in three bf16 parts (common.h: Parts), 128 x 128 tiles, parts shared through LDS.
//
// Eight waves of 64 x 32, slabs of 32 k.  Every value is cut into parts once a workgroup: a wave loads two of the tile's sixteen 16-row
// blocks into registers, two slabs ahead, cuts them (72 vector instructions a slab) and writes the fragments to LDS as the matrix
// instructions read them, lane by lane (a ring of three stages of 48 KB, one barrier a slab).  us,
// operands straight to registers (gemm_generic.hip) / K split over waves (gemm_wave.hip) / here: 1024 x 4096 x 1024 NT 71 / 65 / 51, NN 61 / 68 / 52,
// TN 58 / 65 / 50; 2048 x 2048 x 4096 NT 242 / 208 / 179.  Those two cut a value once a wave, two to eight times a workgroup, and with the
// operands in LDS as fp32 values and the cutting behind the reads the same tiles took 66 us at 1024 x 4096 x 1024 NT; leaving the cutting out
// altogether, 45.  What bounds it now: the MFMAs (0.97 to 1.2 PFLOP/s of products of parts), then LDS: 147 KB read and 48 KB written a slab.
#include "common.h"

namespace mtnlg {

namespace {

constexpr int WAVES = 8, TILE = 128, SLAB_K = 32, STAGES = 3;
constexpr int BLOCK = 3 * 1024;             // bytes of a 16-row block's three fragments
constexpr int STAGE = 16 * BLOCK;           // blocks of A, then of B
constexpr uint32_t RECORDS = 0xFFFFFFE0u, OUTSIDE = 0xFFFFFFF0u;   // bytes a descriptor covers at most; an offset beyond

struct PartsArgs {
  int64_t M, N, K, lda, ldb;
  const float *A, *B;
  float *C;
  EpiArgs ea;
  int tiles_m, tiles_n;
};

typedef __attribute__((ext_vector_type(2))) float f32x2;

// Two 16-row blocks of an operand, 32 k at a time: element 4 h + e of a block is k = 16 h + 4 g + e of its row, lane l = 16 g + r.
//   K-contiguous: block b holds row 16 b + r.
//   Row-contiguous ([k][row] in memory): row 2 r + b: a load takes neighbouring rows, and the epilogue undoes that.
// Rows past the edge lie outside the descriptor and arrive as zeros, and so does what lies past K.
struct Pair {
  float v[2][8];
  // first: element (first row of the blocks, k = 0), row row0 of the operand; slabs past the last one: zeros
  template <bool ROWC>
  __device__ __forceinline__ void load(const float *first, int64_t ld, int64_t rows_left, int64_t row0, int64_t k0, int64_t K, int lane) {
    const int g = lane >> 4, r = lane & 15;
    if constexpr (!ROWC) {
      const __amdgpu_buffer_rsrc_t rs = rsrc(first + k0, RECORDS);
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const uint32_t off = (uint32_t)((16 * b + r) * ld * 4 + (16 * h + 4 * g) * 4);
          const f32x4 t = __builtin_bit_cast(
              f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, 16 * b + r < rows_left && k0 + 16 * h + 4 * g < K ? off : OUTSIDE, 0, 0));
#pragma unroll
          for (int e = 0; e < 4; ++e) v[b][4 * h + e] = t[e];
        }
    } else {
      const int64_t left = ((K - k0) * ld - row0) * 4;   // to the end of the matrix
      const __amdgpu_buffer_rsrc_t rs = rsrc(first + k0 * ld, left < 0 ? 0 : left < RECORDS ? (uint32_t)left : RECORDS);
      const uint32_t off = 2 * r < rows_left ? (uint32_t)(4 * g * ld * 4 + r * 8) : OUTSIDE;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t at = (uint32_t)((16 * (e >> 2) + (e & 3)) * ld * 4);   // the same in all lanes
        const f32x2 t = __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(rs, off == OUTSIDE ? OUTSIDE : off + at, 0, 0));
        v[0][e] = t[0];
        v[1][e] = t[1];
      }
    }
  }
  __device__ __forceinline__ static __amdgpu_buffer_rsrc_t rsrc(const float *base, uint32_t records) {
    const uint64_t a = (uint64_t)base;
    const uint64_t u = ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(a >> 32)) << 32) | (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)a);
    return __builtin_amdgcn_make_buffer_rsrc((void *)u, 0, (int)records, 0x00020000);
  }
};

template <int V>
struct Num { static constexpr int value = V; };

template <bool AT, bool BT>
__global__ __launch_bounds__(64 * WAVES, 2) void gemm_parts_kernel(PartsArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wm = wave >> 2, wn = wave & 3;

  // XCD x (workgroup id mod 8) takes a contiguous run of tiles, ordered in blocks of 8 row tiles
  const int tiles = a.tiles_m * a.tiles_n, per_xcd = (tiles + 7) / 8;
  const int pid = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per_xcd || pid >= tiles) return;
  const int per_group = 8 * a.tiles_n, grp = pid / per_group, first_m = grp * 8;
  const int gsz = a.tiles_m - first_m < 8 ? a.tiles_m - first_m : 8;
  const int64_t m0 = (int64_t)(first_m + (pid % per_group) % gsz) * TILE, n0 = (int64_t)((pid % per_group) / gsz) * TILE;

  // Waves 0-3 bring A, 4-7 B, 32 rows each.
  const bool is_a = wave < 4;
  const int64_t row0 = (is_a ? m0 : n0) + 32 * (wave & 3), rows_left = (is_a ? a.M : a.N) - row0, ld = is_a ? a.lda : a.ldb;
  const float *first = (is_a ? a.A : a.B) + ((is_a ? AT : BT) ? row0 : row0 * ld);
  const int nk = (int)((a.K + SLAB_K - 1) / SLAB_K);
  Pair raw[2];   // [slab % 2]
  auto put = [&](auto slot, int stage) {   // the wave's blocks in parts
    constexpr int P = decltype(slot)::value;
    char *to = smem + stage * STAGE + 2 * wave * BLOCK + lane * 16;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      Parts<3> p;
      p.of(raw[P].v[b]);
#pragma unroll
      for (int i = 0; i < 3; ++i) *reinterpret_cast<bf16x8 *>(to + b * BLOCK + i * 1024) = p.p[i];
    }
  };
  auto get = [&](Parts<3> &p, int stage, int block) {
#pragma unroll
    for (int i = 0; i < 3; ++i) p.p[i] = *reinterpret_cast<const bf16x8 *>(smem + stage * STAGE + block * BLOCK + i * 1024 + lane * 16);
  };

  f32x4 acc[4][2], low[4][2];   // low: the sums of the smaller products of parts
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = low[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  Parts<3> ap[2], bp[2][2];   // [block % 2], [slab % 2][block]
  // One body for each way of loading: where the two kinds meet in one, the compiler waits for all loads at their first use.
  auto run = [&](auto rowc) {
    auto load = [&](auto slot, int s) {
      raw[decltype(slot)::value].template load<decltype(rowc)::value != 0>(first, ld, rows_left, row0, (int64_t)s * SLAB_K, a.K, lane);
    };
    load(Num<0>{}, 0);
    load(Num<1>{}, 1);
    put(Num<0>{}, 0);
    load(Num<0>{}, 2);
    put(Num<1>{}, 1);
    load(Num<1>{}, 3);
    __syncthreads();
    get(bp[0][0], 0, 8 + 2 * wn);
    get(bp[0][1], 0, 9 + 2 * wn);
    get(ap[0], 0, 4 * wm);
    int cur = 0;   // slab % STAGES
    auto slab = [&](auto parity, int s) {
      constexpr int P = decltype(parity)::value;
      const int next = cur == STAGES - 1 ? 0 : cur + 1, free = next == STAGES - 1 ? 0 : next + 1;
      auto block = [&](auto num) {   // the MFMAs of block i of A
        constexpr int i = decltype(num)::value;
        if constexpr (i < 3) get(ap[(i + 1) & 1], cur, 4 * wm + i + 1);
        else get(ap[0], next, 4 * wm);
        if constexpr (i >= 2) get(bp[1 - P][i - 2], next, 8 + 2 * wn + i - 2);
        if constexpr (i == 0) put(parity, free);          // slab s + 2
        if constexpr (i == 1) load(parity, s + 4);
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = mma_parts(bp[P][j], ap[i & 1], acc[i][j], 0);
#pragma unroll
        for (int step = 1; step < 6; ++step)
#pragma unroll
          for (int j = 0; j < 2; ++j) low[i][j] = mma_parts(bp[P][j], ap[i & 1], low[i][j], step);
        __builtin_amdgcn_sched_barrier(0);
      };
      block(Num<0>{});
      block(Num<1>{});
      block(Num<2>{});
      block(Num<3>{});
      cur = next;
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // slab s + 2 written everywhere, slab s no longer read
    };
    for (int s = 0; s < nk; s += 2) {
      slab(Num<0>{}, s);
      if (s + 1 < nk) slab(Num<1>{}, s + 1);
    }
  };
  if constexpr (AT == BT) {
    run(Num<AT>{});
  } else {
    if (is_a) run(Num<AT>{});
    else run(Num<BT>{});
  }

  // Where the parts cannot say a value (parts_hold), the tile is taken once more on the fp32 instructions.
  bool odd = false;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc[i][j][e] += low[i][j][e];
        odd = odd || !parts_hold(acc[i][j][e]);
      }
  if (__syncthreads_or(odd)) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
    for (int s = 0; s < nk; ++s) {   // the same blocks as fp32 values: elements 0-3 in the place of the first part, 4-7 of the second
      if (is_a) raw[0].load<AT>(first, ld, rows_left, row0, (int64_t)s * SLAB_K, a.K, lane);
      else raw[0].load<BT>(first, ld, rows_left, row0, (int64_t)s * SLAB_K, a.K, lane);
      __syncthreads();
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          f32x4 t;
#pragma unroll
          for (int e = 0; e < 4; ++e) t[e] = raw[0].v[b][4 * h + e];
          *reinterpret_cast<f32x4 *>(smem + (2 * wave + b) * BLOCK + h * 1024 + lane * 16) = t;
        }
      __syncthreads();
#pragma unroll 1
      for (int h = 0; h < 2; ++h) {
        f32x4 x[4], y[2];
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = *reinterpret_cast<const f32x4 *>(smem + (4 * wm + i) * BLOCK + h * 1024 + lane * 16);
#pragma unroll
        for (int j = 0; j < 2; ++j) y[j] = *reinterpret_cast<const f32x4 *>(smem + (8 + 2 * wn + j) * BLOCK + h * 1024 + lane * 16);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(y[j][e], x[i][e], acc[i][j], 0, 0, 0);
      }
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = parts_sum(acc[i][j]);
  }

#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      f32x4 o = acc[i][v];
      if constexpr (BT) {   // the lane's 8 columns are consecutive, block by block
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = acc[i][(4 * v + e) & 1][(4 * v + e) >> 1];
      }
      const int64_t m = m0 + 64 * wm + 32 * (i >> 1) + (AT ? 2 * r + (i & 1) : 16 * (i & 1) + r), n = n0 + 32 * wn + (BT ? 8 * g + 4 * v : 16 * v + 4 * g);
      if (m < a.M && n < a.N) epilogue4<float>(a.ea, a.C, a.N, m, n, o);
    }
}

template <bool AT, bool BT>
int launch(const PartsArgs &a, hipStream_t st) {
  constexpr int smem = STAGES * STAGE;
  static unsigned long long attr_done = 0;
  int device;
  if (!attr_is_set(attr_done, &device)) {
    if (hipFuncSetAttribute((const void *)gemm_parts_kernel<AT, BT>, hipFuncAttributeMaxDynamicSharedMemorySize, smem) != hipSuccess)
      return MTNLG_HIP_ERROR;
    attr_mark_set(attr_done, device);
  }
  gemm_parts_kernel<AT, BT><<<dim3((unsigned)(((int64_t)a.tiles_m * a.tiles_n + 7) / 8 * 8)), 64 * WAVES, smem, st>>>(a);
  return check_launch();
}

}  // namespace

// Estimated microseconds; one round of 256 tiles costs the same whether it is full or not.
double gemm_parts_time(int64_t M, int64_t N, int64_t K) {
  const int64_t rounds = (((M + TILE - 1) / TILE) * ((N + TILE - 1) / TILE) + 255) / 256;
  return (double)rounds * (8.3 + 0.0405 * (double)K);
}

// fp32 problems that gemm_wave_takes
int gemm_parts(int layout, int64_t M, int64_t N, int64_t K, const void *A, const void *B, void *C, const void *bias, void *aux, uint32_t epi,
               hipStream_t stream) {
  if (layout < 0 || layout > 2 || M <= 0 || N <= 0 || K <= 0) return MTNLG_INVALID_ARG;
  if (!gemm_wave_takes(MTNLG_F32, layout, M, N, K, A, B, C, bias, aux)) return MTNLG_UNSUPPORTED_SHAPE;
  const int64_t tm = (M + TILE - 1) / TILE, tn = (N + TILE - 1) / TILE;
  if (tm * tn > (1 << 28)) return MTNLG_UNSUPPORTED_SHAPE;
  const PartsArgs a{M, N, K, layout == MTNLG_GEMM_TN ? M : K, layout == MTNLG_GEMM_NT ? K : N, static_cast<const float *>(A),
                    static_cast<const float *>(B), static_cast<float *>(C), EpiArgs{bias, aux, epi}, (int)tm, (int)tn};
  LaunchScope scope(MTNLG_K_GEMM_NT + layout, stream);
  if (layout == MTNLG_GEMM_NT) return launch<false, false>(a, stream);
  if (layout == MTNLG_GEMM_NN) return launch<false, true>(a, stream);
  return launch<true, true>(a, stream);
}

}  // namespace mtnlg
