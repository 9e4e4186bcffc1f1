// GEMM for problems with few output tiles, and the fp32 GEMM: the K axis of a tile is split over the eight waves of a workgroup.
//
// What bounds the streaming kernel on such problems is a chain: launch, one slab after the other through a ring that the
// whole workgroup shares, epilogue.  Here every wave owns the whole TB x TB tile (64 x 64 or 32 x 32) for every eighth slab of
// 128 bytes of K (64 bf16 or 32 fp32 values), moved by DMA (buffer_load ... lds) into a stage of its own, so there is no barrier
// before the merge: wait for the slab, take its fragments into registers, ask for the next one, multiply.  At K = 512 bf16
// all of K is one slab a wave.  The partial tiles meet in LDS, where the stages were, and are added in wave order.  A few tiles are a
// chain of latencies (256 x 512 x 1024: 10.6 us on the streaming kernel, 4.5 here); with more, the operands' way from L2 to LDS
// bounds it: 64 x 64 tiles move twice the bytes per FLOP of the streaming kernel's 128 x 128.
//
// fp32: values in three bf16 parts (common.h: Parts), bound by the MFMAs and the vector instructions that make the parts.
#include <math.h>

#include "common.h"

namespace mtnlg {

namespace {

constexpr int WAVES = 8;
constexpr uint32_t RECORDS = 0xFFFFFFE0u, OUTSIDE = 0xFFFFFFF0u;   // bytes a descriptor covers at most; an offset beyond

struct WaveGemmArgs {
  int64_t M, N, K, lda, ldb;
  const void *A, *B;
  void *C;
  EpiArgs ea;
  int tiles_m, tiles_n;
};

typedef __attribute__((ext_vector_type(8))) short i16x8;
typedef __attribute__((ext_vector_type(4))) short i16x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((address_space(3))) i16x4 *lds_i16x4_ptr;

// One operand's slab in a wave's LDS: TB rows x 128 bytes of K.
//   K-contiguous: [TB rows][8 units of 16 bytes], unit c of row r at c ^ (r & 7).
//   Row-contiguous ([k][row] in memory): [k][TB rows], the units of a k-row permuted so that the reads below spread over the banks:
//     bf16 (transposing reads: 16 lanes take 4 k-rows x 32 bytes) by bits 1 and 3 of k; fp32, 32 rows: neighbouring k-rows
//     swap places where bit 2 of k is set; fp32, 64 rows: 256-byte k-rows need nothing.
template <typename E, int TB, bool ROWC>
struct Slab {
  static constexpr int ES = sizeof(E), EPU = 16 / ES, SK = 128 / ES;   // element size, elements of a unit, k of a slab
  static constexpr int NI = TB / 8;          // DMA instructions (1 KB each)
  static constexpr int UPR = TB / EPU;       // row-contiguous: units of a k-row
  static constexpr int BYTES = TB * 128;
  static __device__ __forceinline__ int mask(int k) {
    if constexpr (ES == 4) return 0;
    else if constexpr (TB == 64) return (k & 2) | ((k >> 1) & 4);
    else return (k >> 2) & 2;
  }
  static __device__ __forceinline__ int place(int k) { return ES == 4 && TB == 32 ? k ^ ((k >> 2) & 1) : k; }   // (its own inverse)

  uint32_t off[NI];   // byte offsets of this lane's units from the slab's first element; rows past the edge lie outside
  __device__ __forceinline__ Slab(int64_t ld, int64_t rows_left, int lane) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      if constexpr (!ROWC) {
        const int row = 8 * i + (lane >> 3), c = (lane & 7) ^ (lane >> 3);
        off[i] = row < rows_left ? (uint32_t)(row * ld * ES + c * 16) : OUTSIDE;
      } else {
        const int q = 64 * i + lane, k = place(q / UPR), u = (q % UPR) ^ mask(k);
        off[i] = u * EPU < rows_left ? (uint32_t)(k * ld * ES + u * 16) : OUTSIDE;
      }
    }
  }
  // the slab at k0 into LDS; first: element (first row of the tile, k = 0); what lies past K arrives as zeros
  __device__ __forceinline__ void fetch(const E *first, int64_t ld, int64_t row0, int64_t k0, int64_t K, uint32_t lds, int lane) const {
    if constexpr (!ROWC) {
      const dma_rsrc_t rs = dma_rsrc(first + k0, RECORDS);
      const bool inside = k0 + ((lane & 7) ^ (lane >> 3)) * EPU < K;
#pragma unroll
      for (int i = 0; i < NI; ++i) dma16(rs, lds + i * 1024, inside ? off[i] : OUTSIDE);
    } else {
      const int64_t left = ((K - k0) * ld - row0) * ES;   // to the end of the matrix
      const dma_rsrc_t rs = dma_rsrc(first + k0 * ld, left < RECORDS ? (uint32_t)left : RECORDS);
#pragma unroll
      for (int i = 0; i < NI; ++i) dma16(rs, lds + i * 1024, off[i]);
    }
  }
};

// bf16: fragments of all blocks and both k-steps of a slab.  Lane l = 16 g + r holds row 16 b + r, k = 32 kk + 8 g .. + 7.
template <int TB, bool ROWC>
struct Frag16 {
  bf16x8 v[TB / 16][2];
  __device__ __forceinline__ void read(const char *stage, int lane) {
    using S = Slab<bf16, TB, ROWC>;
    const int g = lane >> 4, r = lane & 15;
#pragma unroll
    for (int b = 0; b < TB / 16; ++b)
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        if constexpr (!ROWC) {
          v[b][kk] = *reinterpret_cast<const bf16x8 *>(stage + (16 * b + r) * 128 + (((kk * 4 + g) ^ (r & 7)) << 4));
        } else {   // lane 16 g + L supplies the address of k-row 8 g + L / 4 (+ 4), rows 4 (L % 4) .. + 3 of the block
          const int u = 2 * b + ((r & 3) >> 1), k = 32 * kk + 8 * g + (r >> 2);
          const char *p = stage + k * (TB * 2) + ((u ^ S::mask(k)) << 4) + (r & 1) * 8;
          const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_ptr)p);
          const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_ptr)(p + 4 * (TB * 2)));
          const i16x8 t = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
          v[b][kk] = __builtin_bit_cast(bf16x8, t);
        }
      }
  }
};

// fp32: element (b, 4 h + e) is k = 16 h + 4 g + e of row 16 b + r, or, row-contiguous, of row (TB / 16) r + b: a read takes
// neighbouring rows, and the epilogue undoes that.
template <int TB, bool ROWC>
struct Frag32 {
  float v[TB / 16][8];
  __device__ __forceinline__ void read(const char *stage, int lane) {
    const int g = lane >> 4, r = lane & 15;
    if constexpr (!ROWC) {
#pragma unroll
      for (int b = 0; b < TB / 16; ++b)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const f32x4 t = *reinterpret_cast<const f32x4 *>(stage + (16 * b + r) * 128 + (((h * 4 + g) ^ (r & 7)) << 4));
#pragma unroll
          for (int e = 0; e < 4; ++e) v[b][4 * h + e] = t[e];
        }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const char *p = stage + Slab<float, TB, ROWC>::place(16 * (e >> 2) + 4 * g + (e & 3)) * (TB * 4) + r * (TB / 4);
        if constexpr (TB == 64) {
          const f32x4 t = *reinterpret_cast<const f32x4 *>(p);
#pragma unroll
          for (int b = 0; b < 4; ++b) v[b][e] = t[b];
        } else {
          const f32x2 t = *reinterpret_cast<const f32x2 *>(p);
          v[0][e] = t[0];
          v[1][e] = t[1];
        }
      }
    }
  }
};

// The tile of workgroup `block` of a problem's grid.
template <typename E, int TB, bool AT, bool BT>
__device__ __forceinline__ void wave_tile(const WaveGemmArgs &a, int block, char *smem) {
  using SA = Slab<E, TB, AT>;
  using SB = Slab<E, TB, BT>;
  constexpr int NB = TB / 16, NV = NB * NB, STAGE = SA::BYTES + SB::BYTES, SK = SA::SK;
  static_assert(NV * 1024 <= STAGE, "a wave's partial tile fits its stage");
  const int lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

  // XCD x (workgroup id mod 8) takes a contiguous run of tiles, ordered in blocks of 8 row tiles
  const int tiles = a.tiles_m * a.tiles_n, per_xcd = (tiles + 7) / 8;
  const int pid = (block & 7) * per_xcd + (block >> 3);
  if (block >> 3 >= per_xcd || pid >= tiles) return;
  const int per_group = 8 * a.tiles_n, grp = pid / per_group, first_m = grp * 8;
  const int gsz = a.tiles_m - first_m < 8 ? a.tiles_m - first_m : 8;
  const int64_t m0 = (int64_t)(first_m + (pid % per_group) % gsz) * TB, n0 = (int64_t)((pid % per_group) / gsz) * TB;

  const E *A = static_cast<const E *>(a.A) + (AT ? m0 : m0 * a.lda), *B = static_cast<const E *>(a.B) + (BT ? n0 : n0 * a.ldb);
  const SA sa(a.lda, a.M - m0, lane);
  const SB sb(a.ldb, a.N - n0, lane);
  char *const stage = smem + wave * STAGE;
  const uint32_t lds = lds_address(stage);
  const int slabs = (int)((a.K + SK - 1) / SK);
  auto fetch = [&](int s) {
    sa.fetch(A, a.lda, m0, (int64_t)s * SK, a.K, lds, lane);
    sb.fetch(B, a.ldb, n0, (int64_t)s * SK, a.K, lds + SA::BYTES, lane);
  };

  f32x4 acc[NB][NB], low[sizeof(E) == 4 ? NB : 1][NB];   // low: fp32, the sums of the smaller products of parts
  auto clear = [&](auto &x) {
#pragma unroll
    for (auto &row : x)
#pragma unroll
      for (f32x4 &v : row) v = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  };
  clear(acc);
  clear(low);
  if (wave < slabs) fetch(wave);
  for (int s = wave; s < slabs; s += WAVES) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's slab has landed
    if constexpr (sizeof(E) == 2) {
      Frag16<TB, AT> af;
      Frag16<TB, BT> bf;
      af.read(stage, lane);
      bf.read(stage + SA::BYTES, lane);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // ... and left the stage
      if (s + WAVES < slabs) fetch(s + WAVES);
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
          for (int kk = 0; kk < 2; ++kk)   // B fragment first: a lane ends up with four consecutive columns of one row
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf.v[j][kk], af.v[i][kk], acc[i][j], 0, 0, 0);
    } else {
      Frag32<TB, AT> af;
      Frag32<TB, BT> bf;
      af.read(stage, lane);
      bf.read(stage + SA::BYTES, lane);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if (s + WAVES < slabs) fetch(s + WAVES);
      Parts<3> ap[NB];
#pragma unroll
      for (int i = 0; i < NB; ++i) ap[i].of(af.v[i]);
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        Parts<3> bp;
        bp.of(bf.v[j]);
#pragma unroll
        for (int i = 0; i < NB; ++i) acc[i][j] = mma_parts(bp, ap[i], acc[i][j], 0);
#pragma unroll
        for (int step = 1; step < 6; ++step)
#pragma unroll
          for (int i = 0; i < NB; ++i) low[i][j] = mma_parts(bp, ap[i], low[i][j], step);
      }
    }
  }
  if constexpr (sizeof(E) == 4) {
    // Where the parts cannot say a value (parts_hold), the wave takes its slabs once more on the fp32 instructions.
    bool odd = false;
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          acc[i][j][e] += low[i][j][e];
          odd = odd || !parts_hold(acc[i][j][e]);
        }
    if (__builtin_amdgcn_ballot_w64(odd) != 0) {
      clear(acc);
#pragma unroll 1
      for (int s = wave; s < slabs; s += WAVES) {
        fetch(s);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        Frag32<TB, AT> af;
        Frag32<TB, BT> bf;
        af.read(stage, lane);
        bf.read(stage + SA::BYTES, lane);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
          for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(bf.v[j][e], af.v[i][e], acc[i][j], 0, 0, 0);
      }
    } else {
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = parts_sum(acc[i][j]);
    }
  }

  // Vector v of row block i: four consecutive columns of one row.  The partial tiles go through LDS, [wave][vector][lane], each into
  // its own wave's stage; wave w adds vectors w, w + 8, ... of all waves in order.
  constexpr bool ROWS_BY_LANE = sizeof(E) == 4 && AT, COLS_BY_LANE = sizeof(E) == 4 && BT;
  f32x4 *red = reinterpret_cast<f32x4 *>(smem);
  constexpr int PITCH = STAGE / 16;   // vectors between two waves
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int v = 0; v < NB; ++v) {
      f32x4 o = acc[i][v];
      if constexpr (COLS_BY_LANE) {   // the lane's 4 NB columns are consecutive, block by block
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = acc[i][(4 * v + e) % NB][(4 * v + e) / NB];
      }
      red[wave * PITCH + (i * NB + v) * 64 + lane] = o;
    }
  __syncthreads();
#pragma unroll 1
  for (int t = wave; t < NV; t += WAVES) {
    f32x4 s = red[t * 64 + lane];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) s += red[w * PITCH + t * 64 + lane];
    const int i = t / NB, v = t % NB;
    const int64_t m = m0 + (ROWS_BY_LANE ? NB * r + i : 16 * i + r), n = n0 + (COLS_BY_LANE ? 4 * NB * g + 4 * v : 16 * v + 4 * g);
    if (m < a.M && n < a.N) epilogue4<E>(a.ea, a.C, a.N, m, n, s);
  }
}

template <typename E, int TB, bool AT, bool BT>
__global__ __launch_bounds__(64 * WAVES, 2) void gemm_wave_kernel(WaveGemmArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  wave_tile<E, TB, AT, BT>(a, blockIdx.x, smem);
}

// Sums over the rows of a matrix, 64 columns to a workgroup: eight lanes take a row's columns, so a wave has eight rows and a pass of
// the workgroup 64, four passes in flight.  One pass over few rows where mtnlg_colsum takes two kernels.
template <typename E>
__device__ __forceinline__ void column_sums(const ColumnSum &s, int64_t rows, int64_t C, int block, bool out_f32, bool accumulate,
                                            char *smem) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t c0 = (int64_t)block * 64 + (lane & 7) * 8;
  const E *in = static_cast<const E *>(s.in) + c0;
  constexpr int STEP = 8 * WAVES;
  float acc[8] = {};
  if (c0 < C) {
    int64_t t = 8 * wave + (lane >> 3);
    for (; t + 3 * STEP < rows; t += 4 * STEP) {
      Raw8<E> v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i].load(in + (t + i * STEP) * C);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] += v[i][e];
    }
    for (; t < rows; t += STEP) {
      Raw8<E> v;
      v.load(in + t * C);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] += v[e];
    }
  }
  float *part = reinterpret_cast<float *>(smem);   // [wave][64]
#pragma unroll
  for (int e = 0; e < 8; ++e) {
#pragma unroll
    for (int off = 8; off < 64; off <<= 1) acc[e] += __shfl_xor(acc[e], off, 64);
  }
  if (lane < 8) store8(part + wave * 64 + lane * 8, acc);
  __syncthreads();
  const int64_t c = (int64_t)block * 64 + threadIdx.x;
  if (threadIdx.x >= 64 || c >= C) return;
  float t = part[threadIdx.x];
#pragma unroll
  for (int w = 1; w < WAVES; ++w) t += part[w * 64 + threadIdx.x];
  if (out_f32) {
    float *out = static_cast<float *>(s.out) + c;
    *out = accumulate ? *out + t : t;
  } else {
    bf16 *out = static_cast<bf16 *>(s.out) + c;
    *out = (bf16)(accumulate ? (float)*out + t : t);
  }
}

// What the backward pass of a linear layer needs of dY, in one launch: dX = dY W (NN), dW = dY^T X (TN) and column sums (the bias gradient, or
// partial sums that the kernel before left).  None needs another's result, and with few tiles each alone leaves most of the chip idle.
struct GroupArgs {
  WaveGemmArgs nn, tn;
  int blocks_nn, blocks_tn;   // multiples of 8
  ColumnSums sums;
  int blocks_sum;             // for each of them
};
template <typename E, int TB>
__global__ __launch_bounds__(64 * WAVES, 2) void gemm_wave_group_kernel(GroupArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  int block = blockIdx.x;
  if (block < a.blocks_nn) return wave_tile<E, TB, false, true>(a.nn, block, smem);
  block -= a.blocks_nn;
  if (block < a.blocks_tn) return wave_tile<E, TB, true, true>(a.tn, block, smem);
  block -= a.blocks_tn;
  const ColumnSum s = a.sums.of[block / a.blocks_sum];
  block %= a.blocks_sum;
  if (a.sums.in_f32) column_sums<float>(s, a.sums.rows, a.sums.C, block, a.sums.out_f32, a.sums.accumulate, smem);
  else column_sums<bf16>(s, a.sums.rows, a.sums.C, block, a.sums.out_f32, a.sums.accumulate, smem);
}

template <typename E, int TB, bool AT, bool BT>
int launch(WaveGemmArgs a, hipStream_t st) {
  constexpr int smem = WAVES * 2 * TB * 128;
  static unsigned long long attr_done = 0;
  int device;
  if (!attr_is_set(attr_done, &device)) {
    if (hipFuncSetAttribute((const void *)gemm_wave_kernel<E, TB, AT, BT>, hipFuncAttributeMaxDynamicSharedMemorySize, smem) != hipSuccess)
      return MTNLG_HIP_ERROR;
    attr_mark_set(attr_done, device);
  }
  gemm_wave_kernel<E, TB, AT, BT><<<dim3((unsigned)(((int64_t)a.tiles_m * a.tiles_n + 7) / 8 * 8)), 64 * WAVES, smem, st>>>(a);
  return check_launch();
}

template <typename E, int TB>
int launch_layout(int layout, WaveGemmArgs a, hipStream_t st) {
  const int64_t tm = (a.M + TB - 1) / TB, tn = (a.N + TB - 1) / TB;
  if (tm * tn > (1 << 28)) return MTNLG_UNSUPPORTED_SHAPE;
  a.tiles_m = (int)tm;
  a.tiles_n = (int)tn;
  if (layout == MTNLG_GEMM_NT) return launch<E, TB, false, false>(a, st);
  if (layout == MTNLG_GEMM_NN) return launch<E, TB, false, true>(a, st);
  return launch<E, TB, true, true>(a, st);
}

template <typename E, int TB>
int launch_group(GroupArgs a, hipStream_t st) {
  auto blocks = [](WaveGemmArgs &p) {
    p.tiles_m = (int)((p.M + TB - 1) / TB);
    p.tiles_n = (int)((p.N + TB - 1) / TB);
    return (p.tiles_m * p.tiles_n + 7) / 8 * 8;
  };
  a.blocks_nn = blocks(a.nn);
  a.blocks_tn = blocks(a.tn);
  constexpr int smem = WAVES * 2 * TB * 128;
  static unsigned long long attr_done = 0;
  int device;
  if (!attr_is_set(attr_done, &device)) {
    if (hipFuncSetAttribute((const void *)gemm_wave_group_kernel<E, TB>, hipFuncAttributeMaxDynamicSharedMemorySize, smem) != hipSuccess)
      return MTNLG_HIP_ERROR;
    attr_mark_set(attr_done, device);
  }
  gemm_wave_group_kernel<E, TB><<<dim3((unsigned)(a.blocks_nn + a.blocks_tn + a.sums.count * a.blocks_sum)), 64 * WAVES, smem, st>>>(a);
  return check_launch();
}

// What a problem costs on tiles of TB rows: rounds of 256 workgroups, us of one workgroup's sum over K.
struct Work {
  double rounds, chain;
  Work(int64_t tb, int64_t M, int64_t N, double chain_) : rounds((double)((M + tb - 1) / tb) * (double)((N + tb - 1) / tb) / 256), chain(chain_) {}
};

}  // namespace

// Whether these kernels can take a problem: whole 16-byte units along every row, whole dwords, and slabs whose rows the 32-bit DMA
// offsets reach.
bool gemm_wave_takes(int dtype, int layout, int64_t M, int64_t N, int64_t K, const void *A, const void *B, const void *C,
                     const void *bias, const void *aux) {
  const int64_t es = dtype == MTNLG_F32 ? 4 : 2, unit = 16 / es;
  const bool at = layout == MTNLG_GEMM_TN, bt = layout != MTNLG_GEMM_NT;
  if ((at ? M : K) % unit || (bt ? N : K) % unit || N % unit) return false;
  if (((uintptr_t)A | (uintptr_t)B | (uintptr_t)C | (uintptr_t)bias | (uintptr_t)aux) & 3) return false;
  const int64_t reach_a = at ? 128 / es * M * es : 64 * K * es, reach_b = bt ? 128 / es * N * es : 64 * K * es;
  return reach_a < (int64_t)RECORDS - 256 && reach_b < (int64_t)RECORDS - 256;
}

// Estimated microseconds, fitted to 150 bf16 problems (graph replays, weights not in the caches) and 270 fp32 ones (the choice between all
// four kernels then cost 0.6 % on average against the best, 19 % at most; 600 others since: 1.4 %, 28 % at most, 768 x 3072 x 2048).  A workgroup's chain is launch, K / 8 and merge; beyond
// 256 workgroups the tiles queue for the L2's bandwidth (bf16) or the matrix and vector pipes (fp32, whose cutting into parts adds to the
// MFMAs).  Measured us, bf16, streaming kernel / 32 / 64: 256 x 512 x 1024 10.6 / 4.5 / 7.0; 512 x 512 x 4096 32 / 8.6 / 15.6;
// 1024 x 1024 x 4096 38 / 24 / 16.5; 1024 x 2048 x 2048 21 / 38 / 20; 2048 x 2048 x 64 5.5 / 16 / 13.
// fp32, operands straight to registers / 32 / 64 / 128 (gemm_parts.hip): 128 x 960 x 512 13 / 5.6 / 11 / 26; 1024 x 1024 x 4096 69 / 71 / 60 /
// 160; 1024 x 4096 x 1024 71 / 72 / 65 / 51, TN 58 / 71 / 65 / 50; 2048 x 2048 x 4096 242 / 268 / 208 / 179; 1600 x 2048 x 3000 147 / 169 / 152 / 120.
static void wave_times(int dtype, int layout, int64_t M, int64_t N, int64_t K, double &us32, double &us64) {
  const double k = (double)K;
  const double t32 = Work(32, M, N, 0).rounds, t64 = Work(64, M, N, 0).rounds;
  const double r32 = t32 > 1 ? t32 : 1, r64 = t64 > 1 ? ceil(t64) : 1;
  if (dtype == MTNLG_F32) {
    const double halves = t32 > 1 ? ceil(2 * t32) / 2 : 1;   // rounds of two workgroups on a compute unit
    us32 = 4.05 + halves * 0.0037 * k + (halves - 1) * 1.16 + 0.00028 * k;
    us64 = r64 * (7.0 + 0.0116 * k);   // (TN took 1.17 times as long while it spilled)
  } else {
    us32 = 2.7 + r32 * k * (layout == MTNLG_GEMM_NT ? 0.0014 : layout == MTNLG_GEMM_NN ? 0.0019 : 0.0023) + (r32 - 1) * 0.85;
    us64 = 1.0 + r64 * (3.2 + k * (layout == MTNLG_GEMM_TN ? 0.0034 : 0.0028));
  }
}
int gemm_wave_pick(int dtype, int layout, int64_t M, int64_t N, int64_t K, double other) {
  double us32, us64;
  wave_times(dtype, layout, M, N, K, us32, us64);
  if (us32 > other && us64 > other) return 0;
  return us32 < us64 ? 32 : 64;
}

// The same for the two products of a group and its column sums: the longest chain where all workgroups run at once, else the chains
// spread over the compute units.
static int pick_group(int dtype, const GemmCall &nn, const GemmCall &tn, int64_t sum_rows, double separate) {
  const bool f32 = dtype == MTNLG_F32;
  auto time = [&](int tb, double launch, double tile, double c_nn, double c_tn) {
    const Work a(tb, nn.M, nn.N, c_nn * (double)nn.K), b(tb, tn.M, tn.N, c_tn * (double)tn.K);
    const double rounds = a.rounds + b.rounds, whole = tb == 64 ? ceil(rounds) : rounds > 1 ? rounds : 1;
    const double longest = fmax(fmax(a.chain, b.chain), 0.5 + 0.004 * (double)sum_rows);
    return launch + whole * tile + fmax(longest, (a.rounds * a.chain + b.rounds * b.chain) * whole / rounds);
  };
  const double us32 = f32 ? time(32, 2.9, 1.16, 0.0040, 0.0040) : time(32, 1.85, 0.85, 0.0019, 0.0023);
  const double us64 = f32 ? INFINITY : time(64, 1.0, 3.2, 0.0028, 0.0034);   // (fp32 on 64 x 64 tiles: both layouts in one kernel spill)
  if (us32 > separate && us64 > separate) return 0;
  return us32 < us64 ? 32 : 64;
}

int gemm_wave(int dtype, int layout, int64_t M, int64_t N, int64_t K, const void *A, const void *B, void *C, const void *bias,
              void *aux, uint32_t epi, int tile, hipStream_t stream) {
  if (layout < 0 || layout > 2 || M <= 0 || N <= 0 || K <= 0) return MTNLG_INVALID_ARG;
  if (!gemm_wave_takes(dtype, layout, M, N, K, A, B, C, bias, aux)) return MTNLG_UNSUPPORTED_SHAPE;
  const WaveGemmArgs a{M, N, K, layout == MTNLG_GEMM_TN ? M : K, layout == MTNLG_GEMM_NT ? K : N, A, B, C, EpiArgs{bias, aux, epi}, 0, 0};
  LaunchScope scope(MTNLG_K_GEMM_NT + layout, stream);
  if (dtype == MTNLG_F32) return tile == 32 ? launch_layout<float, 32>(layout, a, stream) : launch_layout<float, 64>(layout, a, stream);
  return tile == 32 ? launch_layout<bf16, 32>(layout, a, stream) : launch_layout<bf16, 64>(layout, a, stream);
}

// nn, tn: problems that mtnlg_gemm accepts; separate_nn, separate_tn: what a launch of its own is estimated to cost without these kernels.
// Forward and backward of a layer, us with separate launches / so (one launch for 3 to 4): 128 tokens, h 512, FFN 2048, bf16 107 / 76, fp32
// 144 / 110; 512 tokens 131 / 110, 231 / 197; 512 tokens, h 768, FFN 3072 180 / 145, 362 / 314.  By these estimates most larger ones stay
// separate (1000 tokens, h 1024: 277 / 274): the streaming kernels are faster there than what the launches cost.
int gemm_wave_group_tile(int dtype, const GemmCall &nn, const GemmCall &tn, int sums, int64_t sum_rows, int64_t sum_cols, double separate_nn,
                         double separate_tn) {
  if (!gemm_wave_takes(dtype, MTNLG_GEMM_NN, nn.M, nn.N, nn.K, nn.A, nn.B, nn.C, nullptr, nn.aux) ||
      !gemm_wave_takes(dtype, MTNLG_GEMM_TN, tn.M, tn.N, tn.K, tn.A, tn.B, tn.C, nullptr, tn.aux) || sum_cols % 8 ||
      Work(32, nn.M, nn.N, 0).rounds + Work(32, tn.M, tn.N, 0).rounds > 4096)
    return 0;
  double separate = sums == 0 ? 0.0 : sums > 1 ? 3.0 : 6.0;   // one kernel over partial sums, or two
  double us32, us64;
  wave_times(dtype, MTNLG_GEMM_NN, nn.M, nn.N, nn.K, us32, us64);
  separate += fmin(separate_nn, fmin(us32, us64));
  wave_times(dtype, MTNLG_GEMM_TN, tn.M, tn.N, tn.K, us32, us64);
  separate += fmin(separate_tn, fmin(us32, us64));
  return pick_group(dtype, nn, tn, sums ? sum_rows : 0, separate);
}

int gemm_wave_group(int dtype, const GemmCall &nn, const GemmCall &tn, const ColumnSums &sums, int tile, hipStream_t stream) {
  if (tile != 32 && (tile != 64 || dtype == MTNLG_F32)) return MTNLG_INVALID_ARG;
  const GroupArgs a{{nn.M, nn.N, nn.K, nn.K, nn.N, nn.A, nn.B, nn.C, EpiArgs{nullptr, nn.aux, nn.epi}, 0, 0},
                    {tn.M, tn.N, tn.K, tn.M, tn.N, tn.A, tn.B, tn.C, EpiArgs{nullptr, tn.aux, tn.epi}, 0, 0},
                    0, 0, sums, (int)((sums.C + 63) / 64)};
  LaunchScope scope(MTNLG_K_GEMM_NN, stream, MTNLG_K_GEMM_TN);   // the two products have the same number of operations
  if (dtype == MTNLG_F32) return launch_group<float, 32>(a, stream);
  return tile == 32 ? launch_group<bf16, 32>(a, stream) : launch_group<bf16, 64>(a, stream);
}

}  // namespace mtnlg
