// Shared declarations of the gfx950 layer-slice library: element types, status
// handling, launch bookkeeping.  Internal to the GPU library.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/mtnlg.h"

namespace mtnlg {

typedef __bf16 bf16;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;

// Storage <-> fp32.  float -> bf16 is round-to-nearest-even (v_cvt_pk_bf16_f32).
__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(bf16 v) { return (float)v; }
template <typename E> __device__ __forceinline__ E from_f32(float v);
template <> __device__ __forceinline__ float from_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16 from_f32<bf16>(float v) { return (bf16)v; }

// 8 consecutive elements as one unit (16 B for bf16, 32 B for float).
template <typename E> __device__ __forceinline__ void load8(const E *p, float (&out)[8]) {
  if constexpr (sizeof(E) == 2) {
    bf16x8 t = *reinterpret_cast<const bf16x8 *>(p);
#pragma unroll
    for (int i = 0; i < 8; ++i) out[i] = (float)t[i];
  } else {
    f32x4 a = *reinterpret_cast<const f32x4 *>(p);
    f32x4 b = *reinterpret_cast<const f32x4 *>(p + 4);
#pragma unroll
    for (int i = 0; i < 4; ++i) { out[i] = a[i]; out[4 + i] = b[i]; }
  }
}
// 4 consecutive elements as floats (16 bytes of float, 8 of bf16)
template <typename E>
__device__ __forceinline__ f32x4 load4(const E *p) {
  if constexpr (sizeof(E) == 4) {
    return *reinterpret_cast<const f32x4 *>(p);
  } else {
    const bf16x4 t = *reinterpret_cast<const bf16x4 *>(p);
    return f32x4{(float)t[0], (float)t[1], (float)t[2], (float)t[3]};
  }
}
template <typename E> __device__ __forceinline__ void store8(E *p, const float (&in)[8]) {
  if constexpr (sizeof(E) == 2) {
    bf16x8 t;
#pragma unroll
    for (int i = 0; i < 8; ++i) t[i] = (bf16)in[i];
    *reinterpret_cast<bf16x8 *>(p) = t;
  } else {
    f32x4 a, b;
#pragma unroll
    for (int i = 0; i < 4; ++i) { a[i] = in[i]; b[i] = in[4 + i]; }
    *reinterpret_cast<f32x4 *>(p) = a;
    *reinterpret_cast<f32x4 *>(p + 4) = b;
  }
}

// 8 consecutive elements as loaded
template <typename E> struct Raw8;
template <> struct Raw8<bf16> {
  bf16x8 v;
  __device__ __forceinline__ void load(const bf16 *p) { v = *reinterpret_cast<const bf16x8 *>(p); }
  __device__ __forceinline__ float operator[](int e) const { return (float)v[e]; }
};
template <> struct Raw8<float> {
  f32x4 a, b;
  __device__ __forceinline__ void load(const float *p) {
    a = *reinterpret_cast<const f32x4 *>(p);
    b = *reinterpret_cast<const f32x4 *>(p + 4);
  }
  __device__ __forceinline__ float operator[](int e) const { return e < 4 ? a[e] : b[e - 4]; }
};

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
  return v;
}

// Global -> LDS DMA (buffer_load ... lds): every lane moves 16 (or 4) bytes from base + its byte
// offset to LDS byte address lds_dst + 16 (or 4) * lane; lds_dst is the same for the whole wave.  Issued as
// inline assembly on purpose: once the compiler has seen such a write to LDS it makes the next LDS
// read it cannot tell apart from it wait for all outstanding memory operations, which empties a
// ring of several stages at every tile.  Kernels that use these count their outstanding DMAs
// themselves (s_waitcnt vmcnt(N) before the barrier that publishes a stage).  The LDS address
// travels in M0, which each statement declares as clobbered.
typedef __attribute__((ext_vector_type(4))) int dma_rsrc_t;
// base: the same in every lane; records: bytes the bounds check lets through, offsets beyond read zeros
__device__ __forceinline__ dma_rsrc_t dma_rsrc(const void *base, uint32_t records = 0xFFFFFFFFu) {
  const uint64_t a = (uint64_t)base;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a), hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
  return dma_rsrc_t{(int)lo, (int)(hi & 0xFFFF), (int)records, 0x00020000};
}
// LDS byte address of a pointer into shared memory (what M0 takes)
__device__ __forceinline__ uint32_t lds_address(const void *p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void *)p;
}
// The compiler keeps M0 out of register allocation ("reserved") and warns about it in a clobber list; the
// clobber is still what tells it that its own M0 initialisations do not survive these statements.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
// TAG only tells call sites apart: the compiler merges identical asm statements on the two sides
// of a branch into one burst in front of it, which is exactly what spreading them tries to avoid.
template <int TAG = 0>
__device__ __forceinline__ void dma16(dma_rsrc_t rs, uint32_t lds_dst, uint32_t byte_offset) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds ; site %3" ::"s"(
                   __builtin_amdgcn_readfirstlane(lds_dst)),
               "v"(byte_offset), "s"(rs), "n"(TAG)
               : "memory", "m0");
}
// ... with a further byte offset that is the same in every lane (a scalar register: instructions whose lane offsets
// differ by uniform amounts share one vector register)
template <int TAG = 0>
__device__ __forceinline__ void dma16(dma_rsrc_t rs, uint32_t lds_dst, uint32_t byte_offset, uint32_t uniform_offset) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %4 offen lds ; site %3" ::"s"(
                   __builtin_amdgcn_readfirstlane(lds_dst)),
               "v"(byte_offset), "s"(rs), "n"(TAG), "s"(__builtin_amdgcn_readfirstlane(uniform_offset))
               : "memory", "m0");
}
template <int TAG = 0>
__device__ __forceinline__ void dma4(dma_rsrc_t rs, uint32_t lds_dst, uint32_t byte_offset) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds ; site %3" ::"s"(
                   __builtin_amdgcn_readfirstlane(lds_dst)),
               "v"(byte_offset), "s"(rs), "n"(TAG)
               : "memory", "m0");
}

#pragma clang diagnostic pop

// GeLU in fp32.  tanh form: 0.5 z (1 + tanh(sqrt(2/pi) (z + 0.044715 z^3))); erf form:
// 0.5 z (1 + erf(z / sqrt 2)).
__device__ __forceinline__ float gelu_f(float z, bool erf_form) {
  if (erf_form) return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f));
  float inner = 0.79788456080286536f * (z + 0.044715f * z * z * z);
  return 0.5f * z * (1.0f + tanhf(inner));
}
__device__ __forceinline__ float gelu_grad_f(float z, bool erf_form) {
  if (erf_form) {
    float cdf = 0.5f * (1.0f + erff(z * 0.70710678118654752f));
    float pdf = __expf(-0.5f * z * z) * 0.39894228040143268f;
    return cdf + z * pdf;
  }
  float inner = 0.79788456080286536f * (z + 0.044715f * z * z * z);
  float th = tanhf(inner);
  float dinner = 0.79788456080286536f * (1.0f + 3.0f * 0.044715f * z * z);
  return 0.5f * (1.0f + th) + 0.5f * z * (1.0f - th * th) * dinner;
}

// The tanh form again for the epilogue of the bf16 MFMA GEMMs, where the library tanhf (some 40 instructions an
// element) would cost a 256 x 320 tile 25 us of vector ALU time with the matrix pipes idle.  With
// s = 1 / (1 + exp(-2 u)), u = sqrt(2/pi) (z + 0.044715 z^3):  0.5 (1 + tanh u) = s, so GeLU(z) = z s and
// GeLU'(z) = s + 2 z u' s (1 - s), 1 - s = exp(-2 u) s.  Hardware exp2 and reciprocal (1 ulp each): relative error
// of a few 1e-7, two orders below the rounding of the bf16 result; no cancellation for very negative z, unlike
// 1 + tanh.  The exponent is clamped so that exp(-2 u) s stays finite.  8 and 13 instructions an element.
__device__ __forceinline__ float gelu_sigmoid_f(float z, float z2, float &e) {   // returns s, e = exp(-2 u)
  constexpr float K1 = -2.0f * 1.4426950408889634f * 0.79788456080286536f, K3 = K1 * 0.044715f;   // -2 u log2(e) = z (K1 + K3 z^2)
  e = __builtin_amdgcn_exp2f(fminf(z * (K1 + K3 * z2), 115.0f));
  return __builtin_amdgcn_rcpf(1.0f + e);
}
__device__ __forceinline__ float gelu_tanh_fast_f(float z) {
  float e;
  return z * gelu_sigmoid_f(z, z * z, e);
}
__device__ __forceinline__ float gelu_tanh_grad_fast_f(float z) {
  constexpr float D1 = 2.0f * 0.79788456080286536f, D3 = D1 * 3.0f * 0.044715f;   // 2 u' = D1 + D3 z^2
  const float z2 = z * z;
  float e;
  const float s = gelu_sigmoid_f(z, z2, e);
  return s + (z * (D1 + D3 * z2)) * (e * s) * s;
}

// GEMM epilogue shared by the GEMM kernels: bias, GeLU (pre-activation kept in aux),
// residual from aux, accumulate, fp32 or storage-dtype output.  One element at a time.
struct EpiArgs {
  const void *bias;
  void *aux;
  uint32_t flags;
};

template <typename E>
__device__ __forceinline__ void epilogue_store(const EpiArgs &ea, void *C, int64_t ldc, int64_t m,
                                               int64_t n, float acc) {
  if (ea.flags & MTNLG_EPI_BIAS) acc += to_f32(static_cast<const E *>(ea.bias)[n]);
  if (ea.flags & MTNLG_EPI_GELU) {
    static_cast<E *>(ea.aux)[m * ldc + n] = from_f32<E>(acc);
    acc = gelu_f(acc, (ea.flags & MTNLG_EPI_GELU_ERF) != 0);
  }
  if (ea.flags & MTNLG_EPI_RESIDUAL) acc += to_f32(static_cast<const E *>(ea.aux)[m * ldc + n]);
  if (ea.flags & MTNLG_EPI_GELU_GRAD)
    acc *= gelu_grad_f(to_f32(static_cast<const E *>(ea.aux)[m * ldc + n]), (ea.flags & MTNLG_EPI_GELU_ERF) != 0);
  if (ea.flags & MTNLG_EPI_OUT_F32) {
    float *c = static_cast<float *>(C) + m * ldc + n;
    *c = (ea.flags & MTNLG_EPI_ACCUMULATE) ? *c + acc : acc;
  } else {
    E *c = static_cast<E *>(C) + m * ldc + n;
    *c = from_f32<E>((ea.flags & MTNLG_EPI_ACCUMULATE) ? to_f32(*c) + acc : acc);
  }
}

template <bool FAST> __device__ __forceinline__ float gelu_of(float z, bool erf_form) {
  if constexpr (FAST) { if (!erf_form) return gelu_tanh_fast_f(z); }
  return gelu_f(z, erf_form);
}
template <bool FAST> __device__ __forceinline__ float gelu_grad_of(float z, bool erf_form) {
  if constexpr (FAST) { if (!erf_form) return gelu_tanh_grad_fast_f(z); }
  return gelu_grad_f(z, erf_form);
}
// 4 consecutive outputs of row m at column n (n + 3 < N and everything aligned for 4-element accesses).  FAST: the forms of the streaming
// bf16 kernels, for problems that those take too; they do not reach the limits for |z| of 10^13 and above, which the library's tanhf does.
template <typename E, bool FAST = sizeof(E) == 2>
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
    for (int e = 0; e < 4; ++e) v[e] = gelu_of<FAST>(v[e], (ea.flags & MTNLG_EPI_GELU_ERF) != 0);
  }
  if (ea.flags & (MTNLG_EPI_RESIDUAL | MTNLG_EPI_GELU_GRAD)) {
    const f32x4 t = load4(static_cast<const E *>(ea.aux) + off);
    if (ea.flags & MTNLG_EPI_RESIDUAL) {
      v += t;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] *= gelu_grad_of<FAST>(t[e], (ea.flags & MTNLG_EPI_GELU_ERF) != 0);
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

// One operand of v_mfma_f32_16x16x32_bf16 in N parts that add up to the 8 values of a chunk: bf16 elements are one part, fp32
// elements three, each the rounded rest of the ones before it (8 + 8 + 8 bits: the rest after three is zero; fp32 products from bf16 ones in
// this way: Henry, Tang, Heinecke, "Leveraging the bfloat16 artificial intelligence datatype for higher-precision computations", 2019).
// Three parts are those of the value times PARTS_SCALE, with which the last bit of the smallest fp32 value, 2^-149, is a normal bf16
// value: cut as they are, values lose digits from about 2^-110 down, which a sum does not show if the other factor is large (A about 2^-118,
// B 2^60: results off by 9e-6).  Values of 2^104 and above have no such parts, their sums are not finite (parts_hold).
constexpr float PARTS_SCALE = 0x1p24f, PARTS_UNSCALE = 0x1p-24f;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
template <int N>
struct Parts {
  bf16x8 p[N];
  __device__ __forceinline__ void of(const float (&x)[8]) {
    // (-1, 0) and (0, -1); in registers, because the compiler writes the first as the inline constant of 32 bits, which is the second
    unsigned first = 0xBF80u, second = 0xBF800000u;
    asm("" : "+s"(first), "+s"(second));
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
      float lo = N > 1 ? x[e] * PARTS_SCALE : x[e], hi = N > 1 ? x[e + 1] * PARTS_SCALE : x[e + 1];
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const bf16x2 t = {(bf16)lo, (bf16)hi};
        p[i][e] = t[0];
        p[i][e + 1] = t[1];
        if (i + 1 < N) {   // the rest in one instruction a value
          lo = __builtin_amdgcn_fdot2_f32_bf16(t, __builtin_bit_cast(bf16x2, first), lo, false);
          hi = __builtin_amdgcn_fdot2_f32_bf16(t, __builtin_bit_cast(bf16x2, second), hi, false);
        }
      }
    }
  }
};
// The product of a block in parts: fp32 sums of products that are exact.  Of three parts each way the six largest products; what is
// left out is at most 2^-24 of the product of the two values (second parts are up to 2^-8 of a value, third ones 2^-17).  The largest (step 0) and the other five (steps 1 .. 5) belong in separate
// accumulators: the matrix instructions round a product down to the last bits of a much larger accumulator, and in one
// accumulator the small products moved every result by -2e-8 to -1e-7 of the typical one (1024 x 1024 x 1024 to 4096), which a sum over
// the rows of the result shows (7.6e-7 instead of 3.1e-7 with fp32 instructions, and 1.7e-7 so).
template <int N>
__device__ __forceinline__ f32x4 mma_parts(const Parts<N> &b, const Parts<N> &a, f32x4 acc, int step) {
  constexpr int PB[6] = {0, 2, 0, 1, 1, 0}, PA[6] = {0, 0, 2, 1, 0, 1};
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(b.p[N == 1 ? 0 : PB[step]], a.p[N == 1 ? 0 : PA[step]], acc, 0, 0, 0);
}
// Whether a sum of such products is what fp32 products would give: the parts cannot say an infinity, nor a value of 2^104 and above (the
// rest of an infinite part is NaN), and scaled sums end at 2^80.  A sum that holds is taken back by parts_sum.
__device__ __forceinline__ bool parts_hold(float sum) { return fabsf(sum) < INFINITY; }
__device__ __forceinline__ f32x4 parts_sum(f32x4 scaled) { return scaled * (PARTS_UNSCALE * PARTS_UNSCALE); }

// ---- host side -------------------------------------------------------------
// Brackets a launch with HIP events when per-class timing is on (profile.cpp).
struct LaunchScope {
  int cls;
  hipStream_t stream;
  long idx;  // slot in the record list, -1 when timing is off
  LaunchScope(int cls_, hipStream_t s, int also = -1);   // also: a second class that does as much of the launch's work
  ~LaunchScope();
};

inline int check_launch() { return hipGetLastError() == hipSuccess ? MTNLG_OK : MTNLG_HIP_ERROR; }

// Kernel attributes (dynamic LDS size) are set once per device and kernel: `done` is a bit mask of
// the devices on which the attribute of one kernel has been set (devices beyond 63 set it every time).
// Thread-safe; a race sets the attribute twice, which is harmless.
inline bool attr_is_set(unsigned long long &done, int *device) {
  if (hipGetDevice(device) != hipSuccess) { *device = -1; return false; }
  if (*device < 0 || *device > 63) return false;
  return (__atomic_load_n(&done, __ATOMIC_ACQUIRE) >> *device) & 1ull;
}
inline void attr_mark_set(unsigned long long &done, int device) {
  if (device >= 0 && device <= 63) __atomic_fetch_or(&done, 1ull << device, __ATOMIC_RELEASE);
}

#define MTNLG_TRY(expr)            \
  do {                             \
    int st__ = (expr);             \
    if (st__ != MTNLG_OK) return st__; \
  } while (0)

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// internal launchers shared between translation units
constexpr int64_t GEMM_GENERIC_MAX_ROWS = 65535 * 64;
int gemm_generic(int dtype, int layout, int64_t M, int64_t N, int64_t K, const void *A,
                 const void *B, void *C, const void *bias, void *aux, uint32_t epi,
                 hipStream_t stream);
double gemm_mfma_time(int layout, int64_t M, int64_t N, int64_t K, size_t ws_bytes);   // estimated microseconds of that tile
bool gemm_wave_takes(int dtype, int layout, int64_t M, int64_t N, int64_t K, const void *A, const void *B, const void *C,
                     const void *bias, const void *aux);
// One product of a linear layer's backward pass, row lengths as of dense matrices; and sums over the rows of up to three dense [rows][C]
// matrices, fp32 or bf16 in and out, up to 64 columns to a workgroup.
struct GemmCall {
  int64_t M, N, K;
  const void *A, *B;
  void *C, *aux;
  uint32_t epi;
};
struct ColumnSum {
  const void *in;
  void *out;
};
struct ColumnSums {
  int count;
  int64_t rows, C;
  bool in_f32, out_f32, accumulate;
  ColumnSum of[3];
};
// One launch for both products and the sums: which tile it would take (32 or 64), 0 where separate launches are estimated to be faster or
// have to be taken; sums: how many matrices, of how many rows and columns
int gemm_wave_group_tile(int dtype, const GemmCall &nn, const GemmCall &tn, int sums, int64_t sum_rows, int64_t sum_cols, double separate_nn,
                         double separate_tn);
int gemm_wave_group(int dtype, const GemmCall &nn, const GemmCall &tn, const ColumnSums &sums, int tile, hipStream_t stream);
// LayerNorm backward without the sums over rows; left: what is to be added up afterwards, over so many rows at most
int layernorm_bwd_rows(int dtype, int64_t T, int64_t h, const void *x, const void *gamma, const float *mean, const float *rstd,
                       const void *dout, const void *dres, void *dx, void *dgamma, void *dbeta, void *colsum_dx, int grad_f32,
                       int accumulate, void *workspace, ColumnSums *left, hipStream_t stream);
int layernorm_bwd_most_sums(int64_t T);
int gemm_wave(int dtype, int layout, int64_t M, int64_t N, int64_t K, const void *A, const void *B, void *C, const void *bias,
              void *aux, uint32_t epi, int tile, hipStream_t stream);   // tile: 32 or 64
// fp32 problems that gemm_wave_takes, on 128 x 128 tiles
double gemm_parts_time(int64_t M, int64_t N, int64_t K);
int gemm_parts(int layout, int64_t M, int64_t N, int64_t K, const void *A, const void *B, void *C, const void *bias, void *aux, uint32_t epi,
               hipStream_t stream);
// the faster of the two tiles if it is estimated below `other` microseconds, else 0
int gemm_wave_pick(int dtype, int layout, int64_t M, int64_t N, int64_t K, double other);
double gemm_generic_time(int layout, int64_t M, int64_t N, int64_t K);   // of an fp32 problem on 64 x 64 tiles
double gemm_direct_time(int64_t M, int64_t N, int64_t K);   // ... on the fp32 instructions, infinite for sums that these are not for
bool gemm_generic_small_tile(int layout, int64_t M, int64_t N);   // 32 x 32 tiles, not 64 x 64, where accesses are aligned: fp32
bool gemm_generic_small_tile_bf16(int layout, int64_t M, int64_t N);
// returns MTNLG_UNSUPPORTED_SHAPE when the MFMA kernel cannot take this problem
// ws (nullable): scratch for the split-K tail, see gemm_mfma_workspace_bytes
// prof_class: kernel class the launch is timed under (-1: MTNLG_K_GEMM_NT + layout)
// tile: one of gemm_tile, or -1 to let gemm_mfma_pick_tile choose (what every product call does)
enum gemm_tile { GEMM_TILE_STREAM_256x256 = 0, GEMM_TILE_STREAM_256x320, GEMM_TILE_RAGGED_256, GEMM_TILE_RAGGED_128,
                 GEMM_TILE_RAGGED_128_DEEP };
int gemm_mfma_bf16(int layout, int64_t M, int64_t N, int64_t K, const void *A, const void *B,
                   void *C, const void *bias, void *aux, uint32_t epi, void *ws, size_t ws_bytes,
                   hipStream_t stream, int prof_class = -1, int tile = -1);
int gemm_mfma_pick_tile(int layout, int64_t M, int64_t N, int64_t K, size_t ws_bytes);
size_t gemm_mfma_workspace_bytes(int64_t M, int64_t N, int64_t K);
int attention_fwd_f32(int dtype, int b, int s, int n, int d, float scale, const void *qkv,
                         void *a, float *lse, hipStream_t stream);
int attention_bwd_f32(int dtype, int b, int s, int n, int d, float scale, const void *qkv,
                         const void *a, const float *lse, const void *da, void *dqkv, void *ws,
                         hipStream_t stream);

// MFMA attention (bf16): which head sizes it takes, its scratch need, its launchers
bool attention_mfma_supported(int dtype, int d);
// ... and whether it takes this problem (grid limits, 32-bit byte offsets inside one sequence)
bool attention_mfma_takes(int dtype, int b, int s, int n, int d);
constexpr int ATTENTION_F32_MAX_SEQ = 4096;   // sequence limit of the fp32 matrix-instruction kernels
size_t attention_bwd_workspace_bytes(int b, int s, int n, int d);
int attention_fwd_mfma(int b, int s, int n, int d, float scale, const void *qkv, void *a, float *lse,
                       hipStream_t stream);
int attention_bwd_mfma(int b, int s, int n, int d, float scale, const void *qkv, const void *a,
                       const float *lse, const void *da, void *dqkv, void *ws, hipStream_t stream);
// ... with P and dS in fp32, for the other head sizes (bf16): whether these kernels are the faster ones, and can take the call
bool attention_exact_fwd_takes(int dtype, int b, int s, int n, int d, const void *qkv, const void *a);
bool attention_exact_bwd_takes(int dtype, int b, int s, int n, int d, const void *qkv, const void *a, const void *da, const void *dqkv);
int attention_fwd_exact(int b, int s, int n, int d, float scale, const void *qkv, void *a, float *lse, hipStream_t stream);
int attention_bwd_exact(int b, int s, int n, int d, float scale, const void *qkv, const void *a, const float *lse, const void *da,
                        void *dqkv, void *ws, hipStream_t stream);
// 16 rows to a wave (attention_fwd16.hip, attention_bwd64.hip), called by those above where that is the faster
int attention_fwd_mfma16(int b, int s, int n, int d, float scale, const void *qkv, void *a, float *lse, hipStream_t stream);   // of head sizes 64, 128, 160
int attention_fwd_exact16(int b, int s, int n, int d, float scale, const void *qkv, void *a, float *lse, hipStream_t stream);
int attention_bwd64(int b, int s, int n, float scale, const void *qkv, const void *a, const float *lse, const void *da, void *dqkv, void *ws,
                    hipStream_t stream);   // of head size 64
int attention_bwd_exact64(int b, int s, int n, int d, float scale, const void *qkv, const void *a, const float *lse, const void *da, void *dqkv,
                          void *ws, hipStream_t stream);

}  // namespace mtnlg
