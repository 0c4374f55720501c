// GEMMs of the layer (paper appendix: QKV, attention output projection, MLP h->4h/t and 4h/t->h, and
// for each the input-gradient and weight-gradient products of the backward pass).
//
//   mode NN: C[M,N] = A[M,K] B[K,N]          forward      Y  = X W
//   mode NT: C[M,N] = A[M,K] B[N,K]^T        input grad   dX = dY W^T
//   mode TN: C[M,N] = A[K,M]^T B[K,N]        weight grad  dW = X^T dY
//
// bf16 path (gfx950): v_mfma_f32_16x16x32_bf16, 256 x 256 block tile, two LDS stages of 64 k filled by direct
// global->LDS loads, two groups of waves that alternate between the matrix cores and memory.  An operand whose
// reduction index is the slow memory index (B in NN, both in TN) stays in its memory order in LDS and is gathered
// into MFMA fragments by transposing LDS reads.
// fp32 path: v_mfma_f32_32x32x2_f32, operands straight from memory (small configurations).
#include "colsum.h"
#include "gelu.h"
#include <type_traits>

namespace ptdp {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;

// ------------------------------------------------------------------------------------------------
// fp32: v_mfma_f32_32x32x2_f32 (fp32 products and sums), operands straight from memory into fragments.  A workgroup is
// KG waves on one tile of 32 NB x 32 NB outputs; wave w takes the 32-wide k-chunks w, w + KG, ... and the partial tiles
// are added in LDS in wave order.  Lane (r = lane & 31, half = lane >> 5) carries k 8 q + 4 half + e of row r in element
// e of group q: the product's k order is free as long as both operands share it, and a k-contiguous row then gives one
// 16-byte load per group.  The next chunk is requested before the current one is multiplied.  fp32 calls are small and
// bound by one wave's chain of loads; before, by the k-steps of the few workgroups that 64 x 64 tiles of plain FMAs gave.
// us: 256 x 256 x 256 40 -> 4.2; 1024 x 1024 x 1024 191 -> 30; 4096 x 4096 x 1024 730 -> 358.
// VA, VB: the operand's rows are k-contiguous, 16-byte aligned and a multiple of four long; otherwise any strides.
// ------------------------------------------------------------------------------------------------
constexpr int kF32Chunk = 32;
template <bool V> struct F32Operand {
  const float* row;
  size_t ks;   // k stride (V: 1)
  // CLIP: k from kend on are zeros
  template <bool CLIP> __device__ __forceinline__ void load(f32x4_t (&f)[4], int k0, int half, int kend) const {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int k = k0 + 8 * q + 4 * half;
      if (V) {
        if (CLIP && k >= kend) f[q] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        else f[q] = *reinterpret_cast<const f32x4_t*>(row + k);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (CLIP && k + e >= kend) f[q][e] = 0.f;
          else f[q][e] = row[(size_t)(k + e) * ks];
        }
      }
    }
  }
};
constexpr int f32_most_waves(int nb) { return nb == 1 ? 8 : 4; }   // waves that share a tile's k range

// What an output stage does beside writing C.  EPI_GELU (NN): C = A B and g = GeLU(C + b).  EPI_GELU_GRAD (NT): C = (A B^T) * GeLU'(z + b), and
// the column sums of C over blocks of rows to part[block][N].  Both from what a kernel of its own would read: the product as it is stored.
// EPI_BDA (NN, bf16): C = z + Drop(A B + b), the residual sum behind the last layer's second MLP product.
enum { EPI_PLAIN = 0, EPI_GELU = 1, EPI_GELU_GRAD = 2, EPI_BDA = 3 };
template <int KIND, int MODE = PTDP_GELU_ERF> struct Epi {   // MODE: PTDP_GELU_*
  static constexpr int kKind = KIND, kMode = MODE;
};
template <typename T> struct GeluArgs {
  const T *b, *z;
  T* g;
  float* part;
  uint64_t key;   // EPI_BDA: of the dropout
  uint32_t thr;
  float scale;
};
// One tile by the workgroup's first kg waves.  SOME: there may be more, which only take part in the end.
template <bool VA, bool VB, int NB, bool SOME, class EPI>
__device__ __forceinline__ void gemm_f32_tile(const float* __restrict__ A, const float* __restrict__ B, float* C, const float* __restrict__ bias,
                                              int M, int N, int K, size_t a_rs, size_t a_cs, size_t b_rs, size_t b_cs, int accumulate,
                                              int tile_m, int tile_n, int kg, float* part, const GeluArgs<float>& e) {
  constexpr int kTile = 32 * NB, kPitch = kTile + 8;   // rows 4 apart (the two halves of a register) in different banks
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, l31 = lane & 31, half = lane >> 5;
  const int m0 = tile_m * kTile, n0 = tile_n * kTile;
  F32Operand<VA> oa[NB];
  F32Operand<VB> ob[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) {   // rows past the end repeat the last one: their outputs are not written
    oa[i].row = A + (size_t)min(m0 + i * 32 + l31, M - 1) * a_rs;
    oa[i].ks = a_cs;
    ob[i].row = B + (size_t)min(n0 + i * 32 + l31, N - 1) * b_cs;
    ob[i].ks = b_rs;
  }
  f32x16_t acc[NB][NB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  f32x4_t fa[2][NB][4], fb[2][NB][4];
  const int step = kg * kF32Chunk;
  auto load = [&](int set, int k) {
    if (k >= K) return;
    if (k + kF32Chunk <= K) {
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        oa[i].template load<false>(fa[set][i], k, half, K);
        ob[i].template load<false>(fb[set][i], k, half, K);
      }
    } else {
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        oa[i].template load<true>(fa[set][i], k, half, K);
        ob[i].template load<true>(fb[set][i], k, half, K);
      }
    }
  };
  auto multiply = [&](int set) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
          for (int j = 0; j < NB; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[set][i][q][e], fb[set][j][q][e], acc[i][j], 0, 0, 0);
  };
  int k = !SOME || wave < kg ? wave * kF32Chunk : K;
  load(0, k);
  // What the output stage reads at a thread's first places, requested behind the first chunk: its trip to memory would come last.  At
  // clamped addresses: under a condition the compiler waits for it at once (one layer of 256 x 256 97.0 us without, 95.1 so, 98.1 under one).
  constexpr int kAhead = NB == 1 ? 2 : 0;
  float ahead[kAhead > 0 ? kAhead : 1];
  if (EPI::kKind == EPI_GELU_GRAD || accumulate) {
    const float* from = EPI::kKind == EPI_GELU_GRAD ? e.z : C;
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int x = threadIdx.x + u * blockDim.x;
      ahead[u] = from[(size_t)min(m0 + x / kTile, M - 1) * N + min(n0 + x % kTile, N - 1)];
    }
  }
  for (; k < K; k += 2 * step) {
    load(1, k + step);
    multiply(0);
    if (k + step >= K) break;
    load(0, k + 2 * step);
    multiply(1);
  }
  float* mine = part + wave * (kTile * kPitch);
  if (!SOME || wave < kg) {
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) mine[(i * 32 + 8 * (r >> 2) + 4 * half + (r & 3)) * kPitch + j * 32 + l31] = acc[i][j][r];
  }
  __syncthreads();
  auto finish = [&](int x, auto read) {
    const int r = x / kTile, c = x % kTile, m = m0 + r, n = n0 + c;
    if (m >= M || n >= N) return;
    float v = 0.f;
    for (int w = 0; w < kg; ++w) v += part[w * (kTile * kPitch) + r * kPitch + c];
    if (bias) v += bias[n];
    const size_t at = (size_t)m * N + n;
    if (EPI::kKind == EPI_GELU_GRAD) {
      v *= gelu_grad_f<EPI::kMode>(read(e.z, at) + e.b[n]);
      part[r * kPitch + c] = v;   // in the place that this thread alone has read
      C[at] = v;
    } else {
      C[at] = accumulate ? read(C, at) + v : v;
    }
    if (EPI::kKind == EPI_GELU) e.g[at] = gelu_f<EPI::kMode>(v + e.b[n]);
  };
  int x = threadIdx.x;
#pragma unroll
  for (int u = 0; u < kAhead; ++u, x += blockDim.x)
    if (x < kTile * kTile) finish(x, [&](const float*, size_t) { return ahead[u]; });
  for (; x < kTile * kTile; x += blockDim.x) finish(x, [](const float* p, size_t at) { return p[at]; });
  if (EPI::kKind == EPI_GELU_GRAD) {   // a column's sum over the tile's rows: one column a thread, four sums of every fourth row
    __syncthreads();
    const int c = threadIdx.x, rows = min(kTile, M - m0);
    if (c < kTile && n0 + c < N) {
      float t[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int r = 0; r < kTile; ++r) t[r & 3] += r < rows ? part[r * kPitch + c] : 0.f;
      e.part[(size_t)tile_m * N + n0 + c] = (t[0] + t[1]) + (t[2] + t[3]);
    }
  }
}
template <bool VA, bool VB, int NB, class EPI = Epi<EPI_PLAIN>>
__global__ void __launch_bounds__(64 * f32_most_waves(NB))
gemm_f32_kernel(const float* __restrict__ A, const float* __restrict__ B, float* C, const float* __restrict__ bias,
                int M, int N, int K, size_t a_rs, size_t a_cs, size_t b_rs, size_t b_cs, int accumulate, GeluArgs<float> e) {
  extern __shared__ __attribute__((aligned(16))) float part[];
  gemm_f32_tile<VA, VB, NB, false, EPI>(A, B, C, bias, M, N, K, a_rs, a_cs, b_rs, b_cs, accumulate, blockIdx.y, blockIdx.x, blockDim.x >> 6, part, e);
}

// The same on one 16 x 16 tile (v_mfma_f32_16x16x4_f32), for outputs of fewer 32 x 32 tiles than the chip has compute units, where
// the matrix work of a tile is what its compute unit takes: four times as many workgroups.  Lane (r = lane & 15, q = lane >> 4)
// carries k 16 g + 4 q + e of row r in element e of group g.  Four k-chunks of a wave are requested at a time.
// us before and now, NN: 256 x 256 x 768 9.0 -> 4.5, x 1024 11.3 -> 5.2, 48 x 1536 x 512 6.8 -> 5.3, 128 x 512 x 2048 20.6 -> 8.5, 333 x 320 x
// 1280 14.2 -> 10.4.  Errors against 64 bits are the same.
template <bool V> struct F32Operand16 {
  const float* row;
  size_t ks;   // k stride (V: 1)
  __device__ __forceinline__ void load(f32x4_t (&f)[2], int k0, int q, int K) const {   // k from K on are zeros
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      const int k = k0 + 16 * g + 4 * q;
      if (V) {
        f[g] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        if (k < K) f[g] = *reinterpret_cast<const f32x4_t*>(row + k);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) f[g][e] = k + e < K ? row[(size_t)(k + e) * ks] : 0.f;
      }
    }
  }
};
constexpr int kF32TinyWaves = 8, kF32TinyAhead = 4;
template <bool VA, bool VB, class EPI>
__device__ __forceinline__ void gemm_f32_tiny_tile(const float* __restrict__ A, const float* __restrict__ B, float* C, const float* __restrict__ bias,
                                                   int M, int N, int K, size_t a_rs, size_t a_cs, size_t b_rs, size_t b_cs, int accumulate,
                                                   int tile_m, int tile_n, float (*part)[16][17], const GeluArgs<float>& e) {
  static_assert(EPI::kKind != EPI_GELU_GRAD, "the partial column sums have room for one row per 32 rows");
  // kg is kF32TinyWaves, read from the launch: as a constant the loops come out 1.5 % slower (a fp32 layer of 66 x 768)
  const int wave = threadIdx.x >> 6, kg = blockDim.x >> 6, lane = threadIdx.x & 63, l15 = lane & 15, q = lane >> 4;
  const int m0 = tile_m * 16, n0 = tile_n * 16;
  // rows past the end repeat the last one: their outputs are not written
  const F32Operand16<VA> oa{A + (size_t)min(m0 + l15, M - 1) * a_rs, a_cs};
  const F32Operand16<VB> ob{B + (size_t)min(n0 + l15, N - 1) * b_cs, b_rs};
  f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
  const int step = kg * kF32Chunk;
  const int x = threadIdx.x, m = m0 + (x >> 4), n = n0 + (x & 15);
  const size_t at = (size_t)m * N + n;
  const bool mine = x < 256 && m < M && n < N;
  float old = 0.f;   // requested ahead, as above
  if (accumulate) old = C[(size_t)min(m, M - 1) * N + min(n, N - 1)];
  for (int k = wave * kF32Chunk; k < K; k += kF32TinyAhead * step) {
    f32x4_t fa[kF32TinyAhead][2], fb[kF32TinyAhead][2];
#pragma unroll
    for (int u = 0; u < kF32TinyAhead; ++u) {
      if (k + u * step < K) {
        oa.load(fa[u], k + u * step, q, K);
        ob.load(fb[u], k + u * step, q, K);
      }
    }
#pragma unroll
    for (int u = 0; u < kF32TinyAhead; ++u) {
      if (k + u * step < K) {
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[u][g][e], fb[u][g][e], acc, 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) part[wave][4 * q + r][l15] = acc[r];
  __syncthreads();
  if (!mine) return;
  float v = 0.f;
  for (int w = 0; w < kg; ++w) v += part[w][x >> 4][x & 15];
  if (bias) v += bias[n];
  C[at] = accumulate ? old + v : v;
  if (EPI::kKind == EPI_GELU) e.g[at] = gelu_f<EPI::kMode>(v + e.b[n]);
}
template <bool VA, bool VB, class EPI = Epi<EPI_PLAIN>>
__global__ void __launch_bounds__(64 * kF32TinyWaves)
gemm_f32_tiny_kernel(const float* __restrict__ A, const float* __restrict__ B, float* C, const float* __restrict__ bias,
                     int M, int N, int K, size_t a_rs, size_t a_cs, size_t b_rs, size_t b_cs, int accumulate, GeluArgs<float> e) {
  __shared__ float part[kF32TinyWaves][16][17];
  gemm_f32_tiny_tile<VA, VB, EPI>(A, B, C, bias, M, N, K, a_rs, a_cs, b_rs, b_cs, accumulate, blockIdx.y, blockIdx.x, part, e);
}

// Weight gradients of one layer (C_j[M_j, N_j] += A_j^T B_j, sharing K) whose tiles have the same size as one launch: alone each is a
// few microseconds of a part of the chip.  A workgroup's tile, the number of waves that share its k range (kg) and so every bit of
// the result are those of a launch of its own.  A layer of 256 x 256 tokens: four launches 21.9 us, one 12.5 (the pass 130.3 -> 124.4).
constexpr int kMaxMultiF32 = 4;
struct MultiF32 {
  const float *A[kMaxMultiF32], *B[kMaxMultiF32];
  float* C[kMaxMultiF32];
  int M[kMaxMultiF32], N[kMaxMultiF32], kg[kMaxMultiF32], start[kMaxMultiF32], n, K;   // start: first workgroup
};
// sums: column sums that the launch's first n_sums workgroups finish, see gemm_bf16_small_multi_kernel.
template <bool TINY>
__global__ void __launch_bounds__(64 * f32_most_waves(1))
gemm_f32_multi_kernel(MultiF32 a, ColsumBatchArgs sums, int n_sums) {
  constexpr int kTile = TINY ? 16 : 32;
  extern __shared__ __attribute__((aligned(16))) float part[];
  const int id = (int)blockIdx.x - n_sums;
  if (id < 0) {
    colsum_finish_id(sums, id + n_sums, blockDim.x >> 6, part);
    return;
  }
  // constant indices only: the arguments stay in scalar registers
  const float *A = a.A[0], *B = a.B[0];
  float* C = a.C[0];
  int M = a.M[0], N = a.N[0], kg = a.kg[0], first = 0;
#pragma unroll
  for (int q = 1; q < kMaxMultiF32; ++q)
    if (q < a.n && id >= a.start[q]) {
      A = a.A[q]; B = a.B[q]; C = a.C[q];
      M = a.M[q]; N = a.N[q]; kg = a.kg[q]; first = a.start[q];
    }
  const int tiles_n = (N + kTile - 1) / kTile, t = id - first;
  if constexpr (TINY)
    gemm_f32_tiny_tile<false, false, Epi<EPI_PLAIN>>(A, B, C, nullptr, M, N, a.K, 1, M, N, 1, 1, t / tiles_n, t % tiles_n,
                                                reinterpret_cast<float (*)[16][17]>(part), {});
  else
    gemm_f32_tile<false, false, 1, true, Epi<EPI_PLAIN>>(A, B, C, nullptr, M, N, a.K, 1, M, N, 1, 1, t / tiles_n, t % tiles_n, kg, part, {});
}

template <bool VA, bool VB, int NB, class EPI = Epi<EPI_PLAIN>>
static int launch_gemm_f32_t(const float* A, const float* B, float* C, const float* bias, int M, int N, int K, size_t a_rs, size_t a_cs,
                             size_t b_rs, size_t b_cs, int accumulate, int kg, hipStream_t st, const GeluArgs<float>& e = {}) {
  auto kern = gemm_f32_kernel<VA, VB, NB, EPI>;
  constexpr int kTile = 32 * NB, kPart = kTile * (kTile + 8) * (int)sizeof(float);
  static once_flag_t done[kMaxDevices];
  if (set_dynamic_smem(reinterpret_cast<const void*>(kern), f32_most_waves(NB) * kPart, done) != PTDP_OK) return PTDP_E_HIP;
  hipLaunchKernelGGL(kern, dim3((N + kTile - 1) / kTile, (M + kTile - 1) / kTile), dim3(64 * kg), kg * kPart, st, A, B, C, bias, M, N, K,
                     a_rs, a_cs, b_rs, b_cs, accumulate, e);
  return PTDP_OK;
}
static int compute_units();
// 64 x 64 tiles (half the operand traffic) once they give every SIMD a wave, 32 x 32 before; up to 8 (4) waves share a
// tile's k range, fewer when the tiles alone fill the chip or the range has fewer chunks.  us with 32 x 32 and 64 x 64: 1024 x
// 1024 (256 tiles of 64 x 64) over k = 256 13.6, 13.2, over 1024 45, 29; 768 x 768 (144 tiles) 10.5, 13.0 and 33, 28.  16 waves
// per CU or 4: 512 x 512 x 1024 12.6, 11.4; 2048 x 2048 x 256 47, 36; 1536 x 1536 x 1024 81, 92; 3072 x 3072 x 1024 264, 264.
// 16 x 16 tiles up to two per compute unit, where a 32 x 32 tile's waves would have more than one k-chunk: 256 x 512 x 1024 (512
// tiles of 16 x 16) 11.6 -> 8.8; 500 x 288 x 1152 (576) 13.5 and 12.5 NN, 13.7 and 16.9 TN; 256 x 256 x 256 4.4 either way.  With more
// than one tile per compute unit smaller tiles pay only where they do not just read the long side of a thin output in shorter pieces:
// 1260 random calls with 257 to 512 tiles, time with 16 x 16 over time with 32 x 32 tiles, averages of outputs with a short side of
// up to 32, 33 to 64, 65 to 100:  NN with no more columns than rows 0.83, 0.88, 0.87;  others with k up to 512 0.92, 0.84, 0.86;  to 1024 NN
// and NT 1.00, 0.89, 0.88, TN 1.17, 0.99, 0.92;  to 4096 1.08, 1.02, 0.98;  beyond 1.08, 1.02, 0.95 (wider: 119 x 812 x 7783 TN 75, 81 us).
struct F32Form {
  int tile, kg;   // 16, 32 or 64 rows and columns; waves of a workgroup
};
static F32Form f32_form(bool va, bool vb, int M, int N, int K) {
  const long long ncu = compute_units(), t1 = (long long)((M + 31) / 32) * ((N + 31) / 32), t2 = (long long)((M + 63) / 64) * ((N + 63) / 64);
  const long long t16 = (long long)((M + 15) / 16) * ((N + 15) / 16);
  const int thin = M < N ? M : N;
  const bool two_rounds = (va && !vb && N <= M) || (thin > 64 && K <= 4096) || (thin > 32 && K <= (va ? 1024 : 512));
  if (K > kF32TinyWaves * kF32Chunk && (t16 <= ncu || (t16 <= 2 * ncu && two_rounds))) return {16, kF32TinyWaves};
  const bool big = t2 >= ncu;
  int kg = f32_most_waves(big ? 2 : 1);
  while (kg > 1 && (kg > (K + kF32Chunk - 1) / kF32Chunk || (big ? t2 : t1) * kg > 16 * ncu)) kg /= 2;
  return {big ? 64 : 32, kg};
}
template <bool VA, bool VB, class EPI = Epi<EPI_PLAIN>>
static int launch_gemm_f32(const float* A, const float* B, float* C, const float* bias, int M, int N, int K, size_t a_rs, size_t a_cs,
                           size_t b_rs, size_t b_cs, int accumulate, hipStream_t st, const GeluArgs<float>& e = {}) {
  const F32Form f = f32_form(VA, VB, M, N, K);
  if (f.tile == 16) {
    if constexpr (EPI::kKind == EPI_GELU_GRAD) return PTDP_E_STATE;   // the callers ask for the form first
    else
      hipLaunchKernelGGL((gemm_f32_tiny_kernel<VA, VB, EPI>), dim3((N + 15) / 16, (M + 15) / 16), dim3(64 * kF32TinyWaves), 0, st, A, B, C, bias, M, N,
                         K, a_rs, a_cs, b_rs, b_cs, accumulate, e);
    return PTDP_OK;
  }
  if (f.tile == 64) {
    if constexpr (EPI::kKind != EPI_PLAIN) return PTDP_E_STATE;
    else return launch_gemm_f32_t<VA, VB, 2>(A, B, C, bias, M, N, K, a_rs, a_cs, b_rs, b_cs, accumulate, f.kg, st);
  }
  return launch_gemm_f32_t<VA, VB, 1, EPI>(A, B, C, bias, M, N, K, a_rs, a_cs, b_rs, b_cs, accumulate, f.kg, st, e);
}

template <bool TINY> static int launch_f32_multi(const MultiF32& a, int blocks, const ColsumBatchArgs& sums, hipStream_t st) {
  constexpr int kPart = (TINY ? 16 * 17 : 32 * 40) * (int)sizeof(float);   // a wave's partial tile
  constexpr int kRed = kFinishRed * (int)sizeof(float);
  static once_flag_t done[kMaxDevices];
  if (set_dynamic_smem(reinterpret_cast<const void*>(gemm_f32_multi_kernel<TINY>), f32_most_waves(1) * kPart, done) != PTDP_OK) return PTDP_E_HIP;
  int kg = 1;
  for (int j = 0; j < a.n; ++j) kg = a.kg[j] > kg ? a.kg[j] : kg;
  const int n_sums = sums.first[kMaxColsumJobs], smem = n_sums > 0 && kg * kPart < kRed ? kRed : kg * kPart;
  static_assert(kRed <= f32_most_waves(1) * kPart, "within the limit set above");
  hipLaunchKernelGGL(gemm_f32_multi_kernel<TINY>, dim3(n_sums + blocks), dim3(64 * kg), smem, st, a, sums, n_sums);
  return PTDP_OK;
}
// Weight gradients of a layer: those of 16 x 16 tiles and those of 32 x 32 tiles as one launch each, 64 x 64 tiles (which fill the
// chip) one by one.  *sums: finished in the last of the shared launches (and then empty), if there is one.
static int launch_f32_tn_multi(int n, const void* const* A, const void* const* B, float* const* C, const int* M, const int* N, int K,
                               ColsumBatch* sums, hipStream_t st) {
  MultiF32 m[2];
  long long blocks[2] = {0, 0};
  for (int x = 0; x < 2; ++x) {
    m[x].n = 0;
    m[x].K = K;
  }
  for (int j = 0; j < n; ++j) {
    if (M[j] == 0 || N[j] == 0) continue;
    const float *a = (const float*)A[j], *b = (const float*)B[j];
    const F32Form f = f32_form(false, false, M[j], N[j], K);
    if (f.tile == 64) {
      const int rc = launch_gemm_f32_t<false, false, 2>(a, b, C[j], nullptr, M[j], N[j], K, 1, M[j], N[j], 1, 1, f.kg, st);
      if (rc != PTDP_OK) return rc;
      continue;
    }
    const int x = f.tile == 16 ? 0 : 1, q = m[x].n++;
    m[x].A[q] = a;
    m[x].B[q] = b;
    m[x].C[q] = C[j];
    m[x].M[q] = M[j];
    m[x].N[q] = N[j];
    m[x].kg[q] = f.kg;
    m[x].start[q] = (int)blocks[x];
    blocks[x] += (long long)((M[j] + f.tile - 1) / f.tile) * ((N[j] + f.tile - 1) / f.tile);
  }
  for (int x = 0; x < 2; ++x) {
    if (m[x].n == 0) continue;
    for (int q = m[x].n; q < kMaxMultiF32; ++q) {   // unused slots repeat the first (never selected)
      m[x].A[q] = m[x].A[0]; m[x].B[q] = m[x].B[0]; m[x].C[q] = m[x].C[0];
      m[x].M[q] = m[x].M[0]; m[x].N[q] = m[x].N[0]; m[x].kg[q] = m[x].kg[0]; m[x].start[q] = 0;
    }
    ColsumBatch none, *take = x == 0 && m[1].n > 0 ? &none : sums;
    double bytes = 0.0;
    const ColsumBatchArgs finish = colsum_batch_args(*take, &bytes);
    const int rc = x == 0 ? launch_f32_multi<true>(m[x], (int)blocks[x], finish, st) : launch_f32_multi<false>(m[x], (int)blocks[x], finish, st);
    if (rc != PTDP_OK) return rc;
    take->n = 0;
  }
  return PTDP_OK;
}

// ------------------------------------------------------------------------------------------------
// bf16 MFMA kernel: 256 x 256 x 64 block tile, 8 waves in two groups of four (one wave of each group per SIMD).
//
// LDS holds two stages of four half-tiles of 16 KiB (rows 0-127 and 128-255 of each operand, 64 k deep), filled by
// direct global->LDS loads (buffer_load ... lds, 16 bytes per lane, out-of-range lanes deliver zeros).
//   k-contiguous operand: [128 rows][8 chunks of 16 B]; chunk c of row r sits in slot c ^ ((r >> 1) & 7), so that the
//     16 neighbouring rows of one fragment read fall into 16 different 16-byte bank groups.
//   k-slow operand (memory [k][row]): [64 k][16 chunks of 16 B]; chunk c of k-row k sits in slot
//     c ^ (2 * (k & 3)) ^ (8 * ((k >> 3) & 1)): the k-rows that one transposing read gathers in a cycle (k & 3 and
//     (k >> 3) & 1 take all values) land in different bank groups.  MFMA fragments are gathered with
//     ds_read_b64_tr_b16: within 16 lanes, lane i receives element (i & 3) of the 8-byte rows addressed by lanes
//     (i >> 2) + {0, 4, 8, 12}.
// ------------------------------------------------------------------------------------------------
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4_t;
typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s16x8_t;
typedef __attribute__((address_space(3))) void lds_void_t;

constexpr uint32_t kOob = 0x80000000u;  // beyond any num_records this kernel accepts (< 2 GiB)

// Buffer descriptor (raw, no stride, no swizzle): 48-bit base, bytes, data format dword.
typedef uint32_t rsrc_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ rsrc_t make_rsrc(const void* p, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(p);
  rsrc_t r = {(uint32_t)a, (uint32_t)(a >> 32) & 0xffffu, bytes, 0x00020000u};
  return r;
}
__device__ __forceinline__ uint32_t lds_offset(const char* p) {
  return (uint32_t)reinterpret_cast<uintptr_t>((lds_void_t*)p);
}

// Global -> LDS loads (lane i lands at dst + 16*i; dst wave-uniform) are written as assembly: the compiler makes
// every LDS read that it cannot prove disjoint wait for every such load in flight.  The main loop orders these
// loads itself, by counted vmcnt waits and barriers.
__device__ __forceinline__ void load_lds_16(rsrc_t r, char* dst, uint32_t voff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
               :: "s"(lds_offset(dst)), "v"(voff), "s"(r) : "memory", "m0");
}
// two wave-loads whose destinations lie 1 KiB apart: the instruction's offset field moves the destination (and the
// source: the second lane offset passed in is 1024 bytes short); soff is added to the source only
__device__ __forceinline__ void load_lds_16x2(rsrc_t r, char* dst, uint32_t v0, uint32_t v1, uint32_t soff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
               "buffer_load_dwordx4 %1, %3, %4 offen lds\n\t"
               "buffer_load_dwordx4 %2, %3, %4 offen offset:1024 lds"
               :: "s"(lds_offset(dst)), "v"(v0), "v"(v1), "s"(r), "s"(soff) : "memory", "m0");
}

__device__ __forceinline__ void load_lds_16x4(rsrc_t r, char* dst, uint32_t v0, uint32_t v1, uint32_t v2, uint32_t v3, uint32_t soff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
               "buffer_load_dwordx4 %1, %5, %6 offen lds\n\t"
               "buffer_load_dwordx4 %2, %5, %6 offen offset:1024 lds\n\t"
               "buffer_load_dwordx4 %3, %5, %6 offen offset:2048 lds\n\t"
               "buffer_load_dwordx4 %4, %5, %6 offen offset:3072 lds"
               :: "s"(lds_offset(dst)), "v"(v0), "v"(v1), "v"(v2), "v"(v3), "s"(r), "s"(soff) : "memory", "m0");
}

constexpr int BK = 64;
constexpr int kBM = 256, kBN = 256, kGemmThreads = 512;
constexpr int kHalfBytes = 128 * BK * 2, kStageBytes = 4 * kHalfBytes, kGemmSmem = 2 * kStageBytes;

// A wave's share of one operand's half-tiles: two wave-loads of 1 KiB each (16 rows, or 8 k-rows, per wave).
// A k-tile that lies inside K whole is requested with as few instructions as the hardware allows: the lane offsets
// are loop constants and the k advance rides in the scalar offset (which the descriptor's bounds check excludes);
// the last, partial k-tile, tiles past the end (all lanes out of range) and operands with short rows take the
// general form with its per-lane checks.  Either way a call issues two loads: the main loop counts them.
// W: rows of a half-tile that exist.  128: half h is rows h * 128 + r of the block.  96 (of 192): rows of the block (r / 48) * 96 + h * 48 + r % 48,
// so that a wave's share of both halves is 96 neighbouring rows; the other 32 are out of range.
template <bool KSLOW, int W = 128> struct HalfLoad {
  __device__ __forceinline__ static int row_of_96(int h, int r) { return (r / 48) * 96 + h * 48 + r % 48; }
  uint32_t off[2][2];  // [half][load]: byte offset of the lane's chunk at k-tile 0 minus 1024 * load, or kOob if its row is out of range
  uint32_t kstep;      // byte advance per k-tile
  int kpos[2];         // k of the lane's chunk inside the k-tile
  bool plain;          // no offset above goes negative

  // the descriptor's base is the block's first row (k-contiguous: base + row0*ld; k-slow: base + row0)
  __device__ __forceinline__ void init(size_t ld, int rows_left, int wave, int lane) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      if (!KSLOW) {
        const int row = wave * 16 + i * 8 + (lane >> 3);
        const int chunk = (lane & 7) ^ ((row >> 1) & 7);
        kpos[i] = chunk * 8;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          if (W == 128) off[h][i] = h * 128 + row < rows_left ? (uint32_t)(((size_t)(h * 128 + row) * ld + chunk * 8) * 2) - i * 1024u : kOob;
          else off[h][i] = row < W && row_of_96(h, row) < rows_left ? (uint32_t)(((size_t)row_of_96(h, row) * ld + chunk * 8) * 2) - i * 1024u : kOob;
        }
      } else {
        const int k = wave * 8 + i * 4 + (lane >> 4);
        const int chunk = (lane & 15) ^ (2 * (k & 3)) ^ (8 * ((k >> 3) & 1));
        kpos[i] = k;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int at = row_of_96(h, chunk * 8);
          if (W == 128) off[h][i] = h * 128 + chunk * 8 < rows_left ? (uint32_t)(((size_t)k * ld + h * 128 + chunk * 8) * 2) - i * 1024u : kOob;
          else off[h][i] = chunk * 8 < W && at < rows_left ? (uint32_t)(((size_t)k * ld + at) * 2) - i * 1024u : kOob;
        }
      }
    }
    kstep = KSLOW ? (uint32_t)(BK * ld * 2) : (uint32_t)(BK * 2);
    plain = ld >= 128;   // row i*8 (k-row i*4) of a wave's share starts at least 1024 * i bytes into the block
  }
  // LEAN: the caller knows that the k-tile lies inside K whole and that plain is set
  template <int H, bool LEAN> __device__ __forceinline__ void issue(rsrc_t r, char* half, int wave, int kt, int kend) const {
    char* dst = half + wave * 2048;
    if (LEAN) {
      load_lds_16x2(r, dst, off[H][0], off[H][1], (uint32_t)kt * kstep);
    } else {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const bool ok = off[H][i] != kOob && kt * BK + kpos[i] < kend;
        load_lds_16(r, dst + i * 1024, ok ? off[H][i] + i * 1024u + (uint32_t)kt * kstep : kOob);
      }
    }
  }
};

// MFMA fragments of v_mfma_f32_16x16x32_bf16 for NB blocks of 16 rows starting at row w0 of a half-tile: lane & 15 is
// the row inside the block, lane >> 4 selects which 8 of the 32 k of step ks (0, 1) the lane carries.  One LDS address
// per stage and swizzle pattern; everything else is in the instructions' offset fields.
#define PTDP_LDS(T, addr) ((__attribute__((address_space(3))) T*)(uintptr_t)(addr))
template <bool KSLOW, int NB> struct FragRead {
  uint32_t base[2][KSLOW ? NB : 2];
  __device__ __forceinline__ void init(const char* smem, int w0, int lane) {
    const int r = lane & 15, G = lane >> 4;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const uint32_t stage = lds_offset(smem) + s * kStageBytes;
      if (!KSLOW) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) base[s][ks] = stage + (w0 + r) * 128 + (((ks * 4 + G) ^ (r >> 1)) * 16);
      } else {
#pragma unroll
        for (int i = 0; i < NB; ++i) {
          const int n0 = w0 + i * 16 + 4 * (r & 3), k = 8 * G + (r >> 2);
          base[s][i] = stage + k * 256 + (((n0 >> 3) ^ (2 * (r >> 2)) ^ (8 * (G & 1))) * 16) + (n0 & 7) * 2;
        }
      }
    }
  }
  // S: stage, at: byte offset of the half-tile in the stage
  template <int S> __device__ __forceinline__ bf16x8_t get(int at, int i, int ks) const {
    if (!KSLOW) {
      return *PTDP_LDS(const bf16x8_t, base[S][ks] + at + i * 2048);
    } else {
      const uint32_t p = base[S][i] + at + ks * (32 * 256);
      const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(PTDP_LDS(s16x4_t, p));
      const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(PTDP_LDS(s16x4_t, p + 4 * 256));
      const s16x8_t v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      return __builtin_bit_cast(bf16x8_t, v);
    }
  }
};

// Operands of one GEMM call as the kernels see them.  N is the number of columns this launch covers;
// ldb / ldc are the row lengths of the full B (k-slow form) and C, so that a launch may cover a column
// range of a larger problem.  a_end / b_end: one past the last byte of the operands (descriptor bounds).
struct GemmArgs {
  const bf16_t* A;
  const bf16_t* B;
  const bf16_t* bias;
  const char* a_end;
  const char* b_end;
  int M, N, K;
  size_t lda, ldb, ldc;
};

// A wave's outputs are NS strips of RB x 2 blocks of 16 x 16.  The MFMA's A operand is the B fragment, so that a lane
// holds row lane & 15 of a block and its four columns 4 * (lane >> 4) .. +3: consecutive in memory, written without a
// trip through LDS.  256 x 256 tile: strip 2*ha + hb covers rows ha*128 + (wave/4)*64 .. +63 and columns hb*128 +
// (wave%4)*32 .. +31.
template <int NS, int RB> using StripAcc = f32x4_t[NS][RB][2];
typedef StripAcc<4, 4> TileAcc;
template <int NS, int RB> __device__ __forceinline__ void zero_acc(StripAcc<NS, RB>& acc) {
#pragma unroll
  for (int b = 0; b < NS; ++b)
#pragma unroll
    for (int i = 0; i < RB; ++i) acc[b][i][0] = acc[b][i][1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
}

// acc += A[m0.., k] B[n0.., k] over k-tiles kt0 .. kt1-1.
// A k-tile is four phases, one per quadrant of the wave's outputs; a phase is a memory part (the LDS reads the
// phase needs, two global->LDS loads) and an arithmetic part (16 MFMAs, 256 cycles), with a barrier after each.  The
// second group of waves enters one barrier later, so that on every SIMD one wave computes while the other reads and
// requests: neither the requests' issue slots nor the reads' latency idle the matrix cores.  Bound by MFMA issue and the
// clock that power allows.  Measured against the form in which all eight waves were in the same part at a time (same
// box, random operands, TFLOP/s): NT 8192^3 1462 -> 1607, NN 1429 -> 1600, NN 2048 x 25600 x 12800 1372 -> 1535, NN
// 2048 x 12288 x 1536 1009 -> 1151, TN 8192^3 1313 -> 1403.  Touching the panels' lines of a later k-tile into L2 gained
// 7-12 % there and costs 2-3 % here: a request now has six phases (1.5 k-tiles) to land.
//   phase:     0             1             2             3
//   reads      A0(t)         B1(t)         A1(t)         B0(t+1)      (fragments)
//   requests   A1(t+1)       B0(t+2)       A0(t+2)       B1(t+2)      (half-tiles)
//   computes   A0 x B0       A0 x B1       A1 x B1       A1 x B0
// A half-tile is requested one phase after the phase in which every wave has finished reading its predecessor (two
// tiles older, same place) and is read six phases later; the wait in front of that read leaves the ten younger loads
// in flight (vmcnt counts loads in order), so the queue never drains inside the loop.
template <bool TA, bool TB>
__device__ __forceinline__ void gemm_mainloop(TileAcc& acc, const GemmArgs& g, int m0, int n0, int kt0, int kt1, char* smem) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;   // wave-uniform: LDS bases and M0 values stay in scalar registers
  // buffer descriptors start at the block's first row so that lane offsets stay small
  const bf16_t* a_base = TA ? g.A + m0 : g.A + (size_t)m0 * g.lda;
  const bf16_t* b_base = TB ? g.B + n0 : g.B + (size_t)n0 * g.ldb;
  const size_t a_left = (size_t)(g.a_end - reinterpret_cast<const char*>(a_base));
  const size_t b_left = (size_t)(g.b_end - reinterpret_cast<const char*>(b_base));
  const rsrc_t ra = make_rsrc(a_base, (uint32_t)(a_left < 0x7fffffffu ? a_left : 0x7fffffffu));
  const rsrc_t rb = make_rsrc(b_base, (uint32_t)(b_left < 0x7fffffffu ? b_left : 0x7fffffffu));
  const int kend = min(g.K, kt1 * BK);  // k-tiles from kt1 on read as zeros

  HalfLoad<TA> la;
  HalfLoad<TB> lb;
  la.init(g.lda, g.M - m0, wave, lane);
  lb.init(g.ldb, g.N - n0, wave, lane);
  FragRead<TA, 4> fa;
  FragRead<TB, 2> fb;
  fa.init(smem, (wave >> 2) * 64, lane);
  fb.init(smem, (wave & 3) * 32, lane);
  // byte offsets of the half-tiles in a stage: A0, A1, B0, B1
  constexpr int kA0 = 0, kA1 = kHalfBytes, kB0 = 2 * kHalfBytes, kB1 = 3 * kHalfBytes;

  // the requests of the phases before phase 0 of the first tile, in the loop's order
  lb.template issue<0, false>(rb, smem + kB0, wave, kt0, kend);
  la.template issue<0, false>(ra, smem + kA0, wave, kt0, kend);
  lb.template issue<1, false>(rb, smem + kB1, wave, kt0, kend);
  la.template issue<1, false>(ra, smem + kA1, wave, kt0, kend);
  lb.template issue<0, false>(rb, smem + kStageBytes + kB0, wave, kt0 + 1, kend);
  la.template issue<0, false>(ra, smem + kStageBytes + kA0, wave, kt0 + 1, kend);
  lb.template issue<1, false>(rb, smem + kStageBytes + kB1, wave, kt0 + 1, kend);

  auto barrier = [] {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  auto wait_loads = [] { asm volatile("s_waitcnt vmcnt(10)" ::: "memory"); };
  auto wait_reads = [] { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); };

  bf16x8_t af[4][2], bfr[2][2][2];   // bfr[t & 1] holds B0 of tile t, the other set B1 and then B0 of tile t+1
  wait_loads();
  barrier();
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) bfr[0][j][ks] = fb.template get<0>(kB0, j, ks);
  if (wave >= 4) {   // the second group runs one part behind the first, which refills what was read here while the second multiplies
    wait_reads();
    barrier();
  }

  auto compute = [&](f32x4_t (&c)[4][2], const bf16x8_t (&b)[2][2]) {
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) c[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j][ks], af[i][ks], c[i][j], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
  };
  auto tile = [&](auto parity, auto lean, int t) {
    constexpr int S = decltype(parity)::value, O = S ^ 1;
    constexpr bool LEAN = decltype(lean)::value;
    char* own = smem + S * kStageBytes;
    char* other = smem + O * kStageBytes;
    // phase 0
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) af[i][ks] = fa.template get<S>(kA0, i, ks);
    la.template issue<1, LEAN>(ra, other + kA1, wave, t + 1, kend);
    wait_loads();
    barrier();
    compute(acc[0], bfr[S]);
    barrier();
    // phase 1
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) bfr[O][j][ks] = fb.template get<S>(kB1, j, ks);
    lb.template issue<0, LEAN>(rb, own + kB0, wave, t + 2, kend);
    wait_loads();
    barrier();
    compute(acc[1], bfr[O]);
    barrier();
    // phase 2
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) af[i][ks] = fa.template get<S>(kA1, i, ks);
    la.template issue<0, LEAN>(ra, own + kA0, wave, t + 2, kend);
    wait_loads();
    barrier();
    compute(acc[3], bfr[O]);
    barrier();
    // phase 3: its reads are used in the next tile's phase 0, but have to be complete by this phase's end (the place
    // is refilled from the next tile's phase 1 on)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) bfr[O][j][ks] = fb.template get<O>(kB0, j, ks);
    lb.template issue<1, LEAN>(rb, own + kB1, wave, t + 2, kend);
    wait_loads();
    barrier();
    wait_reads();
    compute(acc[2], bfr[S]);
    barrier();
  };
  constexpr std::integral_constant<int, 0> even{};
  constexpr std::integral_constant<int, 1> odd{};
  int t = kt0;
  if (la.plain && lb.plain)
    for (; (t + 4) * BK <= kend; t += 2) {   // every tile requested here (up to t + 3) lies inside K whole
      tile(even, std::true_type{}, t);
      tile(odd, std::true_type{}, t + 1);
    }
  for (; t + 1 < kt1; t += 2) {
    tile(even, std::false_type{}, t);
    tile(odd, std::false_type{}, t + 1);
  }
  if (t < kt1) tile(even, std::false_type{}, t);
  if (wave < 4) barrier();
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the requests past the last k-tile (zeros) have landed
}

// Output forms.
enum { OUT_BF16 = 0, OUT_F32_STORE = 1, OUT_F32_RMW = 2, OUT_F32_RMW_LINES = 3 };
// Gradient accumulators are touched once per launch: non-temporal accesses (.._LINES) where the rows of C start on a line of 128
// bytes.  Elsewhere the two parts of a line belong to different accesses and the second would fetch it again: us for += 7016
// x 9080 x 248 non-temporal 194, plain 151 (8192 x 8200 x 2048 323, 309); 25600 x 12800 x 2048 the other way round, 1296, 1408.
static inline bool whole_lines(size_t ldc) { return ldc * sizeof(float) % 128 == 0; }
constexpr size_t kWideRow = (size_t)1 << 23;   // bytes; rows of C from here on take 64-bit addresses

// GeluRows: z at a lane's places of the output (as gemm_epilogue leaves them with the lanes), zeros past the end.
template <int NS, int RB> struct GeluRows {
  typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
  u32x4_t v[NS][RB];
  template <int BM, int BN>
  __device__ __forceinline__ void load(const bf16_t* z, const int (&row)[NS], const int (&col)[NS], size_t ldc, int M, int N, int m0, int n0) {
    const int lane = threadIdx.x & 63, l15 = lane & 15, q = lane >> 4, c8 = 16 * (q & 1) + 8 * (q >> 1);
    const uint32_t pitch = (uint32_t)ldc * 2, records = (uint32_t)(min(BM, M - m0) - 1) * pitch + (uint32_t)min(BN, N - n0) * 2;
    const auto r = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(z) + (size_t)m0 * ldc + n0, 0, records, 0x00020000);
#pragma unroll
    for (int b = 0; b < NS; ++b)
#pragma unroll
      for (int i = 0; i < RB; ++i)
        v[b][i] = __builtin_amdgcn_raw_buffer_load_b128(r, n0 + col[b] + c8 < N ? (uint32_t)(row[b] + l15 + i * 16) * pitch + (col[b] + c8) * 2 : kOob, 0, 0);
  }
};

// Lane-to-memory mapping: with four consecutive columns per lane a block's store would cover 16 rows x 64 bytes (fp32)
// or 32 bytes (bf16) of each.  bf16: the two column blocks of a 32-column group change lanes (v_permlane16_swap) so
// that a lane ends up with eight consecutive columns (16 bytes).  fp32: lanes of rows 0-7 and 8-15 change halves (a
// rotation by 8 inside 16 lanes) so that an access covers 8 rows x 128 bytes: whole lines, which the read-modify-write
// of the weight gradients needs (25600 x 12800 x 2048: 1431 us with 64-byte segments, 1315 us with whole lines; 1368 us
// with rows staged through LDS).  All accesses to C go through a buffer descriptor that ends behind the tile's last
// row (columns past N: an offset beyond it), so the stage is free of branches.
// row[b], col[b]: first row and column of strip b inside the BM x BN tile.
// What an output stage adds by column: the bias at a lane's columns in front of the exchange below (four of either block of a strip), or
// GeLU's b at its eight columns behind it.  Places past the end repeat the last ones: nothing is stored there.
template <int NS, class EPI> struct ColumnAdd {
  uint2 bias[NS][2];
  uint4 b[NS];
  __device__ __forceinline__ void load(const bf16_t* from, const int (&col)[NS], int N, int n0) {
    const int q = (threadIdx.x & 63) >> 4, c8 = 16 * (q & 1) + 8 * (q >> 1);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      if constexpr (EPI::kKind != EPI_PLAIN) {
        b[s] = *reinterpret_cast<const uint4*>(from + min(n0 + col[s] + c8, N - 8));
      } else {
#pragma unroll
        for (int j = 0; j < 2; ++j) bias[s][j] = make_uint2(0u, 0u);
        if (from) {
#pragma unroll
          for (int j = 0; j < 2; ++j) bias[s][j] = *reinterpret_cast<const uint2*>(from + min(n0 + col[s] + j * 16 + 4 * q, N - 4));
        }
      }
    }
  }
};
// EPI other than plain (OUT_BF16, rows of less than kWideRow): the exchange leaves a lane with eight consecutive columns of a row, what the
// element-wise kernels give a lane; a block of rows of EPI_GELU_GRAD's sums is the RB * 16 rows of a wave.
template <int OUT, int BM, int BN, int NS, int RB, class EPI = Epi<EPI_PLAIN>>
__device__ __forceinline__ void gemm_epilogue(const StripAcc<NS, RB>& acc, const int (&row)[NS], const int (&col)[NS], void* Cv, size_t ldc,
                                              const ColumnAdd<NS, EPI>& add, int M, int N, int m0, int n0, const GeluArgs<bf16_t>& e = {},
                                              const GeluRows<NS, RB>& zr = {}) {
  static_assert(EPI::kKind == EPI_PLAIN || OUT == OUT_BF16, "from the stored product");
  typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
  typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
  constexpr uint32_t esz = OUT == OUT_BF16 ? 2 : 4;
  constexpr bool kRmw = OUT == OUT_F32_RMW || OUT == OUT_F32_RMW_LINES;
  constexpr int kAux = OUT == OUT_F32_RMW_LINES ? 2 : 0;
  const int lane = threadIdx.x & 63, l15 = lane & 15, q = lane >> 4;
  float bv[NS][2][4];
#pragma unroll
  for (int b = 0; b < NS; ++b)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const uint2 w = EPI::kKind == EPI_PLAIN ? add.bias[b][j] : make_uint2(0u, 0u);
      bv[b][j][0] = __uint_as_float(w.x << 16); bv[b][j][1] = __uint_as_float(w.x & 0xffff0000u);
      bv[b][j][2] = __uint_as_float(w.y << 16); bv[b][j][3] = __uint_as_float(w.y & 0xffff0000u);
    }
  if (ldc >= kWideRow / esz) {   // byte offsets inside a tile would not fit 31 bits: plain 64-bit addresses
#pragma unroll
    for (int b = 0; b < NS; ++b)
#pragma unroll
      for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int m = m0 + row[b] + i * 16 + l15, n = n0 + col[b] + j * 16 + 4 * q;
          if (m >= M || n >= N) continue;
          const size_t at = (size_t)m * ldc + n;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float v = acc[b][i][j][r] + bv[b][j][r];
            if (OUT == OUT_BF16) reinterpret_cast<bf16_t*>(Cv)[at + r] = f32_to_bf16(v);
            else if (kRmw) reinterpret_cast<float*>(Cv)[at + r] += v;
            else reinterpret_cast<float*>(Cv)[at + r] = v;
          }
        }
    return;
  }
  char* origin = reinterpret_cast<char*>(Cv) + ((size_t)m0 * ldc + n0) * esz;
  const uint32_t pitch = (uint32_t)ldc * esz, records = (uint32_t)(min(BM, M - m0) - 1) * pitch + (uint32_t)min(BN, N - n0) * esz;
  const auto rc = __builtin_amdgcn_make_buffer_rsrc(origin, 0, records, 0x00020000);
  if (OUT == OUT_BF16) {
    const int c8 = 16 * (q & 1) + 8 * (q >> 1);   // first of this lane's 8 columns after the exchange
    const size_t first = (size_t)m0 * ldc + n0;
    const auto rg = __builtin_amdgcn_make_buffer_rsrc(e.g + first, 0, EPI::kKind == EPI_GELU ? records : 0, 0x00020000);
#pragma unroll
    for (int b = 0; b < NS; ++b) {
      const int c = col[b] + c8;
      const uint32_t off = n0 + c < N ? (uint32_t)(row[b] + l15) * pitch + c * esz : kOob;
      float gb[8], sum[8];
      if (EPI::kKind != EPI_PLAIN) {
        Vec16<bf16_t> w;
        w.raw = add.b[b];
        w.unpack(gb);
#pragma unroll
        for (int j = 0; j < 8; ++j) sum[j] = 0.f;
      }
#pragma unroll
      for (int i = 0; i < RB; ++i) {
        uint32_t p[2][2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const f32x4_t v = acc[b][i][j];
          p[j][0] = pack_bf16x2(v[0] + bv[b][j][0], v[1] + bv[b][j][1]);
          p[j][1] = pack_bf16x2(v[2] + bv[b][j][2], v[3] + bv[b][j][3]);
        }
        const u32x2_t x = __builtin_amdgcn_permlane16_swap(p[0][0], p[1][0], false, false);
        const u32x2_t y = __builtin_amdgcn_permlane16_swap(p[0][1], p[1][1], false, false);
        u32x4_t out = {x[0], y[0], x[1], y[1]};
        if (EPI::kKind != EPI_PLAIN) {
          Vec16<bf16_t> v, z;
          float f[8], zf[8];
          v.raw = __builtin_bit_cast(uint4, out);
          v.unpack(f);
          if (EPI::kKind == EPI_BDA) {
            bool keep[8];
            z.raw = __builtin_bit_cast(uint4, zr.v[b][i]);
            z.unpack(zf);
            keep_flags<8>(e.key, (uint64_t)(m0 + row[b] + i * 16 + l15) * ldc + (uint64_t)(n0 + c), e.thr, keep);
#pragma unroll
            for (int j = 0; j < 8; ++j) zf[j] += keep[j] ? (f[j] + gb[j]) * e.scale : 0.f;
            v.pack(zf);
            out = __builtin_bit_cast(u32x4_t, v.raw);
          } else if (EPI::kKind == EPI_GELU) {
#pragma unroll
            for (int j = 0; j < 8; ++j) f[j] = gelu_f<EPI::kMode>(f[j] + gb[j]);
            v.pack(f);
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, v.raw), rg, off + i * 16 * pitch, 0, 0);
          } else {
            z.raw = __builtin_bit_cast(uint4, zr.v[b][i]);
            z.unpack(zf);
            const bool there = m0 + row[b] + i * 16 + l15 < M;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              f[j] *= gelu_grad_f<EPI::kMode>(zf[j] + gb[j]);
              sum[j] += there ? f[j] : 0.f;
            }
            v.pack(f);
            out = __builtin_bit_cast(u32x4_t, v.raw);
          }
        }
        __builtin_amdgcn_raw_buffer_store_b128(out, rc, off + i * 16 * pitch, 0, 0);
      }
      if (EPI::kKind == EPI_GELU_GRAD) {   // the sixteen rows of a block are lanes l15
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          sum[j] += row_rotate<8>(sum[j]);
          sum[j] += row_rotate<4>(sum[j]);
          sum[j] += row_rotate<2>(sum[j]);
          sum[j] += row_rotate<1>(sum[j]);
        }
        if (l15 == 0 && n0 + c < N && m0 + row[b] < M) {
          float* p = e.part + (size_t)((m0 + row[b]) / (RB * 16)) * ldc + n0 + c;
          *reinterpret_cast<float4*>(p) = make_float4(sum[0], sum[1], sum[2], sum[3]);
          *reinterpret_cast<float4*>(p + 4) = make_float4(sum[4], sum[5], sum[6], sum[7]);
        }
      }
    }
  } else {
    const bool low = l15 < 8;
    uint32_t off[NS];   // after the exchange: rows l15 & 7 (+ 8 for the second access), columns 16 * (l15 / 8) + 4 * q of 32
#pragma unroll
    for (int b = 0; b < NS; ++b) {
      const int c = col[b] + (l15 >> 3) * 16 + 4 * q;
      off[b] = n0 + c < N ? (uint32_t)(row[b] + (l15 & 7)) * pitch + c * esz : kOob;
    }
    auto at = [&](int b, int i, int half) { return off[b] + (i * 16 + half * 8) * pitch; };
    // the old values of the next strip are requested before the current one is added: two batches of loads in flight
    u32x4_t old[2][RB * 2];
    auto fetch_old = [&](int b) {
#pragma unroll
      for (int i = 0; i < RB * 2; ++i) old[b & 1][i] = __builtin_amdgcn_raw_buffer_load_b128(rc, at(b, i >> 1, i & 1), 0, kAux);
    };
    if (kRmw) fetch_old(0);
#pragma unroll
    for (int b = 0; b < NS; ++b) {
      if (kRmw && b + 1 < NS) fetch_old(b + 1);
#pragma unroll
      for (int i = 0; i < RB; ++i) {
        f32x4_t v[2];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float x = acc[b][i][0][r] + bv[b][0][r], y = acc[b][i][1][r] + bv[b][1][r];
          const float got = __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, low ? y : x), 0x128, 0xf, 0xf, true));   // row_ror:8
          v[0][r] = low ? x : got;
          v[1][r] = low ? got : y;
        }
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          if (kRmw) v[half] += __builtin_bit_cast(f32x4_t, old[b & 1][i * 2 + half]);
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, v[half]), rc, at(b, i, half), 0, kAux);
        }
      }
    }
  }
}

// One 256 x 256 tile over k-tiles kt0 .. kt1-1, written either in the caller's output form (slab == nullptr) or
// as a dense 256 x 256 fp32 slab.
template <bool TA, bool TB, int OUT>
__device__ __forceinline__ void gemm_tile(const GemmArgs& g, void* Cv, float* slab, int m0, int n0, int kt0, int kt1, char* smem) {
  TileAcc acc;
  zero_acc<4, 4>(acc);
  if (kt1 > kt0) gemm_mainloop<TA, TB>(acc, g, m0, n0, kt0, kt1, smem);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wm = (wave >> 2) * 64, wn = (wave & 3) * 32;
  const int row[4] = {wm, wm, wm + 128, wm + 128}, col[4] = {wn, wn + 128, wn, wn + 128};
  ColumnAdd<4, Epi<EPI_PLAIN>> add;
  add.load(slab ? nullptr : g.bias, col, g.N, n0);
  if (slab) gemm_epilogue<OUT_F32_STORE, kBM, kBN, 4, 4>(acc, row, col, slab, kBN, add, kBM, kBN, 0, 0);
  else gemm_epilogue<OUT, kBM, kBN, 4, 4>(acc, row, col, Cv, g.ldc, add, g.M, g.N, m0, n0);
}

// 256 x 192 tiles (NN and NT), for outputs that give too few 256 x 256 tiles for the compute units.  Eight waves of 2 x 32 rows and 2 x 48
// columns in the 256 x 256 kernel's two groups, with two phases to a k-tile: its four would be of twelve MFMAs each, too few for what a
// part costs beside them.
//   phase:     0                  1
//   reads      A0(t), B1(t)       A1(t), B0(t+1)     (fragments; complete at the end of the memory part)
//   requests   A1(t+1), B0(t+2)   A0(t+2), B1(t+2)   (half-tiles, two loads each)
//   computes   A0 x B0, A0 x B1   A1 x B1, A1 x B0
// What a phase has read may be refilled from the next phase's memory part on; a request has three phases to land, and the wait at the end of
// a memory part leaves the eight loads in flight that are younger than what the next one reads.
template <bool TB>
__device__ __forceinline__ void gemm_mid_mainloop(f32x4_t (&acc)[4][2][3], const GemmArgs& g, int m0, int n0, char* smem) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const bf16_t* a_base = g.A + (size_t)m0 * g.lda;
  const bf16_t* b_base = TB ? g.B + n0 : g.B + (size_t)n0 * g.ldb;
  const size_t a_left = (size_t)(g.a_end - reinterpret_cast<const char*>(a_base));
  const size_t b_left = (size_t)(g.b_end - reinterpret_cast<const char*>(b_base));
  const rsrc_t ra = make_rsrc(a_base, (uint32_t)(a_left < 0x7fffffffu ? a_left : 0x7fffffffu));
  const rsrc_t rb = make_rsrc(b_base, (uint32_t)(b_left < 0x7fffffffu ? b_left : 0x7fffffffu));
  const int nk = (g.K + BK - 1) / BK, kend = g.K;
  HalfLoad<false> la;
  HalfLoad<TB, 96> lb;
  la.init(g.lda, g.M - m0, wave, lane);
  lb.init(g.ldb, g.N - n0, wave, lane);
  FragRead<false, 2> fa;
  FragRead<TB, 3> fb;
  fa.init(smem, (wave >> 1) * 32, lane);
  fb.init(smem, (wave & 1) * 48, lane);
  constexpr int kA0 = 0, kA1 = kHalfBytes, kB0 = 2 * kHalfBytes, kB1 = 3 * kHalfBytes;
  char* odd_stage = smem + kStageBytes;

  // the requests of the phases in front of phase 0 of the first tile, in the loop's order
  lb.template issue<0, false>(rb, smem + kB0, wave, 0, kend);
  la.template issue<0, false>(ra, smem + kA0, wave, 0, kend);
  lb.template issue<1, false>(rb, smem + kB1, wave, 0, kend);
  la.template issue<1, false>(ra, smem + kA1, wave, 0, kend);
  lb.template issue<0, false>(rb, odd_stage + kB0, wave, 1, kend);
  la.template issue<0, false>(ra, odd_stage + kA0, wave, 1, kend);
  lb.template issue<1, false>(rb, odd_stage + kB1, wave, 1, kend);

  auto barrier = [] {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  auto wait_all = [] { asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)" ::: "memory"); };
  bf16x8_t af[2][2], b0[2][3][2], b1[3][2];   // b0[t & 1]: B0 of tile t
  wait_all();
  barrier();
#pragma unroll
  for (int j = 0; j < 3; ++j)
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) b0[0][j][ks] = fb.template get<0>(kB0, j, ks);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // by both groups: phase 0 refills this place
  barrier();
  if (wave >= 4) barrier();   // the second group runs one part behind the first

  auto compute = [&](f32x4_t (&c)[2][3], const bf16x8_t (&b)[3][2]) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) c[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j][ks], af[i][ks], c[i][j], 0, 0, 0);
  };
  auto tile = [&](auto parity, auto lean, int t) {
    constexpr int S = decltype(parity)::value, O = S ^ 1;
    constexpr bool LEAN = decltype(lean)::value;
    char* own = smem + S * kStageBytes;
    char* other = smem + O * kStageBytes;
    // phase 0
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
      for (int i = 0; i < 2; ++i) af[i][ks] = fa.template get<S>(kA0, i, ks);
#pragma unroll
      for (int j = 0; j < 3; ++j) b1[j][ks] = fb.template get<S>(kB1, j, ks);
    }
    la.template issue<1, LEAN>(ra, other + kA1, wave, t + 1, kend);
    lb.template issue<0, LEAN>(rb, own + kB0, wave, t + 2, kend);
    wait_all();
    barrier();
    __builtin_amdgcn_s_setprio(1);
    compute(acc[0], b0[S]);
    compute(acc[1], b1);
    __builtin_amdgcn_s_setprio(0);
    barrier();
    // phase 1
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
      for (int i = 0; i < 2; ++i) af[i][ks] = fa.template get<S>(kA1, i, ks);
#pragma unroll
      for (int j = 0; j < 3; ++j) b0[O][j][ks] = fb.template get<O>(kB0, j, ks);
    }
    la.template issue<0, LEAN>(ra, own + kA0, wave, t + 2, kend);
    lb.template issue<1, LEAN>(rb, own + kB1, wave, t + 2, kend);
    wait_all();
    barrier();
    __builtin_amdgcn_s_setprio(1);
    compute(acc[3], b1);
    compute(acc[2], b0[S]);
    __builtin_amdgcn_s_setprio(0);
    barrier();
  };
  constexpr std::integral_constant<int, 0> even{};
  constexpr std::integral_constant<int, 1> odd{};
  int t = 0;
  if (la.plain && lb.plain)
    for (; (t + 4) * BK <= kend; t += 2) {   // every tile requested here (up to t + 3) lies inside K whole
      tile(even, std::true_type{}, t);
      tile(odd, std::true_type{}, t + 1);
    }
  for (; t + 1 < nk; t += 2) {
    tile(even, std::false_type{}, t);
    tile(odd, std::false_type{}, t + 1);
  }
  if (t < nk) tile(even, std::false_type{}, t);
  if (wave < 4) barrier();
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the requests past the last k-tile (zeros) have landed
}

constexpr int kMidN = 192;
template <bool TB>
__device__ __forceinline__ void gemm_mid_tile(const GemmArgs& g, void* Cv, int m0, int n0, char* smem) {
  f32x4_t acc[4][2][3];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) acc[q][i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  gemm_mid_mainloop<TB>(acc, g, m0, n0, smem);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wm = (wave >> 1) * 32, wn = (wave & 1) * 96;
  StripAcc<6, 2> out;   // strip 3 * ha + p: rows ha * 128 + wm .., columns wn + 32 p ..
  int row[6], col[6];
#pragma unroll
  for (int ha = 0; ha < 2; ++ha)
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      row[3 * ha + p] = ha * 128 + wm;
      col[3 * ha + p] = wn + 32 * p;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) out[3 * ha + p][i][j] = acc[2 * ha + (2 * p + j) / 3][i][(2 * p + j) % 3];
    }
  ColumnAdd<6, Epi<EPI_PLAIN>> add;
  add.load(g.bias, col, g.N, n0);
  gemm_epilogue<OUT_BF16, kBM, kMidN, 6, 2>(out, row, col, Cv, g.ldc, add, g.M, g.N, m0, n0);
}

// One workgroup per output tile ("data-parallel" form); `id` is the workgroup's index inside its problem.
// Workgroups are dealt round-robin to the 8 XCDs, each with its own L2.  Each XCD owns the column
// tiles x, x+8, ... of the first 8 * (tiles_n / 8) and works through them in groups of up to 8 row tiles, so that the
// workgroups resident on one XCD share 8 A panels and 4 B panels through that L2.  The columns left over are
// numbered the same way and each XCD takes an eighth of their tiles: dealt out whole they gave some XCDs up to 7 % more work than
// others (50 column tiles: 7 to two of them, 6 to the rest), with the rest idle at the end.  us: a layer of 25600 over eight
// shards 10690 -> 10390, two of 12288 over eight 5650 -> 5540.
template <bool TA, bool TB, int OUT>
__device__ __forceinline__ void gemm_dp_tile(const GemmArgs& g, void* Cv, int id, char* smem) {
  const int tiles_m = (g.M + kBM - 1) / kBM, tiles_n = (g.N + kBN - 1) / kBN;
  const int xcd = id & 7, nx = tiles_n / 8, own = tiles_m * nx;   // whole column tiles per XCD, their tiles
  int t = id >> 3, cols = nx, first = xcd, step = 8;   // the tile among `cols` column tiles first, first + step, ...
  if (t >= own) {
    cols = tiles_n - 8 * nx;
    first = 8 * nx;
    step = 1;
    const int rest = cols * tiles_m, per_xcd = (rest + 7) / 8;
    t -= own;
    if (t >= per_xcd) return;
    t += xcd * per_xcd;
    if (t >= rest) return;
  }
  const int per_group = 8 * cols;                   // tiles of one full group of 8 row tiles
  const int grp = t / per_group, in_grp = t % per_group;
  const int gm = min(8, tiles_m - grp * 8);         // row tiles in this group
  const int tile_m = grp * 8 + in_grp % gm, tile_n = (in_grp / gm) * step + first;
  gemm_tile<TA, TB, OUT>(g, Cv, nullptr, tile_m * kBM, tile_n * kBN, 0, (g.K + BK - 1) / BK, smem);
}
// tiles of the XCD that has the most
static inline long long busiest_xcd(long long tiles_m, long long tiles_n) { return tiles_m * (tiles_n / 8) + (tiles_n % 8 * tiles_m + 7) / 8; }
// workgroups of one problem (a multiple of 8, so that a second problem starts on XCD 0 again)
static inline int dp_blocks(const GemmArgs& g) {
  return 8 * (int)busiest_xcd((g.M + kBM - 1) / kBM, (g.N + kBN - 1) / kBN);  // 8 XCD queues of equal length; surplus workgroups exit at once
}

template <bool TA, bool TB, int OUT>
__global__ void __launch_bounds__(kGemmThreads)
gemm_bf16_dp_kernel(GemmArgs g, void* Cv) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  gemm_dp_tile<TA, TB, OUT>(g, Cv, blockIdx.x, smem);
}

// ------------------------------------------------------------------------------------------------
// Small tiles (BM x BN of 64 or 128, four waves of BM/2 x BN/2 per group), for outputs that give fewer 256 x 256 tiles
// than the chip has compute units: what counts there is the number of workgroups and the length of the dependent
// chain of k-tiles.  LDS is a ring of S k-tiles of 64 per group; the fragments of the next k-tile are read while the
// current one is multiplied (one read after each MFMA; with all reads first the MFMAs wait for the LDS queue: 15-25 %
// slower), and its place in the ring is refilled at once, so that S - 1 k-tiles are in flight; a k-tile costs one
// counted wait and one barrier.  KG = 2: two groups of waves take alternate k-tiles and their sums meet in LDS, for
// calls with at most one workgroup per CU (half the chain).  Bound by that chain (0.3 us per k-tile of a 64 x 64 tile,
// 0.5 us of a 128 x 128 one: a barrier, the requests' issue, the fragment reads, the MFMAs), not by a rate.  Measured
// against 256 x 256 tiles with a split k range (us): NN 664 x 512 x 2048 39.7 -> 8.9, NN 664 x 1536 x 512 15.4 -> 5.8,
// NN 1024 x 2048 x 1024 22.5 -> 9.2, NN 2048 x 4096 x 1024 24.3 -> 19.3, TN += 512 x 2048 x 664 26.9 -> 7.0.
// Operand layouts as above, with rows of BM (BN) elements for a k-slow operand.
// ------------------------------------------------------------------------------------------------
constexpr int kSmallThreads = 256;

// slot of 16-byte chunk c of k-row k in a k-slow tile of ROWS elements per k-row (256 or 128 bytes): the k-rows one
// transposing read gathers in a cycle land in different bank groups (128-byte rows: k & 1 picks the half by itself)
template <int ROWS> __device__ __forceinline__ int kslow_swizzle(int k) {
  return ROWS == 128 ? (2 * (k & 3)) ^ (8 * ((k >> 3) & 1)) : (2 * ((k >> 1) & 1)) ^ (4 * ((k >> 3) & 1));
}

// a wave's share of a ROWS x 64 operand tile: ROWS / 32 wave-loads of 1 KiB (one or two groups share an M0 value)
template <bool KSLOW, int ROWS> struct SmallLoad {
  static constexpr int L = ROWS / 32;
  uint32_t off[L];
  uint32_t kstep;
  bool plain;
  __device__ __forceinline__ int kpos(int i, int wave, int lane) const {
    if (!KSLOW) {
      const int row = (wave * L + i) * 8 + (lane >> 3);
      return ((lane & 7) ^ ((row >> 1) & 7)) * 8;
    }
    constexpr int per = 512 / ROWS;   // k-rows per wave-load
    return (wave * L + i) * per + lane / (64 / per);
  }
  // row0: first row of the tile in the block that the descriptor starts at
  __device__ __forceinline__ void init(size_t ld, int rows_left, int wave, int lane, int row0 = 0) {
#pragma unroll
    for (int i = 0; i < L; ++i) {
      const int k = kpos(i, wave, lane);
      if (!KSLOW) {
        const int row = row0 + (wave * L + i) * 8 + (lane >> 3);
        off[i] = row < rows_left ? (uint32_t)(((size_t)row * ld + k) * 2) - i * 1024u : kOob;
      } else {
        const int chunk = (lane & (ROWS / 8 - 1)) ^ kslow_swizzle<ROWS>(k);
        off[i] = row0 + chunk * 8 < rows_left ? (uint32_t)(((size_t)k * ld + row0 + chunk * 8) * 2) - i * 1024u : kOob;
      }
    }
    kstep = KSLOW ? (uint32_t)(BK * ld * 2) : (uint32_t)(BK * 2);
    plain = ld >= 128;
  }
  // LEAN: the caller knows that the k-tile lies inside K whole and that plain is set
  template <bool LEAN = false> __device__ __forceinline__ void issue(rsrc_t r, char* tile, int wave, int lane, int kt, int kend) const {
    char* dst = tile + wave * L * 1024;
    if (LEAN || (plain && (kt + 1) * BK <= kend)) {
      if constexpr (L == 4) load_lds_16x4(r, dst, off[0], off[1], off[2], off[3], (uint32_t)kt * kstep);
      else load_lds_16x2(r, dst, off[0], off[1], (uint32_t)kt * kstep);
    } else {
#pragma unroll
      for (int i = 0; i < L; ++i) {
        const bool ok = off[i] != kOob && kt * BK + kpos(i, wave, lane) < kend;
        load_lds_16(r, dst + i * 1024, ok ? off[i] + i * 1024u + (uint32_t)kt * kstep : kOob);
      }
    }
  }
};

template <bool KSLOW, int ROWS> struct SmallRead {
  static constexpr int NB = ROWS / 32;   // blocks of 16 rows per wave
  uint32_t base[KSLOW ? NB : 2];
  __device__ __forceinline__ void init(const char* smem, int w0, int lane) {
    const int r = lane & 15, G = lane >> 4;
    if (!KSLOW) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) base[ks] = lds_offset(smem) + (w0 + r) * 128 + (((ks * 4 + G) ^ (r >> 1)) * 16);
    } else {
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const int n0 = w0 + i * 16 + 4 * (r & 3), k = 8 * G + (r >> 2);
        base[i] = lds_offset(smem) + k * (ROWS * 2) + (((n0 >> 3) ^ kslow_swizzle<ROWS>(k)) * 16) + (n0 & 7) * 2;
      }
    }
  }
  // to another stage; opaque, so that what follows stays in the reads' offset fields
  __device__ __forceinline__ void move(int bytes) {
#pragma unroll
    for (int i = 0; i < (KSLOW ? NB : 2); ++i) {
      base[i] += bytes;
      asm("" : "+v"(base[i]));
    }
  }
  __device__ __forceinline__ bf16x8_t get(uint32_t at, int i, int ks) const {
    if (!KSLOW) {
      return *PTDP_LDS(const bf16x8_t, base[ks] + at + i * 2048);
    } else {
      const uint32_t p = base[i] + at + ks * (32 * ROWS * 2);
      const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(PTDP_LDS(s16x4_t, p));
      const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(PTDP_LDS(s16x4_t, p + 4 * ROWS * 2));
      const s16x8_t v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      return __builtin_bit_cast(bf16x8_t, v);
    }
  }
};

template <int BM, int BN, int S, int KG> struct SmallGeom {
  static constexpr int kA = BM * BK * 2, kStage = (BM + BN) * BK * 2, kRing = S * kStage, kSmem = KG * kRing;
  static constexpr int kThreads = KG * kSmallThreads;
};

template <bool TA, bool TB, int OUT, int BM, int BN, int S, int KG, class EPI>
__device__ __forceinline__ void gemm_small_tile(const GemmArgs& g, void* Cv, int m0, int n0, char* smem, const GeluArgs<bf16_t>& e) {
  typedef SmallGeom<BM, BN, S, KG> G;
  constexpr int NS = BN / 64, RB = BM / 32, kLoads = (BM + BN) / 32;   // strips, row blocks; loads per wave and k-tile
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) & 3;
  const int kg = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);   // group of waves: takes k-tiles kg, kg + KG, ...
  const int wm = (wave >> 1) * (BM / 2), wn = (wave & 1) * (BN / 2);
  char* ring = smem + kg * G::kRing;
  const bf16_t* a_base = TA ? g.A + m0 : g.A + (size_t)m0 * g.lda;
  const bf16_t* b_base = TB ? g.B + n0 : g.B + (size_t)n0 * g.ldb;
  const size_t a_left = (size_t)(g.a_end - reinterpret_cast<const char*>(a_base));
  const size_t b_left = (size_t)(g.b_end - reinterpret_cast<const char*>(b_base));
  const rsrc_t ra = make_rsrc(a_base, (uint32_t)(a_left < 0x7fffffffu ? a_left : 0x7fffffffu));
  const rsrc_t rb = make_rsrc(b_base, (uint32_t)(b_left < 0x7fffffffu ? b_left : 0x7fffffffu));
  const int nk = ((g.K + BK - 1) / BK + KG - 1) / KG;   // steps: k-tile step * KG + kg
  SmallLoad<TA, BM> la;
  SmallLoad<TB, BN> lb;
  la.init(g.lda, g.M - m0, wave, lane);
  lb.init(g.ldb, g.N - n0, wave, lane);
  SmallRead<TA, BM> fa;
  SmallRead<TB, BN> fb;
  fa.init(ring, wm, lane);
  fb.init(ring + G::kA, wn, lane);
  auto request = [&](int stage, int kt) {   // k-tiles past the end come back as zeros: the waits count every request
    la.issue(ra, ring + stage * G::kStage, wave, lane, kt * KG + kg, g.K);
    lb.issue(rb, ring + stage * G::kStage + G::kA, wave, lane, kt * KG + kg, g.K);
  };
  int row[NS], col[NS];
#pragma unroll
  for (int b = 0; b < NS; ++b) {
    row[b] = wm;
    col[b] = wn + b * 32;
  }
  // what the output stage reads is requested ahead of everything else and waited for at the end: there it would be one more trip to memory
  // (bias, GeLU's b: layers of 200 to 2000 tokens 0.2 to 0.9 % faster)
  ColumnAdd<NS, EPI> add;
  GeluRows<NS, RB> z;
  constexpr bool kReadsZ = EPI::kKind == EPI_GELU_GRAD || EPI::kKind == EPI_BDA;
  constexpr bool kAddAhead = OUT == OUT_BF16 && (!kReadsZ || NS == 1);   // (128 x 128 tiles with z: registers would spill; += : a bias is rare)
  auto load_add = [&] { add.load(EPI::kKind == EPI_PLAIN ? g.bias : e.b, col, g.N, n0); };
  if (kAddAhead) load_add();
  if (kReadsZ && kg == 0) z.template load<BM, BN>(e.z, row, col, g.ldc, g.M, g.N, m0, n0);
#pragma unroll
  for (int i = 0; i < S; ++i) request(i, i);
  StripAcc<NS, RB> acc;
  zero_acc<NS, RB>(acc);
  bf16x8_t af[2][2][RB], bfr[2][2][2 * NS];   // [k-tile parity][ks][block]
  auto read = [&](int par, uint32_t at) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
      for (int i = 0; i < RB; ++i) af[par][ks][i] = fa.get(at, i, ks);
#pragma unroll
      for (int j = 0; j < 2 * NS; ++j) bfr[par][ks][j] = fb.get(at, j, ks);
    }
  };
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "n"((S - 1) * kLoads) : "memory");
  read(0, 0);
  int stage = 0;
  auto step = [&](auto parity, int t) {
    constexpr int P = decltype(parity)::value;
    // k-tile t is in every wave's registers and t + 1 has landed: read t + 1, refill t's stage, multiply t
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"((S - 2) * kLoads) : "memory");
    const int next = stage + 1 == S ? 0 : stage + 1;
    char* own = ring + stage * G::kStage;
    const uint32_t at = next * G::kStage;
    stage = next;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      if (ks == 0) la.issue(ra, own, wave, lane, (t + S) * KG + kg, g.K);
      else lb.issue(rb, own + G::kA, wave, lane, (t + S) * KG + kg, g.K);
#pragma unroll
      for (int i = 0; i < RB; ++i) af[P ^ 1][ks][i] = fa.get(at, i, ks);
#pragma unroll
      for (int j = 0; j < 2 * NS; ++j) bfr[P ^ 1][ks][j] = fb.get(at, j, ks);
#pragma unroll
      for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int j = 0; j < 2 * NS; ++j)
          acc[j >> 1][i][j & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[P][ks][j], af[P][ks][i], acc[j >> 1][i][j & 1], 0, 0, 0);
      constexpr int kMfma = RB * 2 * NS, kReads = (TA ? 2 : 1) * RB + (TB ? 2 : 1) * 2 * NS, kPer = (kReads + kMfma - 1) / kMfma;
#pragma unroll
      for (int q = 0; q < kMfma; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);      // MFMA
        __builtin_amdgcn_sched_group_barrier(0x100, kPer, 0);   // LDS reads
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  constexpr std::integral_constant<int, 0> even{};
  constexpr std::integral_constant<int, 1> odd{};
  int t = 0;
  for (; t + 1 < nk; t += 2) {
    step(even, t);
    step(odd, t + 1);
  }
  if (t < nk) step(even, t);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the requests past the last k-tile (zeros) have landed
  if constexpr (KG == 2) {   // the second group's sums join the first's through LDS: register r of lane l of wave w at sum[w][r][l]
    static_assert(G::kSmem >= 4 * NS * RB * 8 * 64 * 4, "the partial sums fit in the operand ring");
    f32x4_t* sum = reinterpret_cast<f32x4_t*>(smem) + wave * (NS * RB * 2 * 64) + lane;
    __syncthreads();   // every wave is done with the operands
    if (kg == 1) {
#pragma unroll
      for (int b = 0; b < NS; ++b)
#pragma unroll
        for (int i = 0; i < RB * 2; ++i) sum[(b * RB * 2 + i) * 64] = acc[b][i >> 1][i & 1];
    }
    __syncthreads();
    if (kg == 1) return;
#pragma unroll
    for (int b = 0; b < NS; ++b)
#pragma unroll
      for (int i = 0; i < RB * 2; ++i) acc[b][i >> 1][i & 1] += sum[(b * RB * 2 + i) * 64];
  }
  if (!kAddAhead) load_add();
  gemm_epilogue<OUT, BM, BN, NS, RB, EPI>(acc, row, col, Cv, g.ldc, add, g.M, g.N, m0, n0, e, z);
}

// ------------------------------------------------------------------------------------------------
// 256 x 128 tiles (NN and NT), for outputs that give about one or two of them per compute unit and too few of 256 x 256.
// Two groups of four waves take alternate k-tiles of 64, 128 x 64 outputs to a wave as in the 256 x 256 kernel (a pair of
// 128 x 128 tiles brings 64 KiB a k-tile from L2 to LDS for the same outputs, this one 48), and their sums meet in LDS
// at the end.  A k-tile is the 256 x 256 kernel's four phases, each a memory part and an
// arithmetic part with a barrier behind it; the second group runs kWideLag parts behind the first, so that on every SIMD
// one wave computes while the other reads and requests.
// Three k-tiles of 48 KiB are in LDS; k-tile t is in stage t % 3 and belongs to group t % 2.  A half-tile's place is
// free once its group has read it, and the group refills it a phase later, with the same half-tile of k-tile t + 3:
//   phase:     0             1             2             3
//   reads      A0(t)         B1(t)         A1(t)         B0(t+2)      (fragments)
//   requests   B0(t+3)       A0(t+3)       B1(t+3)       A1(t+3)      (half-tiles: 2, 4, 2, 4 loads a wave)
//   computes   A0 x B0       A0 x B1       A1 x B1       A1 x B0
// The other group reads it 6 + kWideLag parts after the request (first group; 14 - kWideLag for the second): the last
// memory part in front of that which the requesting wave has is four phases, twelve loads, after the request, so each
// waits for all but its twelve youngest loads.
// Bound by MFMA issue on few compute units (0.53 us per k-tile, operands in the caches), by the clock that power allows and
// the way from L2 to LDS with all of them (0.73, operands from memory 0.80), against 0.83 and 1.0 for two 128 x 128 tiles.
// us, operands from memory, before (128 x 128 tiles; the last split along k) and now: 2048 x 4096 x 4096 NN 69.4 -> 59.0, NT 67.4 -> 58.4;
// 2048 x 3072 x 4096 67.7 -> 57.9; 1008 x 7680 x 5120 78.4 -> 72.8.
// ------------------------------------------------------------------------------------------------
constexpr int kWideM = 256, kWideN = 128, kWideLag = 3;
constexpr int kWideStage = (kWideM + kWideN) * BK * 2, kWideSmem = 3 * kWideStage;
template <bool TB>
__device__ __forceinline__ void gemm_wide_tile(const GemmArgs& g, void* Cv, int m0, int n0, char* smem) {
  const int lane = threadIdx.x & 63, wave8 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wave = wave8 & 3, grp = wave8 >> 2;
  const bf16_t* a_base = g.A + (size_t)m0 * g.lda;
  const bf16_t* b_base = TB ? g.B + n0 : g.B + (size_t)n0 * g.ldb;
  const size_t a_left = (size_t)(g.a_end - reinterpret_cast<const char*>(a_base));
  const size_t b_left = (size_t)(g.b_end - reinterpret_cast<const char*>(b_base));
  const rsrc_t ra = make_rsrc(a_base, (uint32_t)(a_left < 0x7fffffffu ? a_left : 0x7fffffffu));
  const rsrc_t rb = make_rsrc(b_base, (uint32_t)(b_left < 0x7fffffffu ? b_left : 0x7fffffffu));
  const int steps = ((g.K + BK - 1) / BK + 1) / 2;   // group grp takes k-tiles 2 * step + grp; past the end they are zeros

  SmallLoad<false, 128> la[2];
  SmallLoad<TB, 64> lb[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    la[h].init(g.lda, g.M - m0, wave, lane, h * 128);
    lb[h].init(g.ldb, g.N - n0, wave, lane, h * 64);
  }
  SmallRead<false, 128> fa;
  SmallRead<TB, 64> fb;
  fa.init(smem, (wave >> 1) * 64, lane);
  fb.init(smem, (wave & 1) * 32, lane);
  // byte offsets of the half-tiles in a stage: A0, A1 (128 rows), B0, B1 (64)
  constexpr int kA = 128 * BK * 2, kB = 64 * BK * 2, kB0 = 2 * kA;

  auto barrier = [] {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  auto wait_loads = [] { asm volatile("s_waitcnt vmcnt(12)" ::: "memory"); };   // all but the youngest k-tile's
  auto wait_reads = [] { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); };
  auto request = [&](int kt, int stage) {
    char* at = smem + stage * kWideStage;
    lb[0].template issue<false>(rb, at + kB0, wave, lane, kt, g.K);
    la[0].template issue<false>(ra, at, wave, lane, kt, g.K);
    lb[1].template issue<false>(rb, at + kB0 + kB, wave, lane, kt, g.K);
    la[1].template issue<false>(ra, at + kA, wave, lane, kt, g.K);
  };
  StripAcc<4, 4> acc;
  zero_acc<4, 4>(acc);
  bf16x8_t af[4][2], bfr[2][2][2];
  auto read_a = [&](uint32_t at) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) af[i][ks] = fa.get(at, i, ks);
  };
  auto read_b = [&](bf16x8_t (&f)[2][2], uint32_t at) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) f[j][ks] = fb.get(at, j, ks);
  };
  auto compute = [&](f32x4_t (&c)[4][2], const bf16x8_t (&b)[2][2]) {
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) c[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j][ks], af[i][ks], c[i][j], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
  };

  // as if by the k-tiles in front of the first: the group refills what the other one reads next
  if (grp == 1) {
    request(0, 0);
    request(2, 2);
    wait_loads();   // k-tile 0
  } else {
    request(1, 1);
  }
  barrier();
  if (grp == 1) {
#pragma unroll
    for (int i = 0; i < kWideLag; ++i) barrier();
  }
  int stage = grp;   // of the group's current k-tile
  fa.move(stage * kWideStage);
  fb.move(stage * kWideStage);
  read_b(bfr[0], kB0);
  wait_reads();   // by the whole group: phase 0 refills this place
  barrier();
  auto tile = [&](auto parity, auto lean, int kt) {
    constexpr int S = decltype(parity)::value, O = S ^ 1;
    constexpr bool LEAN = decltype(lean)::value;
    char* own = smem + stage * kWideStage;
    const int step = stage == 0 ? 2 * kWideStage : -kWideStage;   // to the stage of the group's next k-tile
    stage = stage == 0 ? 2 : stage - 1;
    // phase 0
    read_a(0);
    lb[0].template issue<LEAN>(rb, own + kB0, wave, lane, kt + 3, g.K);
    wait_loads();
    barrier();
    compute(acc[0], bfr[S]);
    barrier();
    // phase 1
    read_b(bfr[O], kB0 + kB);
    la[0].template issue<LEAN>(ra, own, wave, lane, kt + 3, g.K);
    wait_loads();
    barrier();
    compute(acc[1], bfr[O]);
    barrier();
    // phase 2
    read_a(kA);
    fa.move(step);
    lb[1].template issue<LEAN>(rb, own + kB0 + kB, wave, lane, kt + 3, g.K);
    wait_loads();
    barrier();
    compute(acc[3], bfr[O]);
    barrier();
    // phase 3
    fb.move(step);
    read_b(bfr[O], kB0);
    la[1].template issue<LEAN>(ra, own + kA, wave, lane, kt + 3, g.K);
    wait_loads();
    barrier();
    wait_reads();
    compute(acc[2], bfr[S]);
    barrier();
  };
  constexpr std::integral_constant<int, 0> even{};
  constexpr std::integral_constant<int, 1> odd{};
  // every k-tile requested here (up to 2 i + 6) lies inside K whole
  const int lean = la[0].plain && lb[0].plain ? max(0, min((g.K / BK - 6 + 3) / 4 * 2, steps / 2 * 2)) : 0;
  int i = 0;
  for (; i < lean; i += 2) {
    tile(even, std::true_type{}, 2 * i + grp);
    tile(odd, std::true_type{}, 2 * i + 2 + grp);
  }
  for (; i + 1 < steps; i += 2) {
    tile(even, std::false_type{}, 2 * i + grp);
    tile(odd, std::false_type{}, 2 * i + 2 + grp);
  }
  if (i < steps) tile(even, std::false_type{}, 2 * i + grp);
  if (grp == 0) {
#pragma unroll
    for (int q = 0; q < kWideLag; ++q) barrier();
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the requests past the last k-tile (zeros) have landed
  __syncthreads();
  // the groups' sums meet in LDS: group 0 finishes strips 0 and 1, group 1 strips 2 and 3; register r of lane l of wave w at sum[w][r][l]
  f32x4_t* sum = reinterpret_cast<f32x4_t*>(smem) + lane;
  f32x4_t mine[2][4][2];
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const f32x4_t lo = acc[b][r >> 1][r & 1], hi = acc[2 + b][r >> 1][r & 1];
      sum[(((grp ^ 1) * 4 + wave) * 16 + b * 8 + r) * 64] = grp == 0 ? hi : lo;
      mine[b][r >> 1][r & 1] = grp == 0 ? lo : hi;
    }
  __syncthreads();
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const f32x4_t other = sum[((grp * 4 + wave) * 16 + b * 8 + r) * 64];
      mine[b][r >> 1][r & 1] += other;
    }
  const int rm = grp * 128 + (wave >> 1) * 64, cn = (wave & 1) * 32;
  const int row[2] = {rm, rm}, col[2] = {cn, cn + 64};
  ColumnAdd<2, Epi<EPI_PLAIN>> add;
  add.load(g.bias, col, g.N, n0);
  gemm_epilogue<OUT_BF16, kWideM, kWideN, 2, 4>(mine, row, col, Cv, g.ldc, add, g.M, g.N, m0, n0);
}

template <bool TB>
__global__ void __launch_bounds__(kGemmThreads)
gemm_bf16_wide_kernel(GemmArgs g, void* Cv) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int tiles_m = (g.M + kWideM - 1) / kWideM, tiles_n = (g.N + kWideN - 1) / kWideN, tiles = tiles_m * tiles_n;
  const int id = blockIdx.x, per_xcd = (tiles + 7) / 8, t = (id & 7) * per_xcd + (id >> 3);   // numbered as below
  if ((id >> 3) >= per_xcd || t >= tiles) return;
  const int grp = t / (8 * tiles_n), in_grp = t - grp * 8 * tiles_n, gm = min(8, tiles_m - grp * 8);
  gemm_wide_tile<TB>(g, Cv, (grp * 8 + in_grp % gm) * kWideM, (in_grp / gm) * kWideN, smem);
}

template <bool TB>
__global__ void __launch_bounds__(kGemmThreads)
gemm_bf16_mid_kernel(GemmArgs g, void* Cv) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int tiles_m = (g.M + kBM - 1) / kBM, tiles_n = (g.N + kMidN - 1) / kMidN, tiles = tiles_m * tiles_n;
  const int id = blockIdx.x, per_xcd = (tiles + 7) / 8, t = (id & 7) * per_xcd + (id >> 3);   // numbered as below
  if ((id >> 3) >= per_xcd || t >= tiles) return;
  const int grp = t / (8 * tiles_n), in_grp = t - grp * 8 * tiles_n, gm = min(8, tiles_m - grp * 8);
  gemm_mid_tile<TB>(g, Cv, (grp * 8 + in_grp % gm) * kBM, (in_grp / gm) * kMidN, smem);
}

// Tiles are numbered in groups of 8 row tiles, column by column inside a group; each XCD takes one contiguous run, so
// that its workgroups share operand panels through its L2.
// TN: where these runs begin at whole or half groups, all XCDs would start in the same one or two columns, a power of two of rows apart, and
// C (read and written) would come from few memory channels at a time: each group starts an eighth of the columns further.  us for the backward
// of a layer of 8192 over four shards, 200 tokens: 650 -> 583, of 4096, 200 tokens, 582 -> 564, of 4096 over two shards, 1024 tokens, 622 -> 589;
// where the runs begin at other places it would change nothing or cost 1 % (5120, 200 tokens).
template <int BM, int BN> static inline int small_blocks(int M, int N) { return 8 * ((((M + BM - 1) / BM) * ((N + BN - 1) / BN) + 7) / 8); }
template <bool TA, bool TB, int OUT, int BM, int BN, int S, int KG, class EPI = Epi<EPI_PLAIN>>
__device__ __forceinline__ void gemm_small_id(const GemmArgs& g, void* Cv, int id, char* smem, const GeluArgs<bf16_t>& e = {}) {
  const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN, tiles = tiles_m * tiles_n;
  const int per_xcd = (tiles + 7) / 8, t = (id & 7) * per_xcd + (id >> 3);
  if ((id >> 3) >= per_xcd || t >= tiles) return;
  const int grp = t / (8 * tiles_n), in_grp = t - grp * 8 * tiles_n, gm = min(8, tiles_m - grp * 8);
  int tile_n = in_grp / gm;
  if (TA && per_xcd % (4 * tiles_n) == 0) tile_n = (tile_n + (grp & 7) * ((tiles_n + 7) / 8)) % tiles_n;
  gemm_small_tile<TA, TB, OUT, BM, BN, S, KG, EPI>(g, Cv, (grp * 8 + in_grp % gm) * BM, tile_n * BN, smem, e);
}
template <bool TA, bool TB, int OUT, int BM, int BN, int S, int KG>
__global__ void __launch_bounds__(KG * kSmallThreads, 2)
gemm_bf16_small_kernel(GemmArgs g, void* Cv) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  gemm_small_id<TA, TB, OUT, BM, BN, S, KG>(g, Cv, blockIdx.x, smem);
}
// The first MLP product with the GeLU behind it (NN) and the second one's input gradient with the GeLU's (NT, TB false).
template <bool TB, int MODE, int BM, int BN, int S, int KG>
__global__ void __launch_bounds__(KG * kSmallThreads, 2)
gemm_bf16_small_gelu_kernel(GemmArgs g, void* Cv, GeluArgs<bf16_t> e) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  gemm_small_id<false, TB, OUT_BF16, BM, BN, S, KG, Epi<TB ? EPI_GELU : EPI_GELU_GRAD, MODE>>(g, Cv, blockIdx.x, smem, e);
}

// The second MLP product with the residual sum behind it.
template <int BM, int BN, int S, int KG>
__global__ void __launch_bounds__(KG * kSmallThreads, 2)
gemm_bf16_small_bda_kernel(GemmArgs g, void* Cv, GeluArgs<bf16_t> e) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  gemm_small_id<false, true, OUT_BF16, BM, BN, S, KG, Epi<EPI_BDA>>(g, Cv, blockIdx.x, smem, e);
}

// Up to four independent problems of the same form in one launch: each later problem's tiles fill the CUs that the
// last, partial round of the ones before it would leave idle.  start[j] = first workgroup index of problem j
// (multiples of 8, so that every problem starts on XCD 0), start[n] = grid size.
constexpr int kMaxMulti = 4;
struct MultiArgs {
  GemmArgs g[kMaxMulti];
  void* C[kMaxMulti];
  int start[kMaxMulti + 1];
  int n;
};
template <bool TA, bool TB, int OUT>
__global__ void __launch_bounds__(kGemmThreads)
gemm_bf16_dp_multi_kernel(MultiArgs a) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int id = (int)blockIdx.x;
  // constant indices only: the arguments stay in scalar registers
  GemmArgs g = a.g[0];
  void* C = a.C[0];
  int first = a.start[0];
#pragma unroll
  for (int q = 1; q < kMaxMulti; ++q)
    if (q < a.n && id >= a.start[q]) {
      g = a.g[q];
      C = a.C[q];
      first = a.start[q];
    }
  g.bias = nullptr;   // (known here: no sums with it in the output stage)
  gemm_dp_tile<TA, TB, OUT>(g, C, id - first, smem);
}

// The small tiles' form of it.  Its first n_sums workgroups (a multiple of 8) finish the column sums of the layer's backward: as a launch
// of its own that is 5 us of a few dependent loads, here it runs beside the tiles (us per pass, same bits: one fp32 layer of 256 x 256 102.1
// -> 97.5, two of 666 x 512 258.8 -> 250.6, eight of 1024 x 2048 over two shards 2858 -> 2826; of one backward, 2048 tokens of 1024 196.5 ->
// 190.7, 512 of 4096 727 -> 722, 582 of 11520 over eight shards 865 -> 867).  With 256 x 256 tiles the sums are many and the launch long: they stay a launch of their own.
template <bool TA, bool TB, int OUT, int BM, int BN, int S, int KG>
__global__ void __launch_bounds__(KG * kSmallThreads, 2)
gemm_bf16_small_multi_kernel(MultiArgs a, ColsumBatchArgs sums, int n_sums) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int id = (int)blockIdx.x - n_sums;
  if (id < 0) {
    if ((int)blockIdx.x < sums.first[kMaxColsumJobs]) colsum_finish_id(sums, blockIdx.x, KG * kSmallThreads / 64, reinterpret_cast<float*>(smem));
    return;
  }
  GemmArgs g = a.g[0];
  void* C = a.C[0];
  int first = a.start[0];
#pragma unroll
  for (int q = 1; q < kMaxMulti; ++q)
    if (q < a.n && id >= a.start[q]) {
      g = a.g[q];
      C = a.C[q];
      first = a.start[q];
    }
  g.bias = nullptr;
  gemm_small_id<TA, TB, OUT, BM, BN, S, KG>(g, C, id - first, smem);
}

// Remainder form, for the tiles that do not fill a whole round of the machine.  The remaining tiles are cut into
// at most two groups; a group of s tiles gives each tile to g = floor(CUs / s) workgroups, workgroup (tile, part)
// taking k-steps [nk*part/g, nk*(part+1)/g) of its tile.  All workgroups of one part index walk the same k-range
// at the same time, so neighbouring tiles share their operand panels through an XCD's L2 exactly as whole rounds
// do (ranges that start at unrelated k, one per workgroup, share nothing: every panel then streams from memory
// and the kernel runs at the memory system's rate instead of L2's).  With g = 1 a workgroup writes its tile
// in the caller's output form; with g > 1 it stores a dense 256 x 256 fp32 slab (index part*s + tile inside the
// group) and gemm_split_reduce_kernel sums a tile's g slabs in part order: no atomics, no waits between
// workgroups, bit-reproducible.
constexpr size_t kSlabFloats = (size_t)kBM * kBN;
constexpr int kMaxSplitGroups = 2;

struct SplitPlan {
  int dp_cols;                      // column tiles computed in whole rounds, one workgroup per tile
  int n_groups;                     // groups of remainder tiles (0 .. kMaxSplitGroups)
  int tiles[kMaxSplitGroups];       // tiles of each group (remainder tiles are numbered row tile fastest)
  int parts[kMaxSplitGroups];       // workgroups per tile
};
// device view of the groups: first workgroup, first tile and first slab of each
struct SplitGroups {
  int n;
  int tiles[kMaxSplitGroups], parts[kMaxSplitGroups], block0[kMaxSplitGroups], tile0[kMaxSplitGroups], slab0[kMaxSplitGroups];
};
static inline int split_blocks(int tiles, int parts) { return 8 * ((tiles * parts + 7) / 8); }   // 8 XCD queues of equal length

template <bool TA, bool TB, int OUT>
__global__ void __launch_bounds__(kGemmThreads)
gemm_bf16_split_kernel(GemmArgs g, void* Cv, float* slabs, SplitGroups sg) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  int j = 0;
  if (sg.n > 1 && (int)blockIdx.x >= sg.block0[1]) j = 1;
  const int id = (int)blockIdx.x - sg.block0[j];
  const int s = sg.tiles[j], parts = sg.parts[j], units = s * parts;
  // each XCD takes a contiguous run of units in part-major order: one part index (or two), neighbouring tiles
  const int per_xcd = (units + 7) / 8;
  const int unit = (id & 7) * per_xcd + (id >> 3);
  if ((id >> 3) >= per_xcd || unit >= units) return;
  const int part = unit / s, t = unit % s;
  const int tiles_m = (g.M + kBM - 1) / kBM;
  const int tile = sg.tile0[j] + t;
  const int m0 = (tile % tiles_m) * kBM, n0 = (tile / tiles_m) * kBN;
  const int nk = (g.K + BK - 1) / BK;
  const int kt0 = (int)((long long)nk * part / parts), kt1 = (int)((long long)nk * (part + 1) / parts);
  gemm_tile<TA, TB, OUT>(g, Cv, parts == 1 ? nullptr : slabs + (size_t)(sg.slab0[j] + unit) * kSlabFloats, m0, n0, kt0, kt1, smem);
}

// One workgroup per (tile of a split group, 16-row band): sums the tile's slabs in part order and writes
// C = sum (+ bias) as bf16, or C += sum as fp32.  `first` = number of (tile, band) workgroups of group 0.
template <bool OUT_F32>
__global__ void __launch_bounds__(256)
gemm_split_reduce_kernel(const float* __restrict__ slabs, void* Cv, const bf16_t* __restrict__ bias, int M, int N, size_t ldc,
                         SplitGroups sg, int j0, int first) {
  int j = j0, b = (int)blockIdx.x;
  if (b >= first) { j = j0 + 1; b -= first; }
  const int t = b >> 4, band = b & 15;
  const int s = sg.tiles[j], parts = sg.parts[j];
  const int tiles_m = (M + kBM - 1) / kBM;
  const int tile = sg.tile0[j] + t;
  const int row = band * 16 + (threadIdx.x >> 4), c4 = (threadIdx.x & 15) * 4;   // 16 rows x 64 float4 per pass
  float4 sum[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) sum[q] = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int part = 0; part < parts; ++part) {
    const float* slab = slabs + (size_t)(sg.slab0[j] + part * s + t) * kSlabFloats + (size_t)row * kBN + c4;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 v = *reinterpret_cast<const float4*>(slab + q * 64);
      sum[q].x += v.x; sum[q].y += v.y; sum[q].z += v.z; sum[q].w += v.w;
    }
  }
  const int m = (tile % tiles_m) * kBM + row;
  if (m >= M) return;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int n = (tile / tiles_m) * kBN + q * 64 + c4;
    if (n >= N) continue;
    if (OUT_F32) {
      float4* c = reinterpret_cast<float4*>(reinterpret_cast<float*>(Cv) + (size_t)m * ldc + n);
      const float4 o = *c;
      *c = make_float4(o.x + sum[q].x, o.y + sum[q].y, o.z + sum[q].z, o.w + sum[q].w);
    } else {
      float b4[4] = {0.f, 0.f, 0.f, 0.f};
      if (bias) {
        const uint2 bb = *reinterpret_cast<const uint2*>(bias + n);
        b4[0] = __uint_as_float(bb.x << 16); b4[1] = __uint_as_float(bb.x & 0xffff0000u);
        b4[2] = __uint_as_float(bb.y << 16); b4[3] = __uint_as_float(bb.y & 0xffff0000u);
      }
      uint2 o;
      o.x = pack_bf16x2(sum[q].x + b4[0], sum[q].y + b4[1]);
      o.y = pack_bf16x2(sum[q].z + b4[2], sum[q].w + b4[3]);
      *reinterpret_cast<uint2*>(reinterpret_cast<bf16_t*>(Cv) + (size_t)m * ldc + n) = o;
    }
  }
}

template <bool TA, bool TB, int OUT>
static int launch_dp(const GemmArgs& g, void* C, hipStream_t st) {
  auto kern = gemm_bf16_dp_kernel<TA, TB, OUT>;
  static once_flag_t done[kMaxDevices];
  if (set_dynamic_smem(reinterpret_cast<const void*>(kern), kGemmSmem, done) != PTDP_OK) return PTDP_E_HIP;
  hipLaunchKernelGGL(kern, dim3(dp_blocks(g)), dim3(kGemmThreads), kGemmSmem, st, g, C);
  return PTDP_OK;
}

template <bool TA, bool TB, int OUT>
static int launch_split(const GemmArgs& g, void* C, float* slabs, const SplitGroups& sg, int blocks, hipStream_t st) {
  auto kern = gemm_bf16_split_kernel<TA, TB, OUT>;
  static once_flag_t done[kMaxDevices];
  if (set_dynamic_smem(reinterpret_cast<const void*>(kern), kGemmSmem, done) != PTDP_OK) return PTDP_E_HIP;
  hipLaunchKernelGGL(kern, dim3(blocks), dim3(kGemmThreads), kGemmSmem, st, g, C, slabs, sg);
  return PTDP_OK;
}

template <bool TA, bool TB, int OUT, int BM, int BN, int S, int KG>
static int launch_small(const GemmArgs& g, void* C, hipStream_t st) {
  auto kern = gemm_bf16_small_kernel<TA, TB, OUT, BM, BN, S, KG>;
  static once_flag_t done[kMaxDevices];
  constexpr int smem = SmallGeom<BM, BN, S, KG>::kSmem;
  if (set_dynamic_smem(reinterpret_cast<const void*>(kern), smem, done) != PTDP_OK) return PTDP_E_HIP;
  const int blocks = small_blocks<BM, BN>(g.M, g.N);
  hipLaunchKernelGGL(kern, dim3(blocks), dim3(KG * kSmallThreads), smem, st, g, C);
  return PTDP_OK;
}
template <int BM, int BN, int S, int KG>
static int launch_small_bda(const GemmArgs& g, void* C, const GeluArgs<bf16_t>& e, hipStream_t st) {
  auto kern = gemm_bf16_small_bda_kernel<BM, BN, S, KG>;
  static once_flag_t done[kMaxDevices];
  constexpr int smem = SmallGeom<BM, BN, S, KG>::kSmem;
  if (set_dynamic_smem(reinterpret_cast<const void*>(kern), smem, done) != PTDP_OK) return PTDP_E_HIP;
  hipLaunchKernelGGL(kern, dim3(small_blocks<BM, BN>(g.M, g.N)), dim3(KG * kSmallThreads), smem, st, g, C, e);
  return PTDP_OK;
}
template <bool TB, int MODE, int BM, int BN, int S, int KG>
static int launch_small_gelu(const GemmArgs& g, void* C, const GeluArgs<bf16_t>& e, hipStream_t st) {
  auto kern = gemm_bf16_small_gelu_kernel<TB, MODE, BM, BN, S, KG>;
  static once_flag_t done[kMaxDevices];
  constexpr int smem = SmallGeom<BM, BN, S, KG>::kSmem;
  if (set_dynamic_smem(reinterpret_cast<const void*>(kern), smem, done) != PTDP_OK) return PTDP_E_HIP;
  hipLaunchKernelGGL(kern, dim3(small_blocks<BM, BN>(g.M, g.N)), dim3(KG * kSmallThreads), smem, st, g, C, e);
  return PTDP_OK;
}
template <bool TB, int MODE>
static int launch_small_gelu_form(int form, const GemmArgs& g, void* C, const GeluArgs<bf16_t>& e, hipStream_t st) {
  switch (form) {
    case 0: return launch_small_gelu<TB, MODE, 128, 128, 2, 1>(g, C, e, st);
    case 1: return launch_small_gelu<TB, MODE, 128, 128, 2, 2>(g, C, e, st);
    case 2: return launch_small_gelu<TB, MODE, 128, 64, 3, 2>(g, C, e, st);
    case 3: return launch_small_gelu<TB, MODE, 64, 64, 4, 2>(g, C, e, st);
    case 4: return launch_small_gelu<TB, MODE, 128, 64, 2, 1>(g, C, e, st);
    default: return PTDP_E_STATE;   // gelu_form offers no other
  }
}
template <bool TB>
static int launch_wide(const GemmArgs& g, void* C, hipStream_t st) {
  auto kern = gemm_bf16_wide_kernel<TB>;
  static once_flag_t done[kMaxDevices];
  if (set_dynamic_smem(reinterpret_cast<const void*>(kern), kWideSmem, done) != PTDP_OK) return PTDP_E_HIP;
  hipLaunchKernelGGL(kern, dim3(small_blocks<kWideM, kWideN>(g.M, g.N)), dim3(kGemmThreads), kWideSmem, st, g, C);
  return PTDP_OK;
}
constexpr int kMidForm = 6;   // in the order of launch_small_form
template <bool TB>
static int launch_mid(const GemmArgs& g, void* C, hipStream_t st) {
  auto kern = gemm_bf16_mid_kernel<TB>;
  static once_flag_t done[kMaxDevices];
  if (set_dynamic_smem(reinterpret_cast<const void*>(kern), kGemmSmem, done) != PTDP_OK) return PTDP_E_HIP;
  hipLaunchKernelGGL(kern, dim3(small_blocks<kBM, kMidN>(g.M, g.N)), dim3(kGemmThreads), kGemmSmem, st, g, C);
  return PTDP_OK;
}
template <bool TA, bool TB, int OUT>
static int launch_small_form(int form, const GemmArgs& g, void* C, hipStream_t st) {
  switch (form) {
    case 0: return launch_small<TA, TB, OUT, 128, 128, 2, 1>(g, C, st);
    case 1: return launch_small<TA, TB, OUT, 128, 128, 2, 2>(g, C, st);
    case 2: return launch_small<TA, TB, OUT, 128, 64, 3, 2>(g, C, st);
    case 3: return launch_small<TA, TB, OUT, 64, 64, 4, 2>(g, C, st);
    case 4: return launch_small<TA, TB, OUT, 128, 64, 2, 1>(g, C, st);
    default: break;
  }
  if constexpr (TA) return PTDP_E_STATE;   // the others are offered to NN and NT alone
  else return form == kMidForm ? launch_mid<TB>(g, C, st) : launch_wide<TB>(g, C, st);
}
// several problems, see gemm_bf16_dp_multi_kernel; a.start is filled here
template <int OUT, int BM, int BN, int S, int KG>
static int launch_small_multi(MultiArgs& a, const ColsumBatchArgs& sums, hipStream_t st) {
  auto kern = gemm_bf16_small_multi_kernel<true, true, OUT, BM, BN, S, KG>;
  static once_flag_t done[kMaxDevices];
  constexpr int smem = SmallGeom<BM, BN, S, KG>::kSmem;
  if (set_dynamic_smem(reinterpret_cast<const void*>(kern), smem, done) != PTDP_OK) return PTDP_E_HIP;
  int at = 0;
  for (int j = 0; j < kMaxMulti; ++j) {
    a.start[j] = at;
    if (j < a.n) at += small_blocks<BM, BN>(a.g[j].M, a.g[j].N);
  }
  a.start[kMaxMulti] = at;
  static_assert(kFinishRed * (int)sizeof(float) <= smem, "the column sums' LDS");
  const int n_sums = (sums.first[kMaxColsumJobs] + 7) / 8 * 8;
  hipLaunchKernelGGL(kern, dim3(n_sums + at), dim3(KG * kSmallThreads), smem, st, a, sums, n_sums);
  return PTDP_OK;
}

static int compute_units() {
  static std::atomic<int> n[kMaxDevices];
  const int d = device_slot();
  if (d >= 0 && n[d].load(std::memory_order_relaxed) > 0) return n[d].load(std::memory_order_relaxed);
  hipDeviceProp_t prop;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) return 256;
  const int cu = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;
  if (d >= 0) n[d].store(cu, std::memory_order_relaxed);
  return cu;
}

// every split group stores at most one slab per compute unit
size_t gemm_workspace_bytes() { return (size_t)compute_units() * kMaxSplitGroups * kSlabFloats * sizeof(float); }

// Times in microseconds that decide how a call is cut (outputs in bf16, or += into fp32), fitted to measured calls: profiles/gemm_forms.txt has
// most of them with the present kernels, how far each form's model is off there and what picking by these numbers costs.
struct LargeCost {
  double fixed, step, step_alone, round, round_alone;   // 256 x 256 tiles: per k-step and per round (first loads, output), full chip and one tile
  double split_fixed, split_step, split_slab, split_part, split_reduce;   // remainder groups: per k-step, per slab; reduce: per slab of one tile or, if more, of all
  double medium;   // factor for a few rounds of kMediumSteps[0] to [1] k-tiles
};
static const LargeCost kLargeCost[2] = {{3.9, 1.28, 0.78, 8.4, 2.8, 11.5, 1.28, 0.050, 0.26, 0.020, 1.0},
                                        {5.7, 1.33, 1.12, 24.4, 8.7, 3.3, 1.56, 0.023, 0.50, 0.069, 1.05}};
// With += the sums above are 2 % low there and those of 128 x 128 tiles 4 to 8 % high.  Of the TN calls of profiles/gemm_forms.txt that take another form
// since column tiles are dealt evenly 8 of 35 were slower by more than 2 % without the factor, 2 of 31 with it; all together 1.03 and 1.06 times
// as fast (us with 128 x 128 and with 256 x 256 tiles: 19200 x 4800 x 712 220, 241; 11008 x 2752 x 528 73, 80).
constexpr int kMediumSteps[2] = {5, 16};

// Whole tiles: full rounds, then one that fills part of the chip.  The XCD with the most tiles (`busiest`, see gemm_dp_tile) sets the
// number of rounds.  whole: the share of the tiles' outputs that exist.
constexpr int kMixedRounds = 12;   // rounds from which the compute units no longer run in step and one's output overlaps another's products
// and k-tiles, fewer where there are many rounds: shorter ones leave few products to overlap.  us of a layer's backward with 128 x 128 and with 256 x
// 256 tiles for its weight gradients: 4096, 512 tokens (12 rounds of 8 k-tiles) 722, 770; 11520 over eight shards, 582 tokens (13 of 10) 866, 892;
// 8320 over four, 804 tokens (13 of 13) 1053, 1021; 5440, 142 tokens (23 of 3) 963, 917; 7680, 435 tokens (43 of 7) 2089, 1988.
constexpr int kMixedSteps = 12, kManyMixedRounds = 20;
static double large_time(const LargeCost& c, long long tiles, long long busiest, double whole, int nk) {
  const int ncu = compute_units(), per_xcd = ncu >= 8 ? ncu / 8 : 1;
  const long long rounds = (busiest + per_xcd - 1) / per_xcd, left = tiles - (rounds - 1) * ncu;
  const double fill = left >= ncu ? 1.0 : (left > 1 ? (double)left : 1.0) / ncu;
  const double t = c.fixed + (double)(rounds - 1) * (c.step * nk + c.round * whole) + (c.step_alone + (c.step - c.step_alone) * fill) * nk +
                   (c.round_alone + (c.round - c.round_alone) * fill) * whole;
  const bool medium = nk >= kMediumSteps[0] && nk <= kMediumSteps[1] && rounds > 1 && rounds < kManyMixedRounds;
  return (rounds >= (nk >= kMixedSteps ? kMixedRounds : kManyMixedRounds) ? 0.95 * t : t) * (medium ? c.medium : 1.0);
}
// A call that is all remainder is split where that promises to be so much faster: the fit is too low for remainders of half a
// round and more (2048 x 6144 x 12288 whole 241 us, split 256; 2048 x 6400 x 25600 497, 508).  Of the factors 1 to 1.15 the one that
// loses least over the measured calls (1962 us in 1293, 2008 without).  Behind whole rounds the split pays as
// computed (2048 x 12288 x 4608, 384 tiles: 191 us whole, 186 split; 2048 x 25600 x 3200 284, 271).
constexpr double kSplitMargin = 1.06;

// How a call is cut: whole rounds of tiles (whole columns of tiles, so that the remainder is fewer tiles than
// compute units), then the remainder in at most two groups (see gemm_bf16_split_kernel).  A first group of
// 2^a tiles is taken while one group over all remaining tiles would leave more than a tenth of the
// compute units idle; the second group takes what is left.  The split is used when its cost is below that of
// whole tiles (less kSplitMargin).  *time: the plan's cost.
static SplitPlan large_plan(int M, int N, int K, int out_f32, int accumulate, int has_bias, size_t ws_bytes, double* time) {
  const int ncu = compute_units();
  const int tiles_m = (M + kBM - 1) / kBM, tiles_n = (N + kBN - 1) / kBN, nk = (K + BK - 1) / BK;
  const long long tiles = (long long)tiles_m * tiles_n;
  const LargeCost& cost = kLargeCost[out_f32 && accumulate];
  SplitPlan P;
  P.dp_cols = tiles_n;
  P.n_groups = 0;
  for (int j = 0; j < kMaxSplitGroups; ++j) P.tiles[j] = P.parts[j] = 0;
  *time = large_time(cost, tiles, busiest_xcd(tiles_m, tiles_n), (double)M * N / ((double)tiles * kBM * kBN), nk);
  const bool out_ok = (out_f32 && accumulate && !has_bias) || !out_f32;
  if (tiles % ncu == 0 || !out_ok || ws_bytes < gemm_workspace_bytes() || (out_f32 && nk < 64)) return P;
  // whole columns only: the full rounds' tiles, rounded up to a column boundary
  const long long full = (tiles / ncu) * ncu;
  const int dp_cols = (int)((full + tiles_m - 1) / tiles_m);
  int rem = (int)(tiles - (long long)dp_cols * tiles_m);
  if (dp_cols >= tiles_n || rem <= 0 || rem >= ncu) return P;
  int gt[kMaxSplitGroups], gp[kMaxSplitGroups], n = 0;
  while (rem > 0 && n < kMaxSplitGroups) {
    int take = rem;
    if (n + 1 < kMaxSplitGroups && (long long)rem * (ncu / rem) * 10 < (long long)ncu * 9) {
      take = 1;
      while (take * 2 <= rem) take *= 2;
    }
    gt[n] = take;
    gp[n] = ncu / take < nk ? ncu / take : nk;   // never more parts than k-steps
    if (gp[n] < 1) gp[n] = 1;
    rem -= take;
    ++n;
  }
  double t_split = cost.split_fixed;
  int most = 0, slabs = 0;
  for (int j = 0; j < n; ++j) {
    t_split += cost.split_step * ((nk + gp[j] - 1) / gp[j]);
    if (gp[j] <= 1) continue;
    slabs += gt[j] * gp[j];
    if (gp[j] > most) most = gp[j];
  }
  t_split += cost.split_slab * slabs + (cost.split_part * most > cost.split_reduce * slabs ? cost.split_part * most : cost.split_reduce * slabs);
  // (whole columns: the full rounds may come out as one more, partly filled round)
  if (dp_cols > 0) t_split += large_time(cost, (long long)dp_cols * tiles_m, busiest_xcd(tiles_m, dp_cols), 1.0, nk);
  if (most == 0 || t_split * (dp_cols > 0 ? 1.0 : kSplitMargin) >= *time) return P;
  *time = t_split;
  P.dp_cols = dp_cols;
  P.n_groups = n;
  for (int j = 0; j < n; ++j) {
    P.tiles[j] = gt[j];
    P.parts[j] = gp[j];
  }
  return P;
}

// Small tiles: which form (index into the table, the order of launch_small_form), or -1 for the 256 x 256 kernels.  A
// call of n problems with `tiles` workgroups, nk k-tiles and `mb` MB of operands takes about
//   fixed + each * w + steps * (pair * (w / 2) + single * (w % 2)) + per_mb * mb,  w = workgroups per CU, steps = ceil(nk / groups)
// where two workgroups of a form that fits twice on a CU overlap (pair < 2 * single).
struct SmallCost {
  int bm, bn, groups, per_cu;
  double fixed, pair, single, each, per_mb;
};
constexpr int kSmallForms = 6;   // (256 x 192 tiles, kMidForm, have a model of their own: mid_time)  TN has no 256 x 128 tiles: with += they are slower than both neighbours (4096 x 4096 x 2048 90 us, 80 and 81)
static const SmallCost kSmallCost[2][kSmallForms + 1] = {
    {{128, 128, 1, 2, 1.9, 0.741, 0.515, 2.1, 0.135},    // (most calls of 64 to 256 large tiles with short k ranges)
     {128, 128, 2, 1, 0.0, 0.0, 0.992, 3.1, 0.102},      // two wave groups share the k range: long k, at most one workgroup per CU
     {128, 64, 2, 1, 0.0, 0.0, 0.576, 3.9, 0.079},
     {64, 64, 2, 1, 0.7, 0.0, 0.372, 2.7, 0.103},        // the smallest outputs
     {128, 64, 1, 2, 2.4, 0.548, 0.422, 0.9, 0.157},
     {256, 128, 2, 1, 2.3, 0.0, 1.48, 7.2, 0.03},        // 80 to 128 large tiles (about one workgroup per CU), and the like in more rounds
     {256, 192, 1, 1, 0.0, 0.0, 0.0, 0.0, 0.0}},
    {{128, 128, 1, 2, 0.0, 0.742, 0.570, 5.8, 0.163},
     {128, 128, 2, 1, 0.0, 0.0, 0.995, 6.6, 0.127},
     {128, 64, 2, 1, 0.4, 0.0, 0.573, 4.7, 0.072},
     {64, 64, 2, 1, 0.9, 0.0, 0.388, 3.4, 0.087},
     {128, 64, 1, 2, 1.4, 0.510, 0.356, 2.8, 0.159},
     {256, 128, 2, 1, 0.0, 0.0, 0.0, 0.0, 0.0},
     {256, 192, 1, 1, 0.0, 0.0, 0.0, 0.0, 0.0}}};
constexpr int kMinStepsForGroups = 8;   // k-tiles from which two wave groups are considered: below, joining their sums costs what they save
// k-tiles up to which 256 x 128 tiles are considered: longer products are faster on 256 x 256 tiles whose k range is split (us for
// 256 x 128 and split: 2048 x 4096 x 12288 NT 168, 163; x 16384 NN 211, 209, NT 215, 206).  Of the 1293 NN and NT
// calls of profiles/gemm_forms.txt they are picked in 56 and take 0.89 of the best other form's time on average, 1.08 at most.
constexpr int kWideSteps = 120;
// Not considered with that many workgroups per CU over that many k-tiles: the panels no longer stay in the caches and the time is
// up to 1.6 times the above (128 x 64, 16 workgroups, 100 k-tiles).
constexpr int kManyRounds = 16, kManySteps = 32;

// *time: of the best large form, then of the best of all
static int small_form(int rmw, int n, const int* M, const int* N, int K, double* time) {
  const int ncu = compute_units(), nk = (K + BK - 1) / BK;
  int best = -1;
  for (int f = 0; f < (rmw ? kSmallForms - 1 : kSmallForms); ++f) {
    const SmallCost& c = kSmallCost[rmw][f];
    if (c.groups > 1 && nk < kMinStepsForGroups) continue;
    if (c.bm == kWideM && nk > kWideSteps) continue;
    long long tiles = 0;
    double mb = 0.0;
    for (int j = 0; j < n; ++j) {
      tiles += (long long)((M[j] + c.bm - 1) / c.bm) * ((N[j] + c.bn - 1) / c.bn);
      mb += 2e-6 * ((double)M[j] + N[j]) * K;
    }
    if (tiles > (1 << 30)) continue;
    if (tiles > (long long)(kManyRounds - 1) * ncu && nk >= kManySteps) continue;
    const double w = (double)((tiles + ncu - 1) / ncu), steps = (nk + c.groups - 1) / c.groups;
    const double t = c.fixed + c.each * w + c.per_mb * mb + steps * (c.per_cu == 2 ? c.pair * (double)(int)(w / 2) + c.single * (w - 2 * (int)(w / 2)) : c.single * w);
    if (t < *time) {
      *time = t;
      best = f;
    }
  }
  return best;
}

// 256 x 192 tiles, NN (transposing reads of B: twice the read instructions) and NT: a k-tile with all compute units and with few, a call,
// and per round.  Over the calls of profiles/gemm_forms.txt they are off by 13 % (rms).
struct MidCost {
  double step, step_alone, fixed, round, round_full;
};
static const MidCost kMidCost[2] = {{1.19, 0.76, 4.9, 6.0, 3.8}, {1.09, 0.70, 4.6, 6.6, 4.3}};   // [PTDP_GEMM_NN], [PTDP_GEMM_NT]
// Taken where they promise kMidMargin, from two row tiles that are three quarters full (less: a column panel serves so few rows that its way
// from memory counts, 208 x 25600 x 768 NN 22.8 us and 21.8 so, 304 x 20096 x 8944 NT 180 and 199).  us of the best other form and so: NT 2048 x
// 6144 x 12288 240, 209; 2048 x 12288 x 1536 80, 72; 1008 x 10240 x 5120 104, 91; 752 x 25600 x 9216 346, 302; 632 x 14848 x 512 19.0, 17.0; NN
// 2048 x 12288 x 1536 80, 77; 1416 x 6656 x 1280 32.3, 30.8.  Of the 867 calls of profiles/gemm_forms.txt with a longer k than kMidShort they are
// picked in 65, at 1.11 times the speed of the form picked without them on average, 6 of them slower by more than 2 % (2176 x 4224 x 2112
// NN 0.91, 4920 x 2080 x 2080 NN 0.90).  A margin of 1.04 would leave three of those and lose as much elsewhere: calls come out 1.29 % above their
// best form on average, 1.30 now.
constexpr double kMidMargin = 1.02;
// Not for products of up to seven k-tiles, which are mostly their output stages: of 164 such calls that the model would give to them 17 are
// slower by more than 2 %, up to a fifth, and the gain, 1.06 on average, is about 1 us a call.
constexpr int kMidShort = 448;
static double mid_time(int mode, int M, int N, int K) {
  const int ncu = compute_units(), nk = (K + BK - 1) / BK;
  const MidCost& c = kMidCost[mode == PTDP_GEMM_NT];
  const long long tiles = (long long)((M + kBM - 1) / kBM) * ((N + kMidN - 1) / kMidN), rounds = (tiles + ncu - 1) / ncu;
  const double fill = (double)(tiles - (rounds - 1) * ncu) / ncu;
  return c.fixed + (double)(rounds - 1) * (c.step * nk + c.round) + (c.step_alone + (c.step - c.step_alone) * fill) * nk + c.round_full * fill;
}

// The whole decision for one call: a small form, or (-1) the plan of the 256 x 256 kernels.  Small forms exist for bf16
// outputs of NN and NT and for the += of TN: what a layer's calls need.
static int choose_form(int mode, int M, int N, int K, int out_f32, int accumulate, int has_bias, size_t ws_bytes, SplitPlan* P, bool mid = true) {
  double t;
  *P = large_plan(M, N, K, out_f32, accumulate, has_bias, ws_bytes, &t);
  const bool rmw = mode == PTDP_GEMM_TN && out_f32 && accumulate;
  if (!rmw && (mode == PTDP_GEMM_TN || out_f32)) return -1;
  const int form = small_form(rmw, 1, &M, &N, K, &t);
  const int rows = (M + kBM - 1) / kBM * kBM;
  return mid && !rmw && K > kMidShort && rows > kBM && 4 * (long long)M >= 3ll * rows && mid_time(mode, M, N, K) * kMidMargin < t ? kMidForm : form;
}

void gemm_plan_query(int mode, int M, int N, int K, int out_f32, int accumulate, int has_bias, size_t ws_bytes, int* dp_cols,
                     int* n_groups, int* tiles, int* parts) {
  SplitPlan P;
  if (choose_form(mode, M, N, K, out_f32, accumulate, has_bias, ws_bytes, &P) >= 0) {
    P.dp_cols = (N + kBN - 1) / kBN;   // other tiles: nothing is split
    P.n_groups = 0;
  }
  *dp_cols = P.dp_cols;
  *n_groups = P.n_groups;
  for (int j = 0; j < kMaxSplitGroups; ++j) {
    tiles[j] = P.tiles[j];
    parts[j] = P.parts[j];
  }
}

void gemm_form_query(int mode, int M, int N, int K, int out_f32, int accumulate, int has_bias, size_t ws_bytes, int* tile_m,
                     int* tile_n, int* groups) {
  SplitPlan P;
  const int f = choose_form(mode, M, N, K, out_f32, accumulate, has_bias, ws_bytes, &P);
  const SmallCost& c = kSmallCost[0][f >= 0 ? f : 0];
  *tile_m = f >= 0 ? c.bm : kBM;
  *tile_n = f >= 0 ? c.bn : kBN;
  *groups = f >= 0 ? c.groups : 1;
}

template <bool TA, bool TB>
static GemmArgs bf16_args(const void* A, const void* B, const void* bias, int M, int N, int K) {
  GemmArgs g;
  g.A = (const bf16_t*)A;
  g.B = (const bf16_t*)B;
  g.bias = (const bf16_t*)bias;
  g.a_end = (const char*)A + (size_t)M * K * 2;
  g.b_end = (const char*)B + (size_t)N * K * 2;
  g.M = M; g.N = N; g.K = K;
  g.lda = TA ? (size_t)M : (size_t)K;
  g.ldb = TB ? (size_t)N : (size_t)K;
  g.ldc = (size_t)N;
  return g;
}

template <bool TA, bool TB>
static int launch_bf16_mode(const void* A, const void* B, void* C, const void* bias, int M, int N, int K, int out_f32,
                            int accumulate, void* ws, size_t ws_bytes, hipStream_t st) {
  // the kernel addresses each operand through a 31-bit byte offset from the block's first row
  if ((size_t)M * K * 2 >= 0x7fffffffull || (size_t)N * K * 2 >= 0x7fffffffull) return PTDP_E_UNSUPPORTED;
  const GemmArgs g = bf16_args<TA, TB>(A, B, bias, M, N, K);
  SplitPlan P;
  const int form = choose_form(TA ? PTDP_GEMM_TN : (TB ? PTDP_GEMM_NN : PTDP_GEMM_NT), M, N, K, out_f32, accumulate, bias != nullptr,
                               ws != nullptr ? ws_bytes : 0, &P);
  if (form >= 0) {
    if constexpr (TA) return whole_lines(g.ldc) ? launch_small_form<TA, TB, OUT_F32_RMW_LINES>(form, g, C, st) : launch_small_form<TA, TB, OUT_F32_RMW>(form, g, C, st);
    else return launch_small_form<TA, TB, OUT_BF16>(form, g, C, st);
  }
  const int ncu = compute_units();
  const int tiles_m = (M + kBM - 1) / kBM, tiles_n = (N + kBN - 1) / kBN;
  const int n_dp = P.dp_cols < tiles_n ? P.dp_cols * kBN : N;
  if (n_dp > 0) {
    GemmArgs d = g;
    d.N = n_dp;
    int rc;
    if (!out_f32) rc = launch_dp<TA, TB, OUT_BF16>(d, C, st);
    else if (accumulate) rc = whole_lines(g.ldc) ? launch_dp<TA, TB, OUT_F32_RMW_LINES>(d, C, st) : launch_dp<TA, TB, OUT_F32_RMW>(d, C, st);
    else rc = launch_dp<TA, TB, OUT_F32_STORE>(d, C, st);
    if (rc != PTDP_OK) return rc;
  }
  if (n_dp < N) {
    // the remainder as a problem of its own: columns n_dp .. N-1
    GemmArgs r = g;
    r.N = N - n_dp;
    r.B = TB ? g.B + n_dp : g.B + (size_t)n_dp * K;
    r.bias = bias ? (const bf16_t*)bias + n_dp : nullptr;
    void* Cr = out_f32 ? (void*)((float*)C + n_dp) : (void*)((bf16_t*)C + n_dp);
    SplitGroups sg;
    sg.n = P.n_groups;
    int blocks = 0, tile0 = 0, slab0 = 0;
    for (int j = 0; j < kMaxSplitGroups; ++j) {
      sg.tiles[j] = j < P.n_groups ? P.tiles[j] : 0;
      sg.parts[j] = j < P.n_groups ? P.parts[j] : 1;
      sg.block0[j] = blocks;
      sg.tile0[j] = tile0;
      sg.slab0[j] = slab0;
      if (j < P.n_groups) {
        if (P.tiles[j] * P.parts[j] > ncu) return PTDP_E_STATE;   // a group never needs more than one slab per compute unit
        blocks += split_blocks(P.tiles[j], P.parts[j]);
        tile0 += P.tiles[j];
        if (P.parts[j] > 1) slab0 += P.tiles[j] * P.parts[j];
      }
    }
    if (tile0 != tiles_m * ((r.N + kBN - 1) / kBN)) return PTDP_E_STATE;   // the groups cover the remainder exactly
    int rc;
    if (!out_f32) rc = launch_split<TA, TB, OUT_BF16>(r, Cr, (float*)ws, sg, blocks, st);
    else if (accumulate) rc = whole_lines(g.ldc) ? launch_split<TA, TB, OUT_F32_RMW_LINES>(r, Cr, (float*)ws, sg, blocks, st)
                                                 : launch_split<TA, TB, OUT_F32_RMW>(r, Cr, (float*)ws, sg, blocks, st);
    else rc = launch_split<TA, TB, OUT_F32_STORE>(r, Cr, (float*)ws, sg, blocks, st);
    if (rc != PTDP_OK) return rc;
    // one reduce launch over the groups that were split (they are adjacent: a group with one part comes last, if at all)
    int j0 = -1, first = 0, total = 0;
    for (int j = 0; j < P.n_groups; ++j) {
      if (P.parts[j] <= 1) continue;
      if (j0 < 0) { j0 = j; first = P.tiles[j] * 16; }
      else if (j != j0 + 1) return PTDP_E_STATE;
      total += P.tiles[j] * 16;
    }
    if (j0 >= 0) {
      if (out_f32)
        hipLaunchKernelGGL(gemm_split_reduce_kernel<true>, dim3(total), dim3(256), 0, st, (const float*)ws, Cr,
                           (const bf16_t*)nullptr, M, r.N, (size_t)N, sg, j0, first);
      else
        hipLaunchKernelGGL(gemm_split_reduce_kernel<false>, dim3(total), dim3(256), 0, st, (const float*)ws, Cr, r.bias, M, r.N,
                           (size_t)N, sg, j0, first);
    }
  }
  return PTDP_OK;
}

// *sums: finished in this launch where the tiles are small, and then empty
template <int OUT> static int launch_tn_multi(int form, MultiArgs& a, ColsumBatch* sums, hipStream_t st) {
  if (form >= 0) {
    double bytes = 0.0;
    const ColsumBatchArgs finish = colsum_batch_args(*sums, &bytes);
    sums->n = 0;
    switch (form) {
      case 0: return launch_small_multi<OUT, 128, 128, 2, 1>(a, finish, st);
      case 1: return launch_small_multi<OUT, 128, 128, 2, 2>(a, finish, st);
      case 2: return launch_small_multi<OUT, 128, 64, 3, 2>(a, finish, st);
      case 3: return launch_small_multi<OUT, 64, 64, 4, 2>(a, finish, st);
      case 4: return launch_small_multi<OUT, 128, 64, 2, 1>(a, finish, st);
      default: return PTDP_E_STATE;   // += has no other small form
    }
  }
  auto kern = gemm_bf16_dp_multi_kernel<true, true, OUT>;
  static once_flag_t done[kMaxDevices];
  if (set_dynamic_smem(reinterpret_cast<const void*>(kern), kGemmSmem, done) != PTDP_OK) return PTDP_E_HIP;
  hipLaunchKernelGGL(kern, dim3(a.start[kMaxMulti]), dim3(kGemmThreads), kGemmSmem, st, a);
  return PTDP_OK;
}

// the form that all of a launch's bf16 weight gradients take, or -1 for 256 x 256 tiles; sums: with column sums to finish
// Those take kSumsLaunch longer behind 256 x 256 tiles, in a launch of their own: 5 us (1024 wide) to 20 (9568 wide).  Over 135 layers of 480 to
// 25600 (48 to 8192 tokens, one to eight shards) the form taken so is 0.2 % slower than the best of 256 x 256, 128 x 128 and 128 x 64 tiles
// on average, 3.7 % at worst; not counted 0.24, without the medium factor of LargeCost 0.3 and 6.7 %, with neither 0.6 and 8.1 %.  us of the backward
// with 256 x 256 and with 128 x 128 tiles: 2048 tokens of 1024 193.0, 190.7; 596 of 2816 465, 447; 1024 of 4096 over two shards 620, 603; and where
// 256 x 256 stay, 1384 of 4864 over two 1008, 1037.
constexpr double kSumsLaunch = 5.0;
static int tn_multi_form(int n, const int* M, const int* N, int K, bool sums) {
  long long tiles = 0, busiest = 0;
  double outputs = 0.0;
  for (int j = 0; j < n; ++j) {
    const long long tm = (M[j] + kBM - 1) / kBM, tn = (N[j] + kBN - 1) / kBN;
    tiles += tm * tn;
    busiest += busiest_xcd(tm, tn);
    outputs += (double)M[j] * N[j];
  }
  double t = large_time(kLargeCost[1], tiles, busiest, outputs / ((double)tiles * kBM * kBN), (K + BK - 1) / BK);
  if (sums) t += kSumsLaunch;
  return small_form(1, n, M, N, K, &t);
}
bool gemm_tn_multi_takes_sums(int dtype, int n, const int* M, const int* N, int K) {
  if (dtype == PTDP_BF16) return tn_multi_form(n, M, N, K, true) >= 0;
  for (int j = 0; j < n; ++j)
    if (f32_form(false, false, M[j], N[j], K).tile != 64) return true;
  return false;
}
static int gemm_tn_multi(int dtype, int n, const void* const* A, const void* const* B, float* const* C, const int* M, const int* N, int K,
                         ColsumBatch* sums, hipStream_t st) {
  if (n <= 0 || n > kMaxMulti) return PTDP_E_INVALID_ARG;
  bool one_by_one = false;
  double flops = 0.0;
  for (int j = 0; j < n; ++j) {
    if (dtype == PTDP_BF16 && (M[j] == 0 || N[j] == 0 || (size_t)M[j] * K * 2 >= 0x7fffffffull || (size_t)N[j] * K * 2 >= 0x7fffffffull)) one_by_one = true;
    flops += 2.0 * K * (double)M[j] * N[j];
  }
  if (one_by_one) {
    for (int j = 0; j < n; ++j) {
      const int rc = launch_gemm(dtype, PTDP_GEMM_TN, A[j], B[j], C[j], nullptr, M[j], N[j], K, 1, 1, nullptr, 0, st);
      if (rc != PTDP_OK) return rc;
    }
    return PTDP_OK;
  }
  Launch L(PTDP_K_GEMM_TN, flops, st);
  if (dtype == PTDP_F32) {
    const int rc = launch_f32_tn_multi(n, A, B, C, M, N, K, sums, st);
    return rc != PTDP_OK ? rc : L.status();
  }
  MultiArgs a;
  a.n = n;
  int at = 0;
  for (int j = 0; j < kMaxMulti; ++j) {
    const int q = j < n ? j : 0;   // unused slots repeat problem 0 (never selected)
    a.g[j] = bf16_args<true, true>(A[q], B[q], nullptr, M[q], N[q], K);
    a.C[j] = C[q];
    a.start[j] = at;
    if (j < n) at += dp_blocks(a.g[j]);
  }
  a.start[kMaxMulti] = at;
  const int form = tn_multi_form(n, M, N, K, sums->n > 0);
  bool lines = true;
  for (int j = 0; j < n; ++j) lines = lines && whole_lines(N[j]);
  const int rc = lines ? launch_tn_multi<OUT_F32_RMW_LINES>(form, a, sums, st) : launch_tn_multi<OUT_F32_RMW>(form, a, sums, st);
  return rc != PTDP_OK ? rc : L.status();
}
// C_j[M_j,N_j] += A_j^T B_j for j < n <= 4 (fp32 C, both operands [K, .]), sharing K: weight gradients whose inputs
// are all at hand.  In bf16 they run as one launch.  sums (nullable): column sums to finish as well, in that launch where that costs
// less than one of their own.
int launch_gemm_tn_multi(int dtype, int n, const void* const* A, const void* const* B, float* const* C, const int* M,
                         const int* N, int K, const ColsumBatch* sums, hipStream_t st) {
  ColsumBatch left;   // what is not finished with the products
  if (sums) left = *sums;
  const int rc = gemm_tn_multi(dtype, n, A, B, C, M, N, K, &left, st);
  return rc != PTDP_OK ? rc : launch_colsum_batch(left, st);
}

int launch_gemm(int dtype, int mode, const void* A, const void* B, void* C, const void* bias, int M, int N, int K,
                int out_f32, int accumulate, void* ws, size_t ws_bytes, hipStream_t st) {
  if (M == 0 || N == 0) return PTDP_OK;
  const int fam = mode == PTDP_GEMM_NN ? PTDP_K_GEMM_NN : (mode == PTDP_GEMM_NT ? PTDP_K_GEMM_NT : PTDP_K_GEMM_TN);
  Launch L(fam, 2.0 * M * N * K, st);
  if (dtype == PTDP_F32) {
    size_t a_rs = K, a_cs = 1, b_rs = N, b_cs = 1;
    if (mode == PTDP_GEMM_NT) { b_rs = 1; b_cs = K; }
    if (mode == PTDP_GEMM_TN) { a_rs = 1; a_cs = M; }
    const float *a = (const float*)A, *b = (const float*)B, *bi = (const float*)bias;
    const bool va = a_cs == 1 && K % 4 == 0 && ((uintptr_t)A & 15) == 0, vb = b_rs == 1 && K % 4 == 0 && ((uintptr_t)B & 15) == 0;
    int rc;
    if (va && vb) rc = launch_gemm_f32<true, true>(a, b, (float*)C, bi, M, N, K, a_rs, a_cs, b_rs, b_cs, accumulate, st);
    else if (va) rc = launch_gemm_f32<true, false>(a, b, (float*)C, bi, M, N, K, a_rs, a_cs, b_rs, b_cs, accumulate, st);
    else rc = launch_gemm_f32<false, false>(a, b, (float*)C, bi, M, N, K, a_rs, a_cs, b_rs, b_cs, accumulate, st);
    return rc != PTDP_OK ? rc : L.status();
  }
  int rc;
  switch (mode) {
    case PTDP_GEMM_NN: rc = launch_bf16_mode<false, true>(A, B, C, bias, M, N, K, out_f32, accumulate, ws, ws_bytes, st); break;
    case PTDP_GEMM_NT: rc = launch_bf16_mode<false, false>(A, B, C, bias, M, N, K, out_f32, accumulate, ws, ws_bytes, st); break;
    default: rc = launch_bf16_mode<true, true>(A, B, C, bias, M, N, K, out_f32, accumulate, ws, ws_bytes, st); break;
  }
  if (rc != PTDP_OK) return rc;
  return L.status();
}

// The two products next to the MLP's GeLU, with it in their output stage where the call takes small tiles (or is fp32): what a kernel of its
// own costs there is a launch and a trip of the product through memory, while a tile's 25 vector instructions per element are spread over
// most of the chip.  With 256 x 256 tiles they would run with nothing beside them, 15 us a tile: see launch_bias_gelu_*.  So they do in fp32
// with 64 x 64 tiles, where a thread also reads z at sixteen places one after the other: us for forward and backward of a layer of 640, 1392
// tokens, 335 and 674 there, 327 and 652 in kernels of their own; of 1024, 2048 tokens, 721 and 1690, 704 and 1640.  Speed of a pass
// against kernels of their own: one fp32 layer of 256 x 256 1.030, two of 666 x 512 1.043, of 2048 x 1024 under a mask 1.016, eight of 1024 x
// 2048 over two shards 1.020; two of 4096 x 256 1.03, of 8192 x 512 1.00.  z requested behind the k loop instead of in front of it: 1.027,
// 1.028, 1.003, 1.004 of the first four.
// The form that such a call takes, or -1 for a kernel of its own.
static int gelu_form(int mode, int M, int N, int K, size_t ws_bytes) {
  if ((size_t)M * K * 2 >= 0x7fffffffull || (size_t)N * K * 2 >= 0x7fffffffull || (size_t)N * 2 >= kWideRow || N % 8 != 0) return -1;
  SplitPlan P;
  const int form = choose_form(mode, M, N, K, 0, 0, 0, ws_bytes, &P, false);   // (what 256 x 192 tiles gain on small ones is less than the kernel)
  return kSmallCost[0][form >= 0 ? form : 0].bm == kWideM ? -1 : form;
}

// z[M,N] = u[M,K] w[K,N], g = GeLU(z + b)
int launch_gemm_gelu(int dtype, int gelu_mode, const void* u, const void* w, const void* b, void* z, void* g, int M, int N, int K, void* ws,
                     size_t ws_bytes, hipStream_t st) {
  if (M == 0 || N == 0) return PTDP_OK;
  const bool tanh = gelu_mode == PTDP_GELU_TANH, vec = K % 4 == 0 && ((uintptr_t)u & 15) == 0;
  const int form = dtype == PTDP_BF16 ? gelu_form(PTDP_GEMM_NN, M, N, K, ws ? ws_bytes : 0) : (vec && f32_form(true, false, M, N, K).tile != 64 ? 0 : -1);
  if (form < 0) {
    const int rc = launch_gemm(dtype, PTDP_GEMM_NN, u, w, z, nullptr, M, N, K, 0, 0, ws, ws_bytes, st);
    return rc != PTDP_OK ? rc : launch_bias_gelu_fwd(dtype, gelu_mode, z, b, g, M, N, st);
  }
  Launch L(PTDP_K_GEMM_NN, 2.0 * M * N * K, st);
  int rc;
  if (dtype == PTDP_BF16) {
    const GeluArgs<bf16_t> e{(const bf16_t*)b, nullptr, (bf16_t*)g, nullptr, 0, 0, 0.f};
    const GemmArgs a = bf16_args<false, true>(u, w, nullptr, M, N, K);
    rc = tanh ? launch_small_gelu_form<true, PTDP_GELU_TANH>(form, a, z, e, st) : launch_small_gelu_form<true, PTDP_GELU_ERF>(form, a, z, e, st);
  } else {
    const GeluArgs<float> e{(const float*)b, nullptr, (float*)g, nullptr, 0, 0, 0.f};
    const float *A = (const float*)u, *B = (const float*)w;
    rc = tanh ? launch_gemm_f32<true, false, Epi<EPI_GELU, PTDP_GELU_TANH>>(A, B, (float*)z, nullptr, M, N, K, K, 1, N, 1, 0, st, e)
              : launch_gemm_f32<true, false, Epi<EPI_GELU, PTDP_GELU_ERF>>(A, B, (float*)z, nullptr, M, N, K, K, 1, N, 1, 0, st, e);
  }
  return rc != PTDP_OK ? rc : L.status();
}

// The form of that product with the residual sum, or -1 for a kernel of its own.  Where another layer follows the product is launch_gemm's, and
// a recomputed layer may be the last of its segment: both must add k in the same order.  Tiles of any size do, as long as the same number
// of wave groups shares the k range.
static int bda_form(int M, int N, int K, size_t ws_bytes) {
  const int form = gelu_form(PTDP_GEMM_NN, M, N, K, ws_bytes);
  if (form < 0) return -1;
  SplitPlan P;
  const int alone = choose_form(PTDP_GEMM_NN, M, N, K, 0, 0, 0, ws_bytes, &P);
  return alone >= 0 && kSmallCost[0][alone].groups == kSmallCost[0][form].groups ? form : -1;
}

// out[M,N] = resid + Drop(g[M,K] w[K,N] + b); o[M,N]: scratch for the product where the sum is a kernel of its own.  Speed of a pass against that
// everywhere: eight layers of 1024 x 2048 over two shards, one at a time, 1.010; two of 2048 x 1024 under a mask 1.012, of 666 x 512 1.005.
int launch_gemm_bda(int dtype, const void* g, const void* w, const void* b, const void* resid, void* o, void* out, float p, uint64_t key, int M, int N,
                    int K, void* ws, size_t ws_bytes, hipStream_t st) {
  if (M == 0 || N == 0) return PTDP_OK;
  const int form = dtype == PTDP_BF16 ? bda_form(M, N, K, ws ? ws_bytes : 0) : -1;
  if (form < 0) {
    const int rc = launch_gemm(dtype, PTDP_GEMM_NN, g, w, o, nullptr, M, N, K, 0, 0, ws, ws_bytes, st);
    return rc != PTDP_OK ? rc : launch_bda_fwd(dtype, o, b, resid, out, M, N, p, key, st);
  }
  Launch L(PTDP_K_GEMM_NN, 2.0 * M * N * K, st);
  const GemmArgs a = bf16_args<false, true>(g, w, nullptr, M, N, K);
  const GeluArgs<bf16_t> e{(const bf16_t*)b, (const bf16_t*)resid, nullptr, nullptr, key, p > 0.f ? dropout_threshold(p) : 0u, 1.0f / (1.0f - p)};
  int rc;
  switch (form) {
    case 0: rc = launch_small_bda<128, 128, 2, 1>(a, out, e, st); break;
    case 1: rc = launch_small_bda<128, 128, 2, 2>(a, out, e, st); break;
    case 2: rc = launch_small_bda<128, 64, 3, 2>(a, out, e, st); break;
    case 3: rc = launch_small_bda<64, 64, 4, 2>(a, out, e, st); break;
    case 4: rc = launch_small_bda<128, 64, 2, 1>(a, out, e, st); break;
    default: rc = PTDP_E_STATE;   // gelu_form offers no other
  }
  return rc != PTDP_OK ? rc : L.status();
}

// dz[M,N] = (dg[M,K] w[N,K]^T) * GeLU'(z + b), dbias += its column sums (scratch: colsum_scratch_bytes)
int launch_gemm_gelu_bwd(int dtype, int gelu_mode, const void* dg, const void* w, const void* z, const void* b, void* dz, float* dbias,
                         void* scratch, int M, int N, int K, void* ws, size_t ws_bytes, hipStream_t st, ColsumBatch* defer) {
  if (M == 0 || N == 0) return PTDP_OK;
  const bool tanh = gelu_mode == PTDP_GELU_TANH, vec = K % 4 == 0 && (((uintptr_t)dg | (uintptr_t)w) & 15) == 0;
  const int form = dtype == PTDP_BF16 ? gelu_form(PTDP_GEMM_NT, M, N, K, ws ? ws_bytes : 0) : (vec && f32_form(true, true, M, N, K).tile == 32 ? 0 : -1);
  if (form < 0) {
    const int rc = launch_gemm(dtype, PTDP_GEMM_NT, dg, w, dz, nullptr, M, N, K, 0, 0, ws, ws_bytes, st);
    return rc != PTDP_OK ? rc : launch_bias_gelu_bwd(dtype, gelu_mode, dz, z, b, dz, dbias, scratch, M, N, st, defer);
  }
  int rows;   // per row of partial sums
  {
    Launch L(PTDP_K_GEMM_NT, 2.0 * M * N * K, st);
    int rc;
    if (dtype == PTDP_BF16) {
      rows = kSmallCost[0][form].bm / 2;
      const GeluArgs<bf16_t> e{(const bf16_t*)b, (const bf16_t*)z, nullptr, (float*)scratch, 0, 0, 0.f};
      const GemmArgs a = bf16_args<false, false>(dg, w, nullptr, M, N, K);
      rc = tanh ? launch_small_gelu_form<false, PTDP_GELU_TANH>(form, a, dz, e, st) : launch_small_gelu_form<false, PTDP_GELU_ERF>(form, a, dz, e, st);
    } else {
      rows = 32;
      const GeluArgs<float> e{(const float*)b, (const float*)z, nullptr, (float*)scratch, 0, 0, 0.f};
      const float *A = (const float*)dg, *B = (const float*)w;
      rc = tanh ? launch_gemm_f32<true, true, Epi<EPI_GELU_GRAD, PTDP_GELU_TANH>>(A, B, (float*)dz, nullptr, M, N, K, K, 1, 1, K, 0, st, e)
                : launch_gemm_f32<true, true, Epi<EPI_GELU_GRAD, PTDP_GELU_ERF>>(A, B, (float*)dz, nullptr, M, N, K, K, 1, 1, K, 0, st, e);
    }
    if (rc != PTDP_OK || (rc = L.status()) != PTDP_OK) return rc;
  }
  return colsum_finish((const float*)scratch, (M + rows - 1) / rows, N, dbias, nullptr, N, st, defer);
}

}  // namespace ptdp
