// First- and last-stage extras of the GPT model: token + position embedding with hidden dropout (and
// its backward), and the loss over the logit layer's output (softmax cross-entropy, forward and
// backward in one pass over the logits).  The paper counts the embedding tables in eq. (2) and the
// logit layer's GEMMs in its appendix; the GEMMs and the final LayerNorm run through the kernels the
// transformer layers use.  All kernels here are HBM-bound.
#include "common.h"

namespace ptdp {

// ------------------------------------------------------------------------------------------------
// x[i, j, :] = Drop(E_word[token[i, j] - v0] (zero row if outside this shard) + E_pos[i])
// ------------------------------------------------------------------------------------------------
template <typename T>
__global__ void embed_fwd_kernel(const int32_t* __restrict__ tokens, const T* __restrict__ e_word,
                                 const T* __restrict__ e_pos, T* __restrict__ x, size_t total_vec, int nvec_row, int b,
                                 int v0, int vrows, uint64_t key, uint32_t thr, float scale) {
  constexpr int N = Vec16<T>::N;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total_vec; i += (size_t)gridDim.x * blockDim.x) {
    const size_t row = i / nvec_row;
    const int c = (int)(i % nvec_row);
    const int local = tokens[row] - v0;
    Vec16<T> w, p;
    float wf[N], pf[N];
    bool keep[N];
    p.load(e_pos + ((size_t)(row / b) * nvec_row + c) * N);
    p.unpack(pf);
    if (local >= 0 && local < vrows) {
      w.load(e_word + ((size_t)local * nvec_row + c) * N);
      w.unpack(wf);
    } else {
#pragma unroll
      for (int j = 0; j < N; ++j) wf[j] = 0.f;
    }
    keep_flags<N>(key, (uint64_t)i * N, thr, keep);
#pragma unroll
    for (int j = 0; j < N; ++j) wf[j] = keep[j] ? (wf[j] + pf[j]) * scale : 0.f;
    w.pack(wf);
    w.store(x + i * N);
  }
}

// Backward: d = Drop'(dx), d_pos[i, :] += sum_j d[i, j, :] (j in order) and d_word[r, :] += sum over the tokens with id
// v0 + r of d[token, :] in token order, in one launch.  The first row_blocks workgroups take kEmbedRows vocabulary rows
// each: they read the token ids once, note in LDS which tokens name which of their rows (one bit per token, 64 ids per
// ballot) and add up the rows that any token names, each wave its own slices of 64 column vectors: no atomics, no two
// waves touch the same element, rows that no token names are left untouched.  The other workgroups walk the positions.
// Dropping out again from dx costs a hash per four elements and saves writing d and reading it back.  Bound by the
// read-modify-write of d_pos.  Before: a launch that wrote d (50 us) and one workgroup per row whose four waves each read
// all ids twice, one load at a time (81 us; 2048 tokens x 12288, 6400 rows); now about 58 us together.
constexpr int kEmbedThreads = 512, kEmbedRows = 8, kEmbedChunks = 128;   // tokens per round: 64 * kEmbedChunks
template <typename T>
__device__ __forceinline__ void embed_drop(const T* __restrict__ dx, size_t v, uint64_t key, uint32_t thr, float scale, float* af) {
  constexpr int N = Vec16<T>::N;
  Vec16<T> a;
  bool keep[N];
  a.load(dx + v * N);
  a.unpack(af);
  keep_flags<N>(key, (uint64_t)v * N, thr, keep);
#pragma unroll
  for (int e = 0; e < N; ++e) af[e] = keep[e] ? af[e] * scale : 0.f;
}
template <typename T>
__global__ void __launch_bounds__(kEmbedThreads)
embed_bwd_kernel(const int32_t* __restrict__ tokens, const T* __restrict__ dx, float* __restrict__ d_word, float* __restrict__ d_pos,
                 int s, int b, int nvec_row, int v0, int vrows, int row_blocks, uint64_t key, uint32_t thr, float scale) {
  constexpr int N = Vec16<T>::N;
  if ((int)blockIdx.x >= row_blocks) {
    const size_t total = (size_t)s * nvec_row, stride = (size_t)((int)gridDim.x - row_blocks) * kEmbedThreads;
    for (size_t i = (size_t)((int)blockIdx.x - row_blocks) * kEmbedThreads + threadIdx.x; i < total; i += stride) {
      const size_t pos = i / nvec_row;
      const int c = (int)(i % nvec_row);
      float acc[N];
#pragma unroll
      for (int e = 0; e < N; ++e) acc[e] = 0.f;
      for (int j = 0; j < b; ++j) {
        float af[N];
        embed_drop<T>(dx, (pos * b + j) * nvec_row + c, key, thr, scale, af);
#pragma unroll
        for (int e = 0; e < N; ++e) acc[e] += af[e];
      }
      float* o = d_pos + i * N;
#pragma unroll
      for (int e = 0; e < N; ++e) o[e] += acc[e];
    }
    return;
  }
  __shared__ unsigned long long named[kEmbedRows][kEmbedChunks];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, row0 = (int)blockIdx.x * kEmbedRows, rows = min(kEmbedRows, vrows - row0);
  const int id0 = v0 + row0, ntok = s * b;
  for (int base = 0; base < ntok; base += 64 * kEmbedChunks) {
    __syncthreads();   // `named` of the previous round no longer read
#pragma unroll 4
    for (int ch = wave; ch < kEmbedChunks; ch += kEmbedThreads / 64) {
      const int t = base + ch * 64 + lane;
      const uint32_t local = t < ntok ? (uint32_t)tokens[t] - (uint32_t)id0 : ~0u;
      unsigned long long mine = 0;
      if (__any(local < (uint32_t)rows)) {
#pragma unroll
        for (int r = 0; r < kEmbedRows; ++r) {
          const unsigned long long m = __ballot(local == (uint32_t)r);
          if (lane == r) mine = m;
        }
      }
      if (lane < kEmbedRows) named[lane][ch] = mine;
    }
    __syncthreads();
    for (int r = 0; r < rows; ++r) {
      static_assert(kEmbedChunks == 128, "two words per lane");
      const unsigned long long full[2] = {__ballot(named[r][lane] != 0), __ballot(named[r][64 + lane] != 0)};
      if ((full[0] | full[1]) == 0) continue;
      for (int c = wave * 64 + lane; c - lane < nvec_row; c += kEmbedThreads) {
        const bool col_ok = c < nvec_row;
        float acc[N];
#pragma unroll
        for (int e = 0; e < N; ++e) acc[e] = 0.f;
#pragma unroll
        for (int w = 0; w < 2; ++w)
          for (unsigned long long f = full[w]; f; f &= f - 1) {
            const int ch = w * 64 + __ffsll((long long)f) - 1;
            for (unsigned long long m = named[r][ch]; m; m &= m - 1) {
              const size_t t = (size_t)base + ch * 64 + __ffsll((long long)m) - 1;
              if (!col_ok) continue;
              float af[N];
              embed_drop<T>(dx, t * nvec_row + c, key, thr, scale, af);
#pragma unroll
              for (int e = 0; e < N; ++e) acc[e] += af[e];
            }
          }
        if (col_ok) {
          float* o = d_word + ((size_t)(row0 + r) * nvec_row + c) * N;
#pragma unroll
          for (int e = 0; e < N; ++e) o[e] += acc[e];
        }
      }
    }
  }
}

// ------------------------------------------------------------------------------------------------
// Loss over one shard's logits [rows, vrows]: per token m = max, z = sum exp(l - m),
// loss = log z + m - l[target] (target outside the shard: no target term), and in place
// l <- (exp(l - m) / z - [v == target]) * grad_scale.  One workgroup per token; the row is read three
// times, the second and third time from cache.
// ------------------------------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(256)
xent_kernel(T* __restrict__ logits, const int32_t* __restrict__ targets, float* __restrict__ token_loss, int vrows, int v0,
            float grad_scale) {
  constexpr int N = Vec16<T>::N;
  __shared__ float red[16];
  T* row = logits + (size_t)blockIdx.x * vrows;
  const int nvec = vrows / N;
  float mx = -INFINITY;
  for (int v = threadIdx.x; v < nvec; v += blockDim.x) {
    Vec16<T> a;
    float af[N];
    a.load(row + (size_t)v * N);
    a.unpack(af);
#pragma unroll
    for (int j = 0; j < N; ++j) mx = fmaxf(mx, af[j]);
  }
  mx = wave_max(mx);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
  __syncthreads();
  mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  float z = 0.f;
  for (int v = threadIdx.x; v < nvec; v += blockDim.x) {
    Vec16<T> a;
    float af[N];
    a.load(row + (size_t)v * N);
    a.unpack(af);
#pragma unroll
    for (int j = 0; j < N; ++j) z += __expf(af[j] - mx);
  }
  z = block_sum(z, red + 4);
  const int local = targets[blockIdx.x] - v0;
  const bool inside = local >= 0 && local < vrows;
  if (threadIdx.x == 0) {
    float picked = 0.f;
    if (inside) {
      if (sizeof(T) == 2) picked = bf16_to_f32(reinterpret_cast<const bf16_t*>(row)[local]);
      else picked = reinterpret_cast<const float*>(row)[local];
    }
    token_loss[blockIdx.x] = __logf(z) + mx - picked;
  }
  __syncthreads();   // the target logit is read before the row is overwritten
  const float rz = grad_scale / z;
  for (int v = threadIdx.x; v < nvec; v += blockDim.x) {
    Vec16<T> a;
    float af[N];
    a.load(row + (size_t)v * N);
    a.unpack(af);
#pragma unroll
    for (int j = 0; j < N; ++j) {
      af[j] = __expf(af[j] - mx) * rz;
      if (inside && v * N + j == local) af[j] -= grad_scale;
    }
    a.pack(af);
    a.store(row + (size_t)v * N);
  }
}

// loss[0] = mean of token_loss[0 .. n), summed in a fixed order by one workgroup
__global__ void __launch_bounds__(256) loss_mean_kernel(const float* __restrict__ token_loss, float* __restrict__ loss, int n) {
  __shared__ float red[16];
  float a = 0.f;
  for (int i = threadIdx.x; i < n; i += 256) a += token_loss[i];
  a = block_sum(a, red);
  if (threadIdx.x == 0) loss[0] = a / (float)n;
}

static inline int grid_for(size_t total) {
  const size_t blocks = (total + 255) / 256, cap = 256 * 16;
  return (int)(blocks < cap ? (blocks ? blocks : 1) : cap);
}

template <typename T>
static int embed_fwd_t(const int32_t* tokens, const void* e_word, const void* e_pos, void* x, int s, int b, int h, int v0,
                       int vrows, float p, uint64_t key, hipStream_t st) {
  constexpr int N = Vec16<T>::N;
  const size_t total = (size_t)s * b * h / N;
  Launch L(PTDP_K_EMBED, (double)s * b * h * sizeof(T) * 2 + (double)s * h * sizeof(T), st);
  hipLaunchKernelGGL((embed_fwd_kernel<T>), dim3(grid_for(total)), dim3(256), 0, st, tokens, (const T*)e_word,
                     (const T*)e_pos, (T*)x, total, h / N, b, v0, vrows, key, p > 0.f ? dropout_threshold(p) : 0u,
                     1.0f / (1.0f - p));
  return L.status();
}

int launch_embed_fwd(int dtype, const int32_t* tokens, const void* e_word, const void* e_pos, void* x, int s, int b, int h,
                     int v0, int vrows, float p, uint64_t key, hipStream_t st) {
  return dtype == PTDP_BF16 ? embed_fwd_t<bf16_t>(tokens, e_word, e_pos, x, s, b, h, v0, vrows, p, key, st)
                            : embed_fwd_t<float>(tokens, e_word, e_pos, x, s, b, h, v0, vrows, p, key, st);
}

template <typename T>
static int embed_bwd_t(const int32_t* tokens, const void* dx, float* d_e_word, float* d_e_pos, int s, int b,
                       int h, int v0, int vrows, float p, uint64_t key, hipStream_t st) {
  constexpr int N = Vec16<T>::N;
  Launch L(PTDP_K_EMBED, (double)s * b * h * sizeof(T) * 3 + (double)s * h * 8, st);
  const int row_blocks = (vrows + kEmbedRows - 1) / kEmbedRows;
  hipLaunchKernelGGL((embed_bwd_kernel<T>), dim3(row_blocks + grid_for((size_t)s * h / N)), dim3(kEmbedThreads), 0, st, tokens,
                     (const T*)dx, d_e_word, d_e_pos, s, b, h / N, v0, vrows, row_blocks, key, p > 0.f ? dropout_threshold(p) : 0u,
                     1.0f / (1.0f - p));
  return L.status();
}

int launch_embed_bwd(int dtype, const int32_t* tokens, const void* dx, float* d_e_word, float* d_e_pos, int s, int b, int h, int v0, int vrows, float p, uint64_t key, hipStream_t st) {
  return dtype == PTDP_BF16 ? embed_bwd_t<bf16_t>(tokens, dx, d_e_word, d_e_pos, s, b, h, v0, vrows, p, key, st)
                            : embed_bwd_t<float>(tokens, dx, d_e_word, d_e_pos, s, b, h, v0, vrows, p, key, st);
}

int launch_xent(int dtype, void* logits, const int32_t* targets, float* token_loss, float* loss, int rows, int vrows,
                int v0, float grad_scale, hipStream_t st) {
  const size_t esz = dtype == PTDP_BF16 ? 2 : 4;
  Launch L(PTDP_K_XENT, (double)rows * vrows * esz * 2, st);
  if (dtype == PTDP_BF16)
    hipLaunchKernelGGL((xent_kernel<bf16_t>), dim3(rows), dim3(256), 0, st, (bf16_t*)logits, targets, token_loss, vrows, v0,
                       grad_scale);
  else
    hipLaunchKernelGGL((xent_kernel<float>), dim3(rows), dim3(256), 0, st, (float*)logits, targets, token_loss, vrows, v0,
                       grad_scale);
  hipLaunchKernelGGL(loss_mean_kernel, dim3(1), dim3(256), 0, st, (const float*)token_loss, loss, rows);
  return L.status();
}

}  // namespace ptdp
