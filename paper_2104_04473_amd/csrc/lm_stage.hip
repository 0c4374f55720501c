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
// each: they read the token ids once, list the tokens that name one of their rows, row by row in token order, in LDS, and
// add them up, each wave its own slices of 64 column vectors: no atomics, no two waves touch the same element, rows that no
// token names are left untouched.  The other workgroups walk the positions.
// Dropping out again from dx costs a hash per four elements and saves writing d and reading it back.
// Bound by the read-modify-write of d_pos where ids are spread evenly, and by the chain of hashes and additions of the most
// frequent row otherwise (0.2 us a token).  us, before (a launch that wrote d and one workgroup per row whose waves read all
// ids twice, one load at a time) and now, bf16, even ids / ids with frequency 1 / rank: 2048 tokens x 12288, 6400 rows
// 116 / 519 -> 45 / 221; 8192 x 1024, 128 rows 52 / 376 -> 17 / 283; 48 x 1024, 50000 rows 14.9 / 14.5 -> 13.8 / 13.4.
// Batches of 8 gain 15 % on frequent ids and lose 5 % on even ones.
constexpr int kEmbedThreads = 512, kEmbedWaves = kEmbedThreads / 64, kEmbedRows = 8;
constexpr int kEmbedChunks = 128;   // tokens per round: 64 * kEmbedChunks
constexpr int kEmbedBatch = 4;      // tokens of a row requested together
static_assert(kEmbedRows == kEmbedWaves && kEmbedChunks == 128, "a wave lists one row, two words per lane");
// acc += Drop'(a); z = key + kGolden * (index of a's first element / 4), as in keep_flags
template <typename T>
__device__ __forceinline__ void embed_add(const Vec16<T>& a, uint64_t z, uint32_t thr, float scale, float (&acc)[Vec16<T>::N]) {
  constexpr int N = Vec16<T>::N;
  float af[N];
  a.unpack(af);
#pragma unroll
  for (int w = 0; w < N / 4; ++w) {
    const uint64_t r = mix64(z + kGolden * w);
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[4 * w + j] = fmaf((uint32_t)((r >> (16 * j)) & 0xffffu) >= thr ? af[4 * w + j] : 0.f, scale, acc[4 * w + j]);
  }
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
        const size_t v = (pos * b + j) * nvec_row + c;
        Vec16<T> a;
        a.load(dx + v * N);
        embed_add<T>(a, key + kGolden * (v * (N / 4)), thr, scale, acc);
      }
      float* o = d_pos + i * N;
#pragma unroll
      for (int e = 0; e < N; ++e) o[e] += acc[e];
    }
    return;
  }
  __shared__ unsigned long long named[kEmbedRows][kEmbedChunks];   // bit t of word ch: token 64 ch + t of the round names the row
  __shared__ uint16_t list[64 * kEmbedChunks];                     // the tokens of row 0, of row 1, ..
  __shared__ int count[kEmbedRows];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  // rows blockIdx.x, blockIdx.x + row_blocks, ..: frequent ids are often neighbours
  const int row0 = (int)blockIdx.x, rows = (vrows - row0 + row_blocks - 1) / row_blocks, ntok = s * b, slices = (nvec_row + 63) / 64;
  for (int base = 0; base < ntok; base += 64 * kEmbedChunks) {
    const int chunks = min(kEmbedChunks, (ntok - base + 63) / 64);
#pragma unroll 4
    for (int ch = wave; ch < chunks; ch += kEmbedWaves) {
      const int t = base + ch * 64 + lane;
      const uint32_t local = t < ntok ? (uint32_t)tokens[t] - (uint32_t)v0 : ~0u;
      unsigned long long mine = 0;
#pragma unroll
      for (int r = 0; r < kEmbedRows; ++r) {   // (rows past the last one: read by nobody)
        const unsigned long long m = __ballot(local == (uint32_t)(row0 + r * row_blocks));
        if (lane == r) mine = m;
      }
      if (lane < kEmbedRows) named[lane][ch] = mine;
    }
    __syncthreads();
    // wave r counts row r: `before` = the row's tokens ahead of this lane's two words
    unsigned long long word[2];
    int mine = 0, before = 0;
    if (wave < rows) {
      // lane l takes words 2 l and 2 l + 1: tokens in order across the lanes
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        word[h] = 2 * lane + h < chunks ? named[wave][2 * lane + h] : 0;
        mine += __popcll(word[h]);
      }
      before = mine;
#pragma unroll
      for (int d = 1; d < 64; d *= 2) {
        const int up = __shfl_up(before, d, 64);
        if (lane >= d) before += up;
      }
      if (lane == 63) count[wave] = before;
      before -= mine;
    } else if (lane == 63) {
      count[wave] = 0;
    }
    __syncthreads();
    int total = 0;
#pragma unroll
    for (int r = 0; r < kEmbedRows; ++r) {
      if (r == wave) before += total;
      total += count[r];
    }
    if (total > 0) {
      if (wave < rows) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
          for (unsigned long long m = word[h]; m; m &= m - 1)
            list[before++] = (uint16_t)((2 * lane + h) * 64 + __ffsll((long long)m) - 1);
      }
      __syncthreads();
      int first = 0;
      for (int r = 0; r < rows; ++r) {
        const int n = __builtin_amdgcn_readfirstlane(count[r]);
        // the rows' slices go round the waves in one sequence: a row of few slices leaves the other waves to the next rows
        for (int sl = (wave - r * slices) & (kEmbedWaves - 1); n > 0 && sl < slices; sl += kEmbedWaves) {
          const int c = sl * 64 + lane, cc = min(c, nvec_row - 1);
          const uint64_t z_lane = key + kGolden * ((uint64_t)cc * (N / 4));
          float acc[N];
#pragma unroll
          for (int e = 0; e < N; ++e) acc[e] = 0.f;
          for (int i = 0; i < n; i += 64) {
            const int m = min(64, n - i), toks = list[first + i + min(lane, m - 1)];
            for (int k0 = 0; k0 < m; k0 += kEmbedBatch) {
              Vec16<T> a[kEmbedBatch];
              uint64_t z[kEmbedBatch];   // a token's share of z: the same in every lane, so that a lane is left with two products
#pragma unroll
              for (int k = 0; k < kEmbedBatch; ++k) {   // (past the end: the last token again, not added)
                const size_t v = (size_t)(base + __builtin_amdgcn_readlane(toks, min(k0 + k, m - 1))) * nvec_row;
                a[k].load(dx + (v + cc) * N);
                z[k] = kGolden * (v * (N / 4));
              }
#pragma unroll
              for (int k = 0; k < kEmbedBatch; ++k)
                if (k0 + k < m) embed_add<T>(a[k], z_lane + z[k], thr, scale, acc);
            }
          }
          if (c < nvec_row) {
            float* o = d_word + ((size_t)(row0 + r * row_blocks) * nvec_row + c) * N;
#pragma unroll
            for (int e = 0; e < N; ++e) o[e] += acc[e];
          }
        }
        first += n;
      }
    }
    __syncthreads();   // `named`, `count` and `list` are free again
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
