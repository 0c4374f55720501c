// Bandwidth-bound kernels of the layer: LayerNorm, bias+GeLU, bias+dropout+add (paper section 4.2
// names the two fusions; LayerNorm is implied by the 13h term of eq. (2)) and their backward passes.
// All of them move 16 bytes per lane per access, keep fp32 arithmetic, and reduce with wavefront
// shuffles; column sums (bias / LayerNorm parameter gradients) are two-stage and deterministic.
#include "colsum.h"
#include "gelu.h"

namespace ptdp {

static constexpr int kColRows = 32;  // rows per block in the column-sum producers

// The column-sum producers (bias+GeLU backward, bias+dropout+add backward, plain column sums) run workgroups of 64
// column groups (16 bytes each) x 16 row lanes: wave w takes rows r0 + w and r0 + w + 16 of the block's kColRows
// rows, a whole 1 KiB run of one row per access, and width / 512 x rows / 32 workgroups per launch.  The waves' sums
// meet in LDS and are added in a fixed order, one column a thread (by wave 0 alone, eight columns a lane: small and masked layers
// 0.4 % slower, bias+GeLU backward 1024 x 2048 9.2 -> 8.7).  Bound by memory for large calls, by one wave's chain for small ones.
// A wave's two rows go one after the other: sixteen waves hide each other's trips, and both at once (or a loop unrolled for
// more rows) take registers: bias+dropout+add backward 2048 x 12288 22.3 with both requested first, 20.3 so.
// us with 4 row lanes of eight rows each and now, with the finishing launch: bias+GeLU backward 666 x 2048 8.7 -> 7.7, 2048 x
// 4096 15.0 -> 13.6, 2048 x 12288 28.4 -> 28.2, 8192 x 8192 86 -> 76; bias+dropout+add backward 666 x 512 7.1 -> 6.0, 2048 x 25600
// 38.3 -> 36.6, 8192 x 8192 52 -> 46; one row of 1024 4.2 -> 4.4 (waves without a row).
static constexpr int kColLanes = 16;
static inline dim3 colsum_grid(int nvec, int rows) { return dim3((nvec + 63) / 64, (rows + kColRows - 1) / kColRows); }
// column t of a block: the lanes' sums four at a time, then the fours in order
template <int N>
__device__ __forceinline__ float colsum_lanes_sum(const float (*red)[64 * N], int t) {
  float s[kColLanes / 4];
#pragma unroll
  for (int k = 0; k < kColLanes / 4; ++k) s[k] = (red[4 * k][t] + red[4 * k + 1][t]) + (red[4 * k + 2][t] + red[4 * k + 3][t]);
#pragma unroll
  for (int k = 1; k < kColLanes / 4; ++k) s[0] += s[k];
  return s[0];
}
template <int N>
__device__ __forceinline__ void colsum_block_store(float (&acc)[N], float* __restrict__ part, int width) {
  __shared__ __attribute__((aligned(16))) float red[kColLanes][64 * N];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int j = 0; j < N; j += 4) *reinterpret_cast<float4*>(&red[w][lane * N + j]) = make_float4(acc[j], acc[j + 1], acc[j + 2], acc[j + 3]);
  __syncthreads();
  const int t = threadIdx.x, c = blockIdx.x * 64 * N + t;   // one column a thread
  if (t < 64 * N && c < width) part[(size_t)blockIdx.y * width + c] = colsum_lanes_sum<N>(red, t);
}

// ------------------------------------------------------------------------------------------------
// LayerNorm forward: one block per row, the row lives in registers (VPT 16-byte vectors per thread).  Gain and bias are
// requested with the row (without BDA up to 16 values of it per thread, with it up to four vectors): behind the two reductions
// they cost one more round trip, but their registers cost waves.  us for one row alone behind and with, bf16: 2048 x 6144 10.9, 10.2; 666 x
// 12288 7.2, 8.4; 2048 x 12288 17.8, 19.0.
// BDA: the row is first made, x = resid + Drop(in + bias_in), and stored as x_copy (what bda_fwd_kernel does in a pass of its
// own): one read of x and a launch less.  Statistics and output are those of the stored row.  Bound by memory; for small calls by
// the launch and one row's round trips.  us for the two passes and for one, inside a layer: 256 x 256 fp32 7.0 -> 3.5, 2048 x 1024 10.6 -> 6.6,
// 8192 x 2048 35 -> 28, 2048 x 12288 45 -> 42, 2048 x 25600 105 -> 95.
// 128 registers leave room for two workgroups of the widest rows on a compute unit (eight vectors, BDA: 108 us with 134).
// ------------------------------------------------------------------------------------------------
template <typename T> struct LnBda {
  const T *bias, *resid;
  uint64_t key;
  uint32_t thr;
  float scale;
};
template <typename T, int VPT, bool BDA>
__global__ void __launch_bounds__(512, 4)
layernorm_fwd_kernel(const T* __restrict__ x, const T* __restrict__ gain, const T* __restrict__ bias,
                     T* __restrict__ u, float* __restrict__ mu, float* __restrict__ rstd,
                     T* __restrict__ x_copy, int width, float eps, LnBda<T> bda) {
  constexpr int N = Vec16<T>::N;
  constexpr bool kEarly = BDA ? VPT <= 4 : VPT * N <= 16;
  __shared__ float red[16];
  const int nvec = width / N;
  const size_t row = blockIdx.x;
  const T* xr = x + row * width;
  float v[VPT][N];
  float sum = 0.f;
  Vec16<T> t[VPT], res[BDA ? VPT : 1], bin[BDA ? VPT : 1], g[kEarly ? VPT : 1], b[kEarly ? VPT : 1];
#pragma unroll
  for (int i = 0; i < VPT; ++i) {
    const int c = threadIdx.x + i * blockDim.x;
    if (c < nvec) {
      t[i].load(xr + (size_t)c * N);
      if constexpr (BDA) {
        res[i].load(bda.resid + row * width + (size_t)c * N);
        bin[i].load(bda.bias + (size_t)c * N);
      }
    }
  }
  if constexpr (kEarly) {
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
      const int c = threadIdx.x + i * blockDim.x;
      if (c < nvec) {
        g[i].load(gain + (size_t)c * N);
        b[i].load(bias + (size_t)c * N);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < VPT; ++i) {
    const int c = threadIdx.x + i * blockDim.x;
    if (c < nvec) {
      const size_t off = row * width + (size_t)c * N;
      if constexpr (BDA) {
        float af[N], bf[N], rf[N];
        bool keep[N];
        t[i].unpack(af);
        bin[i].unpack(bf);
        res[i].unpack(rf);
        keep_flags<N>(bda.key, (uint64_t)off, bda.thr, keep);
#pragma unroll
        for (int j = 0; j < N; ++j) rf[j] += keep[j] ? (af[j] + bf[j]) * bda.scale : 0.f;
        t[i].pack(rf);
      }
      if (BDA || x_copy) t[i].store(x_copy + off);
      t[i].unpack(v[i]);
#pragma unroll
      for (int j = 0; j < N; ++j) sum += v[i][j];
    }
  }
  const float mean = block_sum(sum, red) / (float)width;
  float sq = 0.f;
#pragma unroll
  for (int i = 0; i < VPT; ++i) {
    const int c = threadIdx.x + i * blockDim.x;
    if (c < nvec) {
#pragma unroll
      for (int j = 0; j < N; ++j) {
        const float d = v[i][j] - mean;
        sq += d * d;
      }
    }
  }
  const float r = rsqrtf(block_sum(sq, red) / (float)width + eps);
  if (threadIdx.x == 0) {
    mu[row] = mean;
    rstd[row] = r;
  }
#pragma unroll
  for (int i = 0; i < VPT; ++i) {
    const int c = threadIdx.x + i * blockDim.x;
    if (c < nvec) {
      Vec16<T> gl, bl, o;
      float gf[N], bf[N], of[N];
      if constexpr (kEarly) {
        gl = g[i];
        bl = b[i];
      } else {
        gl.load(gain + (size_t)c * N);
        bl.load(bias + (size_t)c * N);
      }
      gl.unpack(gf);
      bl.unpack(bf);
#pragma unroll
      for (int j = 0; j < N; ++j) of[j] = gf[j] * ((v[i][j] - mean) * r) + bf[j];
      o.pack(of);
      o.store(u + row * width + (size_t)c * N);
    }
  }
}

// LayerNorm backward: input gradient and the partial sums of the gain / bias gradients in one pass.
//   xhat = (x-mu)*rstd, dxhat = du*gain, dx = resid + rstd*(dxhat - mean(dxhat) - xhat*mean(dxhat*xhat)),
//   dgain[c] = sum_r du*xhat, dbias[c] = sum_r du.
// A block of eight waves walks `rpb` consecutive rows, eight / GW of them at a time: GW waves share a row, so that
// narrow rows cost little or no waiting on other waves and several are under way at once.  Each row of du, x and the
// residual is read once, requested while the previous row is reduced and kept in storage form (fp32 copies would not fit
// next to the column accumulators); every lane keeps the running column sums of its own VPT*N columns.  The groups' sums
// meet in LDS and the block stores them once, as row blockIdx.x of part[][2*width] (gain part first).  dx may alias du or
// resid: a lane overwrites only elements it has read itself.
// Bound by memory for wide rows, by one row's round trip for narrow ones.  us before (one row per block at a time) and
// now, bf16 with residual: 8192 rows x 2048 58 -> 31, 2048 x 4096 26 -> 21.5, 2048 x 12288 58 -> 53, 1024 x 2048
// 11.3 -> 9.9.
// The groups' sums go to LDS all at once and come back four columns a thread (in three rounds of half of the groups each, with one
// float per access: with the finishing launch 666 x 512 13.7 -> 12.8, 2048 x 1024 20.4 -> 18.2, 1024 x 2048 21.8 -> 18.9, 2048 x 4096
// 32.3 -> 28.3, 8192 x 2048 37.3 -> 35.1).
// DROP: the gradient dx, as stored, also goes through the dropout in front of this residual sum, din = Drop'(dx), with the
// column sums of din (what bda_bwd_kernel does in a pass of its own): one read of dx and a launch less.  us for the two
// passes and for one: 8192 x 2048 45 -> 38, 2048 x 12288 77 -> 62, 666 x 512 11.5 -> 5.9.
template <typename T> struct LnDrop {
  T* din;
  float* part;   // [blocks][width]
  uint64_t key;
  uint32_t thr;
  float scale;
};
constexpr int kLnBwdThreads = 512, kLnBwdWaves = kLnBwdThreads / 64;
template <typename T, int VPT, int GW, bool DROP>
__device__ __forceinline__ void
layernorm_bwd_block(const T* du, const T* __restrict__ x, const T* __restrict__ gain, const float* __restrict__ mu,
                    const float* __restrict__ rstd, const T* resid, T* dx, float* __restrict__ part, int rows, int width,
                    int rpb, LnDrop<T> drop) {
  constexpr int N = Vec16<T>::N, NG = kLnBwdWaves / GW, SUMS = DROP ? 3 : 2;
  extern __shared__ __attribute__((aligned(16))) char ln_smem[];
  T* gain_s = reinterpret_cast<T*>(ln_smem);   // the gain row, read twice per row of the block
  __shared__ float red[2][2][kLnBwdWaves];
  const int nvec = width / N, wave = threadIdx.x >> 6, grp = NG == 1 ? 0 : wave / GW, tid = threadIdx.x - grp * GW * 64;
  for (int c = threadIdx.x; c < nvec; c += kLnBwdThreads) {
    Vec16<T> g;
    g.load(gain + (size_t)c * N);
    g.store(gain_s + (size_t)c * N);
  }
  float ag[VPT][N], ab[VPT][N];
#pragma unroll
  for (int i = 0; i < VPT; ++i)
#pragma unroll
    for (int j = 0; j < N; ++j) ag[i][j] = ab[i][j] = 0.f;
  float ad[DROP ? VPT : 1][N];
#pragma unroll
  for (int i = 0; i < (DROP ? VPT : 1); ++i)
#pragma unroll
    for (int j = 0; j < N; ++j) ad[i][j] = 0.f;
  const int r0 = blockIdx.x * rpb, r1 = min(rows, r0 + rpb);
  // the residual gradient is only wanted after the reduction, but requested with the rest: one round trip per row
  typedef Vec16<T> Row[VPT];
  auto load = [&](int r, Row& pa, Row& pb, Row& pr, float& pm, float& prs) {
    if (r >= r1) return;
    const size_t base = (size_t)r * width;
    pm = mu[r];
    prs = rstd[r];
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
      const int c = tid + i * GW * 64;
      if (c < nvec) {
        pa[i].load(du + base + (size_t)c * N);
        pb[i].load(x + base + (size_t)c * N);
        if (resid) pr[i].load(resid + base + (size_t)c * N);
      }
    }
  };
  auto process = [&](int t, Row& a, Row& b, Row& rr, float m, float rs) {
    const int r = r0 + t * NG + grp;
    const bool have = NG == 1 || r < r1;
    float s1 = 0.f, s2 = 0.f;
    if (have) {
#pragma unroll
      for (int i = 0; i < VPT; ++i) {
        const int c = tid + i * GW * 64;
        if (c < nvec) {
          Vec16<T> g;
          float af[N], xf[N], gf[N];
          g.load(gain_s + (size_t)c * N);
          a[i].unpack(af);
          b[i].unpack(xf);
          g.unpack(gf);
#pragma unroll
          for (int j = 0; j < N; ++j) {
            const float xh = (xf[j] - m) * rs, dxh = af[j] * gf[j];
            s1 += dxh;
            s2 += dxh * xh;
            ag[i][j] += af[j] * xh;
            ab[i][j] += af[j];
          }
        }
      }
    }
    s1 = wave_sum(s1);
    s2 = wave_sum(s2);
    if constexpr (GW > 1) {   // both row sums through one barrier; alternating places, so that none is needed behind the reads
      float (&place)[2][kLnBwdWaves] = red[t & 1];
      if ((threadIdx.x & 63) == 0) {
        place[0][wave] = s1;
        place[1][wave] = s2;
      }
      __syncthreads();
      s1 = s2 = 0.f;
#pragma unroll
      for (int w = 0; w < GW; ++w) {
        s1 += place[0][grp * GW + w];
        s2 += place[1][grp * GW + w];
      }
    }
    const float c1 = s1 / (float)width, c2 = s2 / (float)width;
    // the second pass unpacks the stored row again: keeping the first pass's fp32 values alive across the
    // reduction instead would cost two more registers per element and spill
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
      asm volatile("" : "+v"(a[i].raw.x), "+v"(a[i].raw.y), "+v"(a[i].raw.z), "+v"(a[i].raw.w));
      asm volatile("" : "+v"(b[i].raw.x), "+v"(b[i].raw.y), "+v"(b[i].raw.z), "+v"(b[i].raw.w));
    }
    if (have) {
      const size_t base = (size_t)r * width;
#pragma unroll
      for (int i = 0; i < VPT; ++i) {
        const int c = tid + i * GW * 64;
        if (c < nvec) {
          Vec16<T> g, o;
          float af[N], xf[N], gf[N], of[N];
          g.load(gain_s + (size_t)c * N);
          a[i].unpack(af);
          b[i].unpack(xf);
          g.unpack(gf);
          if (resid) {
            rr[i].unpack(of);
          } else {
#pragma unroll
            for (int j = 0; j < N; ++j) of[j] = 0.f;
          }
#pragma unroll
          for (int j = 0; j < N; ++j) of[j] += rs * (af[j] * gf[j] - c1 - (xf[j] - m) * rs * c2);
          o.pack(of);
          o.store(dx + base + (size_t)c * N);
          if constexpr (DROP) {
            const size_t off = base + (size_t)c * N;
            bool keep[N];
            o.unpack(of);
            keep_flags<N>(drop.key, (uint64_t)off, drop.thr, keep);
#pragma unroll
            for (int j = 0; j < N; ++j) {
              of[j] = keep[j] ? of[j] * drop.scale : 0.f;
              ad[i][j] += of[j];
            }
            o.pack(of);
            o.store(drop.din + off);
          }
        }
      }
    }
  };
  const int steps = (r1 - r0 + NG - 1) / NG;   // the same for every group: the barriers are the block's
  __syncthreads();   // gain row visible
  Row a, b, rr, na, nb, nr;
  float m = 0.f, rs = 0.f, nm = 0.f, nrs = 0.f;
  load(r0 + grp, a, b, rr, m, rs);
  for (int t = 0; t < steps; ++t) {
    load(r0 + (t + 1) * NG + grp, na, nb, nr, nm, nrs);
    process(t, a, b, rr, m, rs);
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
      a[i] = na[i];
      b[i] = nb[i];
      rr[i] = nr[i];
    }
    m = nm;
    rs = nrs;
  }
  float* prow = part + (size_t)blockIdx.x * 2 * width;
  if constexpr (NG > 1) {
    // every group puts its sums into LDS, then all threads add them up four columns at a time, in the order of a tree
    float* sums = reinterpret_cast<float*>(ln_smem);   // [group][gain, bias (, din)][column]: the gain row is done with
    __syncthreads();
    float* mine = sums + (size_t)grp * SUMS * width;
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
      const int c = tid + i * GW * 64;
      if (c < nvec) {
#pragma unroll
        for (int j = 0; j < N; j += 4) {
          float* o = mine + (size_t)c * N + j;
          *reinterpret_cast<float4*>(o) = make_float4(ag[i][j], ag[i][j + 1], ag[i][j + 2], ag[i][j + 3]);
          *reinterpret_cast<float4*>(o + width) = make_float4(ab[i][j], ab[i][j + 1], ab[i][j + 2], ab[i][j + 3]);
          if constexpr (DROP) *reinterpret_cast<float4*>(o + 2 * width) = make_float4(ad[i][j], ad[i][j + 1], ad[i][j + 2], ad[i][j + 3]);
        }
      }
    }
    __syncthreads();
    for (int k = 4 * threadIdx.x; k < SUMS * width; k += 4 * kLnBwdThreads) {
      float4 v[NG];
#pragma unroll
      for (int q = 0; q < NG; ++q) v[q] = *reinterpret_cast<const float4*>(sums + (size_t)q * SUMS * width + k);
#pragma unroll
      for (int live = NG / 2; live > 0; live /= 2)
#pragma unroll
        for (int q = 0; q < live; ++q) {
          v[q].x += v[q + live].x;
          v[q].y += v[q + live].y;
          v[q].z += v[q + live].z;
          v[q].w += v[q + live].w;
        }
      *reinterpret_cast<float4*>(k < 2 * width ? prow + k : drop.part + (size_t)blockIdx.x * width + (k - 2 * width)) = v[0];
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < VPT; ++i) {
    const int c = tid + i * GW * 64;
    if (c < nvec) {
#pragma unroll
      for (int j = 0; j < N; ++j) {
        prow[(size_t)c * N + j] = ag[i][j];
        prow[(size_t)width + (size_t)c * N + j] = ab[i][j];
        if constexpr (DROP) drop.part[(size_t)blockIdx.x * width + (size_t)c * N + j] = ad[i][j];
      }
    }
  }
}
template <typename T, int VPT, int GW, bool DROP>
__global__ void __launch_bounds__(kLnBwdThreads)
layernorm_bwd_kernel(const T* du, const T* __restrict__ x, const T* __restrict__ gain, const float* __restrict__ mu,
                     const float* __restrict__ rstd, const T* resid, T* dx, float* __restrict__ part, int rows, int width,
                     int rpb, LnDrop<T> drop) {
  layernorm_bwd_block<T, VPT, GW, DROP>(du, x, gain, mu, rstd, resid, dx, part, rows, width, rpb, drop);
}

// The same with the column sums of another matrix (the QKV bias gradient's first stage) in workgroups of their own behind the
// rows': colsum_rows_kernel's blocks, the sixteen row lanes' sums made by eight waves in two turns, so that the bits are the same.
// One launch less and the sums run beside the rows: fp32 layer 256 wide, 256 tokens 105.2 -> 102.9 us, two layers of 512, 666 tokens
// 267.6 -> 261.7.
template <typename T> struct LnSums {
  const T* in;
  float* part;
  int width, slabs, first;   // slabs of 64 column groups; the first workgroup of the sums
};
template <typename T, int VPT, int GW>
__global__ void __launch_bounds__(kLnBwdThreads)
layernorm_bwd_sums_kernel(const T* du, const T* __restrict__ x, const T* __restrict__ gain, const float* __restrict__ mu,
                          const float* __restrict__ rstd, const T* resid, T* dx, float* __restrict__ part, int rows, int width,
                          int rpb, LnSums<T> q) {
  if ((int)blockIdx.x < q.first) {
    layernorm_bwd_block<T, VPT, GW, false>(du, x, gain, mu, rstd, resid, dx, part, rows, width, rpb, LnDrop<T>{});
    return;
  }
  constexpr int N = Vec16<T>::N;
  extern __shared__ __attribute__((aligned(16))) char ln_smem[];
  float(*red)[64 * N] = reinterpret_cast<float(*)[64 * N]>(ln_smem);
  const int id = (int)blockIdx.x - q.first, tile = id / q.slabs, slab = id - tile * q.slabs;
  const int lane = threadIdx.x & 63, g = slab * 64 + lane, r1 = min(rows, (tile + 1) * kColRows);
  // a wave's four rows are requested at once, at places that exist; those past the end are not added
  constexpr int kTurns = kColLanes / kLnBwdWaves, kPer = kColRows / kColLanes;
  const int w = threadIdx.x >> 6, r0 = tile * kColRows + w;
  Vec16<T> a[kTurns][kPer];
  if (g < q.width / N) {
#pragma unroll
    for (int k = 0; k < kTurns; ++k)
#pragma unroll
      for (int u = 0; u < kPer; ++u) a[k][u].load(q.in + (size_t)min(r0 + k * kLnBwdWaves + u * kColLanes, rows - 1) * q.width + (size_t)g * N);
  }
#pragma unroll
  for (int k = 0; k < kTurns; ++k) {
    float acc[N];
#pragma unroll
    for (int j = 0; j < N; ++j) acc[j] = 0.f;
    if (g < q.width / N) {
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        const bool in = r0 + k * kLnBwdWaves + u * kColLanes < r1;
        float af[N];
        a[k][u].unpack(af);
#pragma unroll
        for (int j = 0; j < N; ++j) acc[j] += in ? af[j] : 0.f;
      }
    }
#pragma unroll
    for (int j = 0; j < N; j += 4)
      *reinterpret_cast<float4*>(&red[w + k * kLnBwdWaves][lane * N + j]) = make_float4(acc[j], acc[j + 1], acc[j + 2], acc[j + 3]);
  }
  __syncthreads();
  const int t = threadIdx.x, c = slab * 64 * N + t;
  if (t < 64 * N && c < q.width) q.part[(size_t)tile * q.width + c] = colsum_lanes_sum<N>(red, t);
}

// The same for rows whose next row does not fit the registers beside the current one (more than four vectors per lane of
// eight waves): one row at a time, requested when its turn comes.  Bound by memory latency: a workgroup of eight waves fills
// the compute unit's registers, so nothing is in flight during a row's reduction (2048 x 25600 bf16: 8 bytes per element of
// three reads and a write, 420 MB in 123 us = 3.4 TB/s).  In bf16 the widest two forms spill (7 vectors per lane: 5
// registers, 8: 59); the form above would spill far more at these widths and takes 180 instead of 127 us.
template <typename T, int VPT>
__global__ void __launch_bounds__(512)
layernorm_bwd_wide_kernel(const T* du, const T* __restrict__ x, const T* __restrict__ gain, const float* __restrict__ mu,
                     const float* __restrict__ rstd, const T* resid, T* dx, float* __restrict__ part, int rows, int width,
                     int rpb) {
  constexpr int N = Vec16<T>::N;
  extern __shared__ __attribute__((aligned(16))) char ln_smem[];
  T* gain_s = reinterpret_cast<T*>(ln_smem);   // the gain row, read twice per row of the block
  __shared__ float red[2][16];
  const int nvec = width / N;
  const int wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  for (int c = threadIdx.x; c < nvec; c += blockDim.x) {
    Vec16<T> g;
    g.load(gain + (size_t)c * N);
    g.store(gain_s + (size_t)c * N);
  }
  float ag[VPT][N], ab[VPT][N];
#pragma unroll
  for (int i = 0; i < VPT; ++i)
#pragma unroll
    for (int j = 0; j < N; ++j) ag[i][j] = ab[i][j] = 0.f;
  const int r0 = blockIdx.x * rpb, r1 = min(rows, r0 + rpb);
  for (int r = r0; r < r1; ++r) {
    const size_t base = (size_t)r * width;
    const float m = mu[r], rs = rstd[r];
    // the residual gradient is only wanted after the reduction, but requested here: one round trip per row
    Vec16<T> a[VPT], b[VPT], rr[VPT];
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
      const int c = threadIdx.x + i * blockDim.x;
      if (c < nvec) {
        a[i].load(du + base + (size_t)c * N);
        b[i].load(x + base + (size_t)c * N);
        if (resid) rr[i].load(resid + base + (size_t)c * N);
      }
    }
    __syncthreads();   // gain row visible (first row); `red` of the previous row no longer read
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
      const int c = threadIdx.x + i * blockDim.x;
      if (c < nvec) {
        Vec16<T> g;
        float af[N], xf[N], gf[N];
        g.load(gain_s + (size_t)c * N);
        a[i].unpack(af);
        b[i].unpack(xf);
        g.unpack(gf);
#pragma unroll
        for (int j = 0; j < N; ++j) {
          const float xh = (xf[j] - m) * rs, dxh = af[j] * gf[j];
          s1 += dxh;
          s2 += dxh * xh;
          ag[i][j] += af[j] * xh;
          ab[i][j] += af[j];
        }
      }
    }
    // both row sums through one pair of barriers
    s1 = wave_sum(s1);
    s2 = wave_sum(s2);
    if ((threadIdx.x & 63) == 0) {
      red[0][wave] = s1;
      red[1][wave] = s2;
    }
    __syncthreads();
    float c1 = 0.f, c2 = 0.f;
    for (int w = 0; w < nw; ++w) {
      c1 += red[0][w];
      c2 += red[1][w];
    }
    c1 /= (float)width;
    c2 /= (float)width;
    // the second pass unpacks the stored row again: keeping the first pass's fp32 values alive across the
    // reduction instead would cost two more registers per element and spill
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
      asm volatile("" : "+v"(a[i].raw.x), "+v"(a[i].raw.y), "+v"(a[i].raw.z), "+v"(a[i].raw.w));
      asm volatile("" : "+v"(b[i].raw.x), "+v"(b[i].raw.y), "+v"(b[i].raw.z), "+v"(b[i].raw.w));
    }
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
      const int c = threadIdx.x + i * blockDim.x;
      if (c < nvec) {
        Vec16<T> g, o;
        float af[N], xf[N], gf[N], of[N];
        g.load(gain_s + (size_t)c * N);
        a[i].unpack(af);
        b[i].unpack(xf);
        g.unpack(gf);
        if (resid) {
          rr[i].unpack(of);
        } else {
#pragma unroll
          for (int j = 0; j < N; ++j) of[j] = 0.f;
        }
#pragma unroll
        for (int j = 0; j < N; ++j) of[j] += rs * (af[j] * gf[j] - c1 - (xf[j] - m) * rs * c2);
        o.pack(of);
        o.store(dx + base + (size_t)c * N);
      }
    }
  }
  float* prow = part + (size_t)blockIdx.x * 2 * width;
#pragma unroll
  for (int i = 0; i < VPT; ++i) {
    const int c = threadIdx.x + i * blockDim.x;
    if (c < nvec) {
#pragma unroll
      for (int j = 0; j < N; ++j) {
        prow[(size_t)c * N + j] = ag[i][j];
        prow[(size_t)width + (size_t)c * N + j] = ab[i][j];
      }
    }
  }
}

__global__ void __launch_bounds__(64 * kFinishWaves)
colsum_finish_kernel(const float* __restrict__ part, int nparts, int stride, float* out0, float* out1, int width) {
  __shared__ float red[kFinishRed];
  colsum_finish_block(ColsumJob{part, nparts, stride, width, out0, out1}, (int)blockIdx.x, kFinishWaves, red);
}

// several finishes in one launch
__global__ void __launch_bounds__(64 * kFinishWaves)
colsum_finish_batch_kernel(ColsumBatchArgs a) {
  __shared__ float red[kFinishRed];
  colsum_finish_id(a, (int)blockIdx.x, kFinishWaves, red);
}

// ------------------------------------------------------------------------------------------------
// bias + GeLU
// ------------------------------------------------------------------------------------------------
template <typename T, int MODE>
__global__ void bias_gelu_fwd_kernel(const T* __restrict__ z, const T* __restrict__ bias, T* __restrict__ g,
                                     size_t total_vec, int nvec_row) {
  constexpr int N = Vec16<T>::N;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total_vec; i += (size_t)gridDim.x * blockDim.x) {
    const int c = (int)(i % nvec_row);
    Vec16<T> a, b;
    float af[N], bf[N];
    a.load(z + i * N);
    b.load(bias + (size_t)c * N);
    a.unpack(af);
    b.unpack(bf);
#pragma unroll
    for (int j = 0; j < N; ++j) af[j] = gelu_f<MODE>(af[j] + bf[j]);
    a.pack(af);
    a.store(g + i * N);
  }
}

// grid (slabs of 64 column groups, row tiles of kColRows); thread owns one 16-byte column group of every sixteenth row.
template <typename T, int MODE>
__global__ void __launch_bounds__(64 * kColLanes)
bias_gelu_bwd_kernel(const T* dg, const T* __restrict__ z, const T* __restrict__ bias, T* dz,
                     float* __restrict__ part, int rows, int width) {
  constexpr int N = Vec16<T>::N;
  const int c = blockIdx.x * 64 + (threadIdx.x & 63);
  const bool valid = c < width / N;
  float bf[N], acc[N];
#pragma unroll
  for (int j = 0; j < N; ++j) acc[j] = 0.f;
  if (valid) {
    Vec16<T> b;
    b.load(bias + (size_t)c * N);
    b.unpack(bf);
    const int r0 = blockIdx.y * kColRows + (threadIdx.x >> 6), r1 = min(rows, (int)(blockIdx.y + 1) * kColRows);
#pragma unroll 1
    for (int r = r0; r < r1; r += kColLanes) {
      const size_t off = (size_t)r * width + (size_t)c * N;
      Vec16<T> a, zz;
      float af[N], zf[N];
      a.load(dg + off);
      zz.load(z + off);
      a.unpack(af);
      zz.unpack(zf);
#pragma unroll
      for (int j = 0; j < N; ++j) {
        af[j] *= gelu_grad_f<MODE>(zf[j] + bf[j]);
        acc[j] += af[j];
      }
      a.pack(af);
      a.store(dz + off);
    }
  }
  colsum_block_store<N>(acc, part, width);
}

// ------------------------------------------------------------------------------------------------
// bias + dropout + add
// ------------------------------------------------------------------------------------------------
template <typename T>
__global__ void bda_fwd_kernel(const T* __restrict__ in, const T* __restrict__ bias, const T* __restrict__ resid,
                               T* __restrict__ out, size_t total_vec, int nvec_row, uint64_t key, uint32_t thr,
                               float scale) {
  constexpr int N = Vec16<T>::N;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total_vec; i += (size_t)gridDim.x * blockDim.x) {
    const int c = (int)(i % nvec_row);
    Vec16<T> a, b, r;
    float af[N], bf[N], rf[N];
    bool keep[N];
    a.load(in + i * N);
    r.load(resid + i * N);
    b.load(bias + (size_t)c * N);
    a.unpack(af);
    b.unpack(bf);
    r.unpack(rf);
    keep_flags<N>(key, (uint64_t)i * N, thr, keep);
#pragma unroll
    for (int j = 0; j < N; ++j) rf[j] += keep[j] ? (af[j] + bf[j]) * scale : 0.f;
    r.pack(rf);
    r.store(out + i * N);
  }
}

template <typename T>
__global__ void __launch_bounds__(64 * kColLanes)
bda_bwd_kernel(const T* __restrict__ dout, T* __restrict__ din, float* __restrict__ part, int rows,
               int width, uint64_t key, uint32_t thr, float scale) {
  constexpr int N = Vec16<T>::N;
  const int c = blockIdx.x * 64 + (threadIdx.x & 63);
  const bool valid = c < width / N;
  float acc[N];
#pragma unroll
  for (int j = 0; j < N; ++j) acc[j] = 0.f;
  if (valid) {
    const int r0 = blockIdx.y * kColRows + (threadIdx.x >> 6), r1 = min(rows, (int)(blockIdx.y + 1) * kColRows);
#pragma unroll 1
    for (int r = r0; r < r1; r += kColLanes) {
      const size_t off = (size_t)r * width + (size_t)c * N;
      Vec16<T> a;
      float af[N];
      bool keep[N];
      a.load(dout + off);
      a.unpack(af);
      keep_flags<N>(key, (uint64_t)off, thr, keep);
#pragma unroll
      for (int j = 0; j < N; ++j) {
        af[j] = keep[j] ? af[j] * scale : 0.f;
        acc[j] += af[j];
      }
      a.pack(af);
      a.store(din + off);
    }
  }
  colsum_block_store<N>(acc, part, width);
}

// part[blockIdx.y][c] = sum of in[r][c] over the block's kColRows rows (first stage of a bias gradient
// whose producer lives in another kernel, e.g. the QKV bias).
template <typename T>
__global__ void __launch_bounds__(64 * kColLanes)
colsum_rows_kernel(const T* __restrict__ in, float* __restrict__ part, int rows, int width) {
  constexpr int N = Vec16<T>::N;
  const int c = blockIdx.x * 64 + (threadIdx.x & 63);
  const bool valid = c < width / N;
  float acc[N];
#pragma unroll
  for (int j = 0; j < N; ++j) acc[j] = 0.f;
  if (valid) {
    const int r0 = blockIdx.y * kColRows + (threadIdx.x >> 6), r1 = min(rows, (int)(blockIdx.y + 1) * kColRows);
#pragma unroll 1
    for (int r = r0; r < r1; r += kColLanes) {
      Vec16<T> a;
      float af[N];
      a.load(in + (size_t)r * width + (size_t)c * N);
      a.unpack(af);
#pragma unroll
      for (int j = 0; j < N; ++j) acc[j] += af[j];
    }
  }
  colsum_block_store<N>(acc, part, width);
}

__global__ void dropout_mask_kernel(uint8_t* keep, int64_t n, uint64_t key, uint32_t thr) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const uint64_t r = mix64(key + kGolden * ((uint64_t)i >> 2));
    keep[i] = ((uint32_t)((r >> (16 * (i & 3))) & 0xffffu) >= thr) ? 1 : 0;
  }
}

// ------------------------------------------------------------------------------------------------
// host launchers
// ------------------------------------------------------------------------------------------------
static inline int ln_threads(int nvec, int* vpt) {
  // smallest register cache that covers the row with at most 512 threads
  int threads = 64;
  while (threads < 512 && threads < nvec) threads <<= 1;
  int v = (nvec + threads - 1) / threads;
  int p = 1;
  while (p < v) p <<= 1;
  *vpt = p;
  return threads;
}

size_t colsum_scratch_bytes(int rows, int width) {
  // one row of `width` floats per tile of kColRows rows (LayerNorm backward passes twice its row width)
  if (rows <= 0 || width <= 0) return 0;
  return (size_t)((rows + kColRows - 1) / kColRows) * (size_t)width * sizeof(float);
}

template <typename T>
static int ln_fwd_t(const void* x, const void* gain, const void* bias, void* u, float* mu, float* rstd, void* x_copy,
                    int rows, int width, float eps, hipStream_t st, const LnBda<T>* bda = nullptr) {
  constexpr int N = Vec16<T>::N;
  int vpt;
  const int threads = ln_threads(width / N, &vpt);
  if (vpt > 8) return PTDP_E_UNSUPPORTED;
  const double bytes = (double)rows * width * sizeof(T) * (bda ? 4 : x_copy ? 3 : 2);
  Launch L(PTDP_K_LN_FWD, bytes, st);
#define PTDP_LN_FWD_FORM(V, BDA, ARGS)                                                                                 \
  hipLaunchKernelGGL((layernorm_fwd_kernel<T, V, BDA>), dim3(rows), dim3(threads), 0, st, (const T*)x, (const T*)gain, \
                     (const T*)bias, (T*)u, mu, rstd, (T*)x_copy, width, eps, ARGS)
#define PTDP_LN_FWD(V)                       \
  if (bda) PTDP_LN_FWD_FORM(V, true, *bda);  \
  else PTDP_LN_FWD_FORM(V, false, LnBda<T>{})
  switch (vpt) {
    case 1: PTDP_LN_FWD(1); break;
    case 2: PTDP_LN_FWD(2); break;
    case 4: PTDP_LN_FWD(4); break;
    default: PTDP_LN_FWD(8); break;
  }
#undef PTDP_LN_FWD
#undef PTDP_LN_FWD_FORM
  return L.status();
}

int launch_layernorm_fwd(int dtype, const void* x, const void* gain, const void* bias, void* u, float* mu,
                         float* rstd, void* x_copy, int rows, int width, float eps, hipStream_t st) {
  if (rows == 0) return PTDP_OK;
  return dtype == PTDP_BF16 ? ln_fwd_t<bf16_t>(x, gain, bias, u, mu, rstd, x_copy, rows, width, eps, st)
                            : ln_fwd_t<float>(x, gain, bias, u, mu, rstd, x_copy, rows, width, eps, st);
}

template <typename T>
static int bda_ln_fwd_t(const void* in, const void* bias_in, const void* resid, void* out, float p, uint64_t key, const void* gain,
                        const void* bias, void* u, float* mu, float* rstd, int rows, int width, float eps, hipStream_t st) {
  const LnBda<T> bda{(const T*)bias_in, (const T*)resid, key, p > 0.f ? dropout_threshold(p) : 0u, 1.0f / (1.0f - p)};
  return ln_fwd_t<T>(in, gain, bias, u, mu, rstd, out, rows, width, eps, st, &bda);
}

int launch_bda_layernorm_fwd(int dtype, const void* in, const void* bias_in, const void* resid, void* out, float p, uint64_t key,
                             const void* gain, const void* bias, void* u, float* mu, float* rstd, int rows, int width, float eps,
                             hipStream_t st) {
  if (rows == 0) return PTDP_OK;
  return dtype == PTDP_BF16 ? bda_ln_fwd_t<bf16_t>(in, bias_in, resid, out, p, key, gain, bias, u, mu, rstd, rows, width, eps, st)
                            : bda_ln_fwd_t<float>(in, bias_in, resid, out, p, key, gain, bias, u, mu, rstd, rows, width, eps, st);
}

int colsum_finish(const float* part, int nparts, int stride, float* out0, float* out1, int width, hipStream_t st, ColsumBatch* defer) {
  if (defer) {
    if (defer->n >= kMaxColsumJobs) return PTDP_E_INVALID_ARG;
    defer->job[defer->n++] = ColsumJob{part, nparts, stride, width, out0, out1};
    return PTDP_OK;
  }
  Launch L(PTDP_K_COLSUM, (double)nparts * stride * sizeof(float), st);
  hipLaunchKernelGGL(colsum_finish_kernel, dim3((width + 63) / 64), dim3(64 * kFinishWaves), 0, st, part, nparts, stride, out0,
                     out1, width);
  return L.status();
}

int launch_colsum_batch(const ColsumBatch& batch, hipStream_t st) {
  if (batch.n == 0) return PTDP_OK;
  double bytes = 0.0;
  const ColsumBatchArgs a = colsum_batch_args(batch, &bytes);
  Launch L(PTDP_K_COLSUM, bytes, st);
  hipLaunchKernelGGL(colsum_finish_batch_kernel, dim3(a.first[kMaxColsumJobs]), dim3(64 * kFinishWaves), 0, st, a);
  return L.status();
}

// Workgroups of column sums up to which they run in LayerNorm backward's launch: about two per compute unit.  Where they are more, the
// launch that is saved weighs little and a kernel of their own reads at a higher rate, in the order in which its input was written.  us
// of a pass through two layers, two launches and one (blocks): 512 wide, 512 tokens (48) 255 -> 250; 1024, 1024 (192) 462 -> 457; 2048, 1024
// (384) 1155 -> 1150; 12288 over eight shards, 2048 (576) 5912 -> 5912; 1024, 4096 (768) 1136 -> 1138; 4096 over four, 4096 (768)
// 2846 -> 2850; 1024, 8192 (1536) 1966 -> 1973; 2048, 8192 (3072) 5238 -> 5269.
static constexpr int kLnSumsBlocks = 512;
// rows walked by one block of the backward kernel: at most 256 blocks (one per compute unit of an MI355X)
static inline int ln_bwd_rows_per_block(int rows) { return rows > 256 ? (rows + 255) / 256 : 1; }

size_t layernorm_bwd_scratch_bytes(int rows, int width) {
  if (rows <= 0 || width <= 0) return 0;
  const int rpb = ln_bwd_rows_per_block(rows);
  return (size_t)((rows + rpb - 1) / rpb) * 2 * (size_t)width * sizeof(float);
}

template <typename T, int VPT, int GW, bool DROP>
static int ln_bwd_launch(const void* du, const void* x, const void* gain, const float* mu, const float* rstd, const void* resid,
                         void* dx, float* part, int rows, int width, int rpb, int nblk, const LnDrop<T>& drop, hipStream_t st) {
  constexpr int NG = kLnBwdWaves / GW, SUMS = DROP ? 3 : 2;
  const size_t gain_bytes = (size_t)width * sizeof(T), sum_bytes = NG > 1 ? (size_t)NG * SUMS * width * sizeof(float) : 0;
  constexpr int kMost = VPT * GW * 64 * Vec16<T>::N * (int)(NG > 1 ? NG * SUMS * sizeof(float) : sizeof(T));   // at the widest row of this form
  auto kern = layernorm_bwd_kernel<T, VPT, GW, DROP>;
  static once_flag_t done[kMaxDevices];
  if (set_dynamic_smem(reinterpret_cast<const void*>(kern), kMost, done) != PTDP_OK) return PTDP_E_HIP;
  hipLaunchKernelGGL(kern, dim3(nblk), dim3(kLnBwdThreads), gain_bytes > sum_bytes ? gain_bytes : sum_bytes, st, (const T*)du,
                     (const T*)x, (const T*)gain, mu, rstd, (const T*)resid, (T*)dx, part, rows, width, rpb, drop);
  return PTDP_OK;
}
template <typename T, int VPT, int GW>
static int ln_bwd_sums_launch(const void* du, const void* x, const void* gain, const float* mu, const float* rstd, const void* resid,
                              void* dx, float* part, int rows, int width, int rpb, int nblk, const LnSums<T>& q, hipStream_t st) {
  constexpr int NG = kLnBwdWaves / GW, kMost = VPT * GW * 64 * Vec16<T>::N * (int)(NG > 1 ? NG * 2 * sizeof(float) : sizeof(T));
  constexpr size_t kRed = (size_t)kColLanes * 64 * Vec16<T>::N * sizeof(float);
  const size_t own = NG > 1 ? (size_t)NG * 2 * width * sizeof(float) : (size_t)width * sizeof(T);   // the sums need more than the gain row
  auto kern = layernorm_bwd_sums_kernel<T, VPT, GW>;
  static once_flag_t done[kMaxDevices];
  if (set_dynamic_smem(reinterpret_cast<const void*>(kern), kMost > (int)kRed ? kMost : (int)kRed, done) != PTDP_OK) return PTDP_E_HIP;
  const int blocks = q.slabs * ((rows + kColRows - 1) / kColRows);
  hipLaunchKernelGGL(kern, dim3(nblk + blocks), dim3(kLnBwdThreads), own > kRed ? own : kRed, st, (const T*)du, (const T*)x,
                     (const T*)gain, mu, rstd, (const T*)resid, (T*)dx, part, rows, width, rpb, q);
  return PTDP_OK;
}
template <typename T, int VPT>
static int ln_bwd_wide_launch(const void* du, const void* x, const void* gain, const float* mu, const float* rstd, const void* resid,
                              void* dx, float* part, int rows, int width, int rpb, int nblk, hipStream_t st) {
  hipLaunchKernelGGL((layernorm_bwd_wide_kernel<T, VPT>), dim3(nblk), dim3(512), (size_t)width * sizeof(T), st, (const T*)du,
                     (const T*)x, (const T*)gain, mu, rstd, (const T*)resid, (T*)dx, part, rows, width, rpb);
  return PTDP_OK;
}
template <typename T>
static int ln_bwd_t(const void* du, const void* x, const void* gain, const float* mu, const float* rstd,
                    const void* resid, void* dx, float* dgain, float* dbias, void* scratch, int rows, int width,
                    hipStream_t st, ColsumBatch* defer, LnDrop<T>* drop = nullptr, LnSums<T>* also = nullptr) {
  constexpr int N = Vec16<T>::N;
  const int slots = (width / N + 63) / 64;   // 64-vector pieces of a row
  if (slots > 8 * kLnBwdWaves) return PTDP_E_UNSUPPORTED;
  float* part = (float*)scratch;
  const int rpb = ln_bwd_rows_per_block(rows), nblk = (rows + rpb - 1) / rpb;
  {
    const double bytes = (double)rows * sizeof(T) * ((double)width * ((resid ? 4 : 3) + (drop ? 1 : 0)) + (also ? also->width : 0));
    if (also) also->first = nblk;
    Launch L(PTDP_K_LN_BWD, bytes, st);
    int rc;
#define PTDP_LN_BWD_WIDE(V) rc = ln_bwd_wide_launch<T, V>(du, x, gain, mu, rstd, resid, dx, part, rows, width, rpb, nblk, st)
#define PTDP_LN_BWD(V, G)                                                                                                       \
  rc = drop ? ln_bwd_launch<T, V, G, true>(du, x, gain, mu, rstd, resid, dx, part, rows, width, rpb, nblk, *drop, st)          \
       : also ? ln_bwd_sums_launch<T, V, G>(du, x, gain, mu, rstd, resid, dx, part, rows, width, rpb, nblk, *also, st)         \
            : ln_bwd_launch<T, V, G, false>(du, x, gain, mu, rstd, resid, dx, part, rows, width, rpb, nblk, LnDrop<T>{}, st)
    // Waves per row: doubled while a lane would hold more than two vectors (2048 columns, 8192 rows: four 50, two 46, one
    // 51 us with the finishing launch) and while a block has fewer rows than groups (their sums' way through LDS costs
    // more than it saves: 1024 rows x 2048 27.7 -> 24.2).  Eight waves hold up to four vectors a lane, beyond that one row at a time.
    int gw = 1;
    while (gw < kLnBwdWaves && (slots > 2 * gw || kLnBwdWaves / gw > rpb)) gw *= 2;
    const int v = (slots + gw - 1) / gw;
    switch (gw * 16 + v) {
      case 16 + 1: PTDP_LN_BWD(1, 1); break;
      case 16 + 2: PTDP_LN_BWD(2, 1); break;
      case 32 + 1: PTDP_LN_BWD(1, 2); break;
      case 32 + 2: PTDP_LN_BWD(2, 2); break;
      case 64 + 1: PTDP_LN_BWD(1, 4); break;
      case 64 + 2: PTDP_LN_BWD(2, 4); break;
      case 128 + 1: PTDP_LN_BWD(1, 8); break;
      case 128 + 2: PTDP_LN_BWD(2, 8); break;
      case 128 + 3: PTDP_LN_BWD(3, 8); break;
      case 128 + 4: rc = ln_bwd_launch<T, 4, 8, false>(du, x, gain, mu, rstd, resid, dx, part, rows, width, rpb, nblk, LnDrop<T>{}, st); break;
      case 128 + 5: PTDP_LN_BWD_WIDE(5); break;
      case 128 + 6: PTDP_LN_BWD_WIDE(6); break;
      case 128 + 7: PTDP_LN_BWD_WIDE(7); break;
      default: PTDP_LN_BWD_WIDE(8); break;
    }
#undef PTDP_LN_BWD
#undef PTDP_LN_BWD_WIDE
    if (rc != PTDP_OK) return rc;
    if (L.status() != PTDP_OK) return L.status();
  }
  return colsum_finish(part, nblk, 2 * width, dgain, dbias, width, st, defer);
}

int launch_layernorm_bwd(int dtype, const void* du, const void* x, const void* gain, const float* mu,
                         const float* rstd, const void* resid, void* dx, float* dgain, float* dbias,
                         void* scratch, int rows, int width, hipStream_t st, ColsumBatch* defer) {
  if (rows == 0) return PTDP_OK;
  return dtype == PTDP_BF16
             ? ln_bwd_t<bf16_t>(du, x, gain, mu, rstd, resid, dx, dgain, dbias, scratch, rows, width, st, defer)
             : ln_bwd_t<float>(du, x, gain, mu, rstd, resid, dx, dgain, dbias, scratch, rows, width, st, defer);
}

// Rows of up to 24 x 64 vectors (12288 bf16 elements): beyond, the third set of column sums does not fit the registers.
template <typename T>
static int ln_bwd_drop_t(const void* du, const void* x, const void* gain, const float* mu, const float* rstd, const void* resid,
                         void* dx, float* dgain, float* dbias, void* scratch, void* din, float* dbias_in, void* scratch_in, float p,
                         uint64_t key, int rows, int width, hipStream_t st, ColsumBatch* defer) {
  if (width / Vec16<T>::N > 24 * 64) {
    const int rc = ln_bwd_t<T>(du, x, gain, mu, rstd, resid, dx, dgain, dbias, scratch, rows, width, st, defer);
    if (rc != PTDP_OK) return rc;
    return launch_bda_bwd(sizeof(T) == 2 ? PTDP_BF16 : PTDP_F32, dx, din, dbias_in, scratch_in, rows, width, p, key, st, defer);
  }
  LnDrop<T> drop{(T*)din, (float*)scratch_in, key, p > 0.f ? dropout_threshold(p) : 0u, 1.0f / (1.0f - p)};
  const int rc = ln_bwd_t<T>(du, x, gain, mu, rstd, resid, dx, dgain, dbias, scratch, rows, width, st, defer, &drop);
  if (rc != PTDP_OK) return rc;
  const int rpb = ln_bwd_rows_per_block(rows), nblk = (rows + rpb - 1) / rpb;
  return colsum_finish(drop.part, nblk, width, dbias_in, nullptr, width, st, defer);
}

size_t layernorm_bwd_drop_scratch_bytes(int rows, int width) {
  const size_t a = colsum_scratch_bytes(rows, width), b = layernorm_bwd_scratch_bytes(rows, width) / 2;
  return a > b ? a : b;
}

int launch_layernorm_bwd_drop(int dtype, const void* du, const void* x, const void* gain, const float* mu, const float* rstd,
                              const void* resid, void* dx, float* dgain, float* dbias, void* scratch, void* din, float* dbias_in,
                              void* scratch_in, float p, uint64_t key, int rows, int width, hipStream_t st, ColsumBatch* defer) {
  if (rows == 0) return PTDP_OK;
  return dtype == PTDP_BF16 ? ln_bwd_drop_t<bf16_t>(du, x, gain, mu, rstd, resid, dx, dgain, dbias, scratch, din, dbias_in, scratch_in,
                                                    p, key, rows, width, st, defer)
                            : ln_bwd_drop_t<float>(du, x, gain, mu, rstd, resid, dx, dgain, dbias, scratch, din, dbias_in, scratch_in,
                                                   p, key, rows, width, st, defer);
}

static inline int stream_grid(size_t total_vec) {
  size_t blocks = (total_vec + 255) / 256;
  const size_t cap = 256 * 32;  // 32 blocks per CU, grid-stride beyond (16: bias+dropout+add 4-5 % slower; 64 and more: the same)
  return (int)(blocks < cap ? (blocks ? blocks : 1) : cap);
}

template <typename T>
static int gelu_fwd_t(int mode, const void* z, const void* bias, void* g, int rows, int width, hipStream_t st) {
  constexpr int N = Vec16<T>::N;
  const size_t total = (size_t)rows * width / N;
  Launch L(PTDP_K_GELU_FWD, (double)rows * width * sizeof(T) * 2, st);
  if (mode == PTDP_GELU_TANH)
    hipLaunchKernelGGL((bias_gelu_fwd_kernel<T, PTDP_GELU_TANH>), dim3(stream_grid(total)), dim3(256), 0, st,
                       (const T*)z, (const T*)bias, (T*)g, total, width / N);
  else
    hipLaunchKernelGGL((bias_gelu_fwd_kernel<T, PTDP_GELU_ERF>), dim3(stream_grid(total)), dim3(256), 0, st,
                       (const T*)z, (const T*)bias, (T*)g, total, width / N);
  return L.status();
}

int launch_bias_gelu_fwd(int dtype, int mode, const void* z, const void* bias, void* g, int rows, int width,
                         hipStream_t st) {
  if (rows == 0) return PTDP_OK;
  return dtype == PTDP_BF16 ? gelu_fwd_t<bf16_t>(mode, z, bias, g, rows, width, st)
                            : gelu_fwd_t<float>(mode, z, bias, g, rows, width, st);
}

template <typename T>
static int gelu_bwd_t(int mode, const void* dg, const void* z, const void* bias, void* dz, float* dbias,
                      void* scratch, int rows, int width, hipStream_t st, ColsumBatch* defer) {
  constexpr int N = Vec16<T>::N;
  const dim3 grid = colsum_grid(width / N, rows);
  float* part = (float*)scratch;
  {
    Launch L(PTDP_K_GELU_BWD, (double)rows * width * sizeof(T) * 3, st);
    if (mode == PTDP_GELU_TANH)
      hipLaunchKernelGGL((bias_gelu_bwd_kernel<T, PTDP_GELU_TANH>), grid, dim3(64 * kColLanes), 0, st, (const T*)dg,
                         (const T*)z, (const T*)bias, (T*)dz, part, rows, width);
    else
      hipLaunchKernelGGL((bias_gelu_bwd_kernel<T, PTDP_GELU_ERF>), grid, dim3(64 * kColLanes), 0, st, (const T*)dg,
                         (const T*)z, (const T*)bias, (T*)dz, part, rows, width);
    if (L.status() != PTDP_OK) return L.status();
  }
  return colsum_finish(part, grid.y, width, dbias, nullptr, width, st, defer);
}

int launch_bias_gelu_bwd(int dtype, int mode, const void* dg, const void* z, const void* bias, void* dz,
                         float* dbias, void* scratch, int rows, int width, hipStream_t st, ColsumBatch* defer) {
  if (rows == 0) return PTDP_OK;
  return dtype == PTDP_BF16 ? gelu_bwd_t<bf16_t>(mode, dg, z, bias, dz, dbias, scratch, rows, width, st, defer)
                            : gelu_bwd_t<float>(mode, dg, z, bias, dz, dbias, scratch, rows, width, st, defer);
}

template <typename T>
static int bda_fwd_t(const void* in, const void* bias, const void* resid, void* out, int rows, int width, float p,
                     uint64_t key, hipStream_t st) {
  constexpr int N = Vec16<T>::N;
  const size_t total = (size_t)rows * width / N;
  Launch L(PTDP_K_BDA_FWD, (double)rows * width * sizeof(T) * 3, st);
  hipLaunchKernelGGL((bda_fwd_kernel<T>), dim3(stream_grid(total)), dim3(256), 0, st, (const T*)in, (const T*)bias,
                     (const T*)resid, (T*)out, total, width / N, key, p > 0.f ? dropout_threshold(p) : 0u,
                     1.0f / (1.0f - p));
  return L.status();
}

int launch_bda_fwd(int dtype, const void* in, const void* bias, const void* resid, void* out, int rows, int width,
                   float p, uint64_t key, hipStream_t st) {
  if (rows == 0) return PTDP_OK;
  return dtype == PTDP_BF16 ? bda_fwd_t<bf16_t>(in, bias, resid, out, rows, width, p, key, st)
                            : bda_fwd_t<float>(in, bias, resid, out, rows, width, p, key, st);
}

template <typename T>
static int bda_bwd_t(const void* dout, void* din, float* dbias, void* scratch, int rows, int width, float p,
                     uint64_t key, hipStream_t st, ColsumBatch* defer) {
  constexpr int N = Vec16<T>::N;
  const dim3 grid = colsum_grid(width / N, rows);
  float* part = (float*)scratch;
  {
    Launch L(PTDP_K_BDA_BWD, (double)rows * width * sizeof(T) * 2, st);
    hipLaunchKernelGGL((bda_bwd_kernel<T>), grid, dim3(64 * kColLanes), 0, st, (const T*)dout, (T*)din, part, rows, width, key,
                       p > 0.f ? dropout_threshold(p) : 0u, 1.0f / (1.0f - p));
    if (L.status() != PTDP_OK) return L.status();
  }
  return colsum_finish(part, grid.y, width, dbias, nullptr, width, st, defer);
}

int launch_bda_bwd(int dtype, const void* dout, void* din, float* dbias, void* scratch, int rows, int width, float p,
                   uint64_t key, hipStream_t st, ColsumBatch* defer) {
  if (rows == 0) return PTDP_OK;
  return dtype == PTDP_BF16 ? bda_bwd_t<bf16_t>(dout, din, dbias, scratch, rows, width, p, key, st, defer)
                            : bda_bwd_t<float>(dout, din, dbias, scratch, rows, width, p, key, st, defer);
}

// Column-sum partials for callers that may not allocate: one array per device, kept until the process
// ends.  In host code `scratch` is only a handle for hipGetSymbolAddress, never a device address: every
// launch below is handed the address looked up once per device, with that device current.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
static std::atomic<void*> g_scratch_ptr[kMaxDevices];

static int static_scratch(void** out) {
  const int d = device_slot();
  if (d < 0) return PTDP_E_HIP;
  void* ptr = g_scratch_ptr[d].load(std::memory_order_acquire);
  if (!ptr) {
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) return PTDP_E_HIP;
    g_scratch_ptr[d].store(ptr, std::memory_order_release);   // racing threads store the same address
  }
  *out = ptr;
  return PTDP_OK;
}

// launch_bda_bwd with the partials in this device's static array (every partial that the finish kernel reads
// is written by the first kernel of the same call, so nothing has to be cleared between calls)
int launch_bda_bwd_static(int dtype, const void* dout, void* din, float* dbias, int rows, int width, float p,
                          uint64_t key, hipStream_t st) {
  if (colsum_scratch_bytes(rows, width) > kStaticScratchBytes) return PTDP_E_TOO_SMALL;
  if (rows == 0) return PTDP_OK;
  void* ptr = nullptr;
  const int rc = static_scratch(&ptr);
  if (rc != PTDP_OK) return rc;
  return launch_bda_bwd(dtype, dout, din, dbias, ptr, rows, width, p, key, st, nullptr);
}

// Rows of up to 24 x 64 vectors: the forms that the launch below has.
bool layernorm_bwd_takes_sums(int dtype, int rows, int width, int in_width) {
  const int n = dtype == PTDP_BF16 ? 8 : 4;
  const dim3 g = colsum_grid(in_width / n, rows);
  return rows > 0 && width / n <= 24 * 64 && (long long)g.x * g.y <= kLnSumsBlocks;
}
template <typename T>
static int ln_bwd_sums_t(const void* du, const void* x, const void* gain, const float* mu, const float* rstd, const void* resid,
                         void* dx, float* dgain, float* dbias, void* scratch, const void* in, float* sums, void* scratch_in,
                         int in_width, int rows, int width, hipStream_t st, ColsumBatch* defer) {
  const dim3 g = colsum_grid(in_width / Vec16<T>::N, rows);
  LnSums<T> also{(const T*)in, (float*)scratch_in, in_width, (int)g.x, 0};
  const int rc = ln_bwd_t<T>(du, x, gain, mu, rstd, resid, dx, dgain, dbias, scratch, rows, width, st, defer, nullptr, &also);
  if (rc != PTDP_OK) return rc;
  return colsum_finish((const float*)scratch_in, g.y, in_width, sums, nullptr, in_width, st, defer);
}
int launch_layernorm_bwd_sums(int dtype, const void* du, const void* x, const void* gain, const float* mu, const float* rstd,
                              const void* resid, void* dx, float* dgain, float* dbias, void* scratch, const void* in, float* sums,
                              void* scratch_in, int in_width, int rows, int width, hipStream_t st, ColsumBatch* defer) {
  return dtype == PTDP_BF16 ? ln_bwd_sums_t<bf16_t>(du, x, gain, mu, rstd, resid, dx, dgain, dbias, scratch, in, sums, scratch_in,
                                                    in_width, rows, width, st, defer)
                            : ln_bwd_sums_t<float>(du, x, gain, mu, rstd, resid, dx, dgain, dbias, scratch, in, sums, scratch_in,
                                                   in_width, rows, width, st, defer);
}

template <typename T>
static int colsum_t(const void* in, float* out, void* scratch, int rows, int width, hipStream_t st, ColsumBatch* defer) {
  constexpr int N = Vec16<T>::N;
  const dim3 grid = colsum_grid(width / N, rows);
  float* part = (float*)scratch;
  {
    Launch L(PTDP_K_COLSUM, (double)rows * width * sizeof(T), st);
    hipLaunchKernelGGL((colsum_rows_kernel<T>), grid, dim3(64 * kColLanes), 0, st, (const T*)in, part, rows, width);
    if (L.status() != PTDP_OK) return L.status();
  }
  return colsum_finish(part, grid.y, width, out, nullptr, width, st, defer);
}

int launch_colsum(int dtype, const void* in, float* out, void* scratch, int rows, int width, hipStream_t st,
                  ColsumBatch* defer) {
  if (rows == 0) return PTDP_OK;
  return dtype == PTDP_BF16 ? colsum_t<bf16_t>(in, out, scratch, rows, width, st, defer)
                            : colsum_t<float>(in, out, scratch, rows, width, st, defer);
}

int launch_dropout_mask(uint8_t* keep, int64_t n, float p, uint64_t key, hipStream_t st) {
  if (n == 0) return PTDP_OK;
  Launch L(PTDP_K_OTHER, (double)n, st);
  hipLaunchKernelGGL(dropout_mask_kernel, dim3(stream_grid((size_t)n)), dim3(256), 0, st, keep, n, key,
                     p > 0.f ? dropout_threshold(p) : 0u);
  return L.status();
}

}  // namespace ptdp
