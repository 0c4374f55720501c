// Fused self-attention of one tensor-parallel shard (paper section 2.3: heads split over the ranks;
// section 4.2: scale + mask + softmax fused, with the implicit causal mask or a general byte mask;
// here the two batched GEMMs Q K^T and P V of the appendix are fused in as well, so the s x s matrix
// never reaches HBM).
//
// qkv is [s, b, 3*hp] with columns [Q heads | K heads | V heads]; for sample j and local head e the
// row of token i starts at qkv + (i*b + j)*3*hp + {0, hp, 2hp} + e*dh.
//
// bf16 forward: S^T = K Q^T and O^T = V^T P^T on v_mfma_f32_32x32x16_bf16, so that the softmax
// probabilities leave the first MFMA already in the register layout the second one wants as its
// B operand.  One wave owns 32 queries; the waves of a block share K and V tiles in LDS.
// fp32: the same two-step form on v_mfma_f32_16x16x4_f32, operands straight from memory.
#include "common.h"
#include <type_traits>

namespace ptdp {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;

// General mask (section 4.2: the fused softmax "with general masking"): a hidden score is replaced
// by this value before the softmax, so a row without any visible key attends uniformly, and no
// gradient flows to q and k through a hidden score.  mask is [b, s, s] bytes, nonzero = hidden.
constexpr float kMaskFill = -10000.f;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;

// ------------------------------------------------------------------------------------------------
// fp32 kernels on v_mfma_f32_16x16x4_f32 (fp32 products and sums).  A workgroup of NW waves (four, or eight
// where workgroups are few) owns 16 queries (forward, dQ) or 16 keys (dK, dV) of one head.  The walk over the other side is PARTS
// partial sums, each over every PARTS-th 16-row tile, that meet in LDS in a fixed order (eight instead of four: error against 64
// bits 1 to 13 % smaller).  PARTS follows from s and dh alone and a wave makes PARTS / NW of them one after the other, so that a
// sample's results have the same bits whatever else is in the call.  Operands come from memory straight into fragments: lane (c = lane & 15,
// g = lane >> 4) carries four consecutive dh of row c (elements 16 i + 4 g .. +3 of step i; both factors of a product
// share that order), and the score tile S^T comes out with column c = the workgroup's row and rows 4 g + r = the tile's,
// which is the second product's B operand as it stands.  These are small calls (fp32 is the precision of small
// configurations): what counts is the length of one wave's chain and the number of waves.  128 tokens x 4 heads x 2
// samples, dh 64: forward 68 -> 9 us, backward 155 -> 25 us against one wave per row that reduced every
// score across the wave.
// ND: steps of 16 dh (dh rounded up; the lanes past dh hold zeros).
// ------------------------------------------------------------------------------------------------
constexpr int kF32Rows = 16;
constexpr int kMaxF32Dh = 256;

template <int ND> struct F32Frag { f32x4_t v[ND]; };
// four consecutive dh of one row per step; `row` must be readable
template <int ND> __device__ __forceinline__ void f32_load(F32Frag<ND>& f, const float* __restrict__ row, int g, int dh) {
#pragma unroll
  for (int i = 0; i < ND; ++i) {
    const int d = 16 * i + 4 * g;
    f.v[i] = d < dh ? *reinterpret_cast<const f32x4_t*>(row + d) : f32x4_t{0.f, 0.f, 0.f, 0.f};
  }
}
// 16 x 16 products of rows a (result rows 4 g + r) and rows b (result column c): MFMAs FIRST .. FIRST + N - 1 of 4 dh each
// (of 4 ND), added up as a tree whose leaves are chains of kF32Leaf.
// One chain over dh had up to twice the error of the tree.
template <int ND, int FIRST = 0, int N = 4 * ND>
__device__ __forceinline__ f32x4_t f32_scores(const F32Frag<ND>& a, const F32Frag<ND>& b) {
  constexpr int kF32Leaf = ND > 10 ? 8 : 4;   // (heads beyond 160: a shorter chain's registers would spill)
  if constexpr (N > kF32Leaf) {
    constexpr int kHalf = (N / kF32Leaf + 1) / 2 * kF32Leaf;
    return f32_scores<ND, FIRST, kHalf>(a, b) + f32_scores<ND, FIRST + kHalf, N - kHalf>(a, b);
  } else {
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = FIRST; i < FIRST + N; ++i) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v[i / 4][i % 4], b.v[i / 4][i % 4], acc, 0, 0, 0);
    return acc;
  }
}
// acc^T[16 dh rows x 16 columns] += X^T w for the tile rows row0 .. row0 + 15 of X (rows from s on count as zeros; their
// weights are zero).  Register r of acc[t]: dh 16 t + 4 g + r of column c.
// A weight that the causal mask hides is zero, but zero times an infinite or undefined element is not: in a tile on the
// diagonal (`vis`: bit r = row 4 g + r is visible to column c) such elements enter the product as zeros and are added
// afterwards to the columns that see them, so that no bit of the other columns depends on them.
template <int ND>
__device__ __forceinline__ void f32_accumulate(f32x4_t (&acc)[ND], f32x4_t w, const float* __restrict__ X, size_t rs, int row0, int s,
                                               int dh, bool diag, uint32_t vis, int lane) {
  const int c = lane & 15, g = lane >> 4;
  auto at = [&](int t, int r) {
    const int row = row0 + 4 * g + r, d = 16 * t + c;
    const float x = X[(size_t)min(row, s - 1) * rs + min(d, dh - 1)];
    return row < s && d < dh ? x : 0.f;
  };
  if (!diag) {
#pragma unroll
    for (int t = 0; t < ND; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(at(t, r), w[r], acc[t], 0, 0, 0);
    return;
  }
  bool finite = true;
#pragma unroll
  for (int t = 0; t < ND; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float x = at(t, r);
      const bool ok = fabsf(x) < INFINITY;
      finite = finite && ok;
      acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(ok ? x : 0.f, w[r], acc[t], 0, 0, 0);
    }
  if (__all(finite)) return;
#pragma unroll 1
  for (int row = 0; row < 16 && row0 + row < s; ++row) {
    const int src = (row >> 2) * 16 + c, k = row & 3;
    const float wr = __shfl(k & 2 ? (k & 1 ? w[3] : w[2]) : (k & 1 ? w[1] : w[0]), src, 64);
    const bool seen = (__shfl((int)vis, src, 64) >> k) & 1;
    const float* x = X + (size_t)(row0 + row) * rs + 4 * g;
#pragma unroll
    for (int t = 0; t < ND; ++t)
      if (16 * t + 4 * g < dh) {
        const f32x4_t v = *reinterpret_cast<const f32x4_t*>(x + 16 * t);
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (seen && !(fabsf(v[r]) < INFINITY)) acc[t][r] += wr * v[r];
      }
  }
}
// Four waves with a part each: waves 1 .. 3 hand theirs to wave 0 (added in that order); returns true in wave 0.  part: 3 * ND * 64 vectors.
template <int ND> __device__ __forceinline__ bool f32_join(f32x4_t (&acc)[ND], f32x4_t* part, int wave, int lane) {
  __syncthreads();
  if (wave > 0) {
#pragma unroll
    for (int t = 0; t < ND; ++t) part[((wave - 1) * ND + t) * 64 + lane] = acc[t];
  }
  __syncthreads();
  if (wave > 0) return false;
#pragma unroll
  for (int w = 0; w < 3; ++w)
#pragma unroll
    for (int t = 0; t < ND; ++t) acc[t] += part[(w * ND + t) * 64 + lane];
  return true;
}
// Eight parts: part w and part w + 4, then those four sums in order.  Four waves make two parts each: the earlier one waits in the
// wave's own place (f32_set_aside) and f32_add_pair adds it to the later one; of eight waves the upper four hand theirs to the lower.
// place: 4 * ND * 64 vectors per sum.
template <int ND> __device__ __forceinline__ void f32_set_aside(f32x4_t (&acc)[ND], f32x4_t* place, int wave, int lane) {
#pragma unroll
  for (int t = 0; t < ND; ++t) {
    place[(wave * ND + t) * 64 + lane] = acc[t];
    acc[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  }
}
// (the products are rounded by themselves, or a form might fuse with the sum behind them what another does not)
template <int ND> __device__ __forceinline__ void f32_scale(f32x4_t (&acc)[ND], float f) {
#pragma clang fp contract(off)
#pragma unroll
  for (int t = 0; t < ND; ++t) acc[t] *= f;
}
template <int ND, int NW> __device__ __forceinline__ void f32_add_pair(f32x4_t (&acc)[ND], const f32x4_t* place, float factor, int wave, int lane) {
  if (NW == 8 && wave >= 4) return;
  f32x4_t other[ND];
#pragma unroll
  for (int t = 0; t < ND; ++t) other[t] = place[(wave * ND + t) * 64 + lane];
  if (NW == 4) f32_scale<ND>(other, factor);
#pragma unroll
  for (int t = 0; t < ND; ++t) acc[t] += other[t];
}
// NS sums at once; sum q ends up in wave q.  factor: of the parts set aside (NW = 4)
template <int ND, int NW, int NS>
__device__ __forceinline__ void f32_join_eight(f32x4_t (&acc)[NS][ND], f32x4_t* place, float factor, int wave, int lane) {
  constexpr int kSum = 4 * ND * 64;
  if (NW == 8) {
    if (wave >= 4) {
#pragma unroll
      for (int q = 0; q < NS; ++q) f32_set_aside<ND>(acc[q], place + q * kSum, wave - 4, lane);
    }
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < NS; ++q) {
    f32_add_pair<ND, NW>(acc[q], place + q * kSum, factor, wave, lane);
    if (wave < 4 && wave != q) {
#pragma unroll
      for (int t = 0; t < ND; ++t) place[q * kSum + (wave * ND + t) * 64 + lane] = acc[q][t];
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NS; ++q)
    if (wave == q) {
#pragma unroll
      for (int t = 0; t < ND; ++t) {
        f32x4_t sum = q == 0 ? acc[q][t] : place[q * kSum + t * 64 + lane];
#pragma unroll
        for (int w = 1; w < 4; ++w) sum += w == q ? acc[q][t] : place[q * kSum + (w * ND + t) * 64 + lane];
        acc[q][t] = sum;
      }
    }
}
// vectors of LDS for `sums` sums
constexpr int f32_places(int nd, int parts, int sums) { return (parts == 8 ? sums * 4 : 3) * nd * 64; }
template <int ND> __device__ __forceinline__ void f32_store(float* row, const f32x4_t (&acc)[ND], int g, int dh) {
#pragma unroll
  for (int t = 0; t < ND; ++t)
    if (16 * t + 4 * g < dh) *reinterpret_cast<f32x4_t*>(row + 16 * t + 4 * g) = acc[t];
}

// Waves on a SIMD that the forward kernel's registers leave with a part to each of four waves; the walk in two turns had taken eight
// registers more and with them one of these waves (1024 workgroups of heads of 96 x 128 30 -> 47 us).
constexpr int f32_fwd_waves(int nd, int nw) { return nw == 8 ? 2 : nd == 2 ? 7 : nd == 4 ? 5 : nd == 6 ? 4 : nd == 8 ? 3 : 1; }
template <int ND, int NW, int PARTS>
__global__ void __launch_bounds__(64 * NW, f32_fwd_waves(ND, NW))
attn_fwd_f32(const float* __restrict__ qkv, float* __restrict__ ctx, float* __restrict__ lse, int s, int b, int heads, int dh,
             const uint8_t* __restrict__ mask, int causal) {
  __shared__ f32x4_t part[f32_places(ND, PARTS, 1)];
  __shared__ float stat[2][PARTS][16];
  const int e = blockIdx.y, j = blockIdx.z, wave = threadIdx.x >> 6, lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
  const int q0 = ((int)gridDim.x - 1 - (int)blockIdx.x) * kF32Rows, my_q = q0 + c;   // long rows first
  const int hp = heads * dh;
  const size_t rs = (size_t)b * 3 * hp;
  const float* base = qkv + (size_t)j * 3 * hp + (size_t)e * dh;
  const float scale = rsqrtf((float)dh);
  F32Frag<ND> q;
  f32_load<ND>(q, base + (size_t)min(my_q, s - 1) * rs, g, dh);
  f32x4_t acc[1][ND];
  f32x4_t (&o)[ND] = acc[0];
#pragma unroll
  for (int t = 0; t < ND; ++t) o[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float m;
  const int ntiles = ((causal ? min(q0 + kF32Rows, s) : s) + kF32Rows - 1) / kF32Rows;
  const uint8_t* mrow = (!causal && mask) ? mask + ((size_t)j * s + min(my_q, s - 1)) * s : nullptr;
#pragma unroll 1
  for (int pt = wave; pt < PARTS; pt += NW) {   // the wave's parts
    float l = 0.f;
    m = -INFINITY;
    for (int kt = pt; kt < ntiles; kt += PARTS) {
      const int key0 = kt * kF32Rows;
      F32Frag<ND> k;
      f32_load<ND>(k, base + hp + (size_t)min(key0 + c, s - 1) * rs, g, dh);
      f32x4_t p = f32_scores<ND>(k, q);
      uint32_t vis = 0;
      float mx = m;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int key = key0 + 4 * g + r;
        p[r] *= scale;
        if (mrow && key < s && mrow[key]) p[r] = kMaskFill;
        const bool ok = key < s && (!causal || key <= my_q);
        p[r] = ok ? p[r] : -INFINITY;
        vis |= (uint32_t)ok << r;
        mx = fmaxf(mx, p[r]);
      }
      const LaneHalves mr = lane_rows(mx);
      const LaneHalves mh = lane_halves(fmaxf(mr.lo, mr.hi));
      mx = fmaxf(mh.lo, mh.hi);
      const float ref = mx == -INFINITY ? 0.f : mx;   // only scores of -inf so far: weights of zero, not exp(-inf + inf)
      const float corr = __expf(m - ref);
      m = mx;
      l *= corr;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        p[r] = __expf(p[r] - ref);
        l += p[r];
      }
#pragma unroll
      for (int t = 0; t < ND; ++t) o[t] *= corr;
      f32_accumulate<ND>(o, p, base + 2 * hp, rs, key0, s, dh, causal && key0 + kF32Rows > q0, vis, lane);
    }
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    if (g == 0) {
      stat[0][pt][c] = m;
      stat[1][pt][c] = l;
    }
    if (pt + NW < PARTS) f32_set_aside<ND>(o, part, wave, lane);
  }
  __syncthreads();
  float mall = stat[0][0][c], lall = 0.f;   // the first part always has a tile
#pragma unroll
  for (int w = 1; w < PARTS; ++w) mall = fmaxf(mall, stat[0][w][c]);
#pragma unroll
  for (int w = 0; w < PARTS; ++w) lall += stat[1][w][c] * __expf(stat[0][w][c] - mall);
  f32_scale<ND>(o, __expf(m - mall));   // a part without a tile: m = -inf, its zeros are multiplied by zero
  if constexpr (PARTS == 8) f32_join_eight<ND, NW, 1>(acc, part, __expf(stat[0][wave][c] - mall), wave, lane);
  else f32_join<ND>(o, part, wave, lane);
  if (wave > 0 || my_q >= s) return;
#pragma unroll
  for (int t = 0; t < ND; ++t) o[t] /= lall;
  f32_store<ND>(ctx + ((size_t)my_q * b + j) * hp + (size_t)e * dh, o, g, dh);
  if (g == 0) lse[((size_t)j * heads + e) * s + my_q] = mall + __logf(lall);
}

// delta = sum_d dctx * ctx of 16 rows (o, dc): the diagonal of ctx dctx^T, summed in the order of dP below: with one visible key
// dP - delta is exactly zero.  Lane (c, g) holds it for row c if the tile's rows are columns, for rows 4 g + r otherwise.
template <int ND> __device__ __forceinline__ float f32_delta_column(const F32Frag<ND>& o, const F32Frag<ND>& dc, int c) {
  const f32x4_t x = f32_scores<ND>(o, dc);
  const float mine = (c & 2) ? ((c & 1) ? x[3] : x[2]) : ((c & 1) ? x[1] : x[0]);
  return __shfl(mine, (c >> 2) * 16 + c, 64);
}
template <int ND> __device__ __forceinline__ f32x4_t f32_delta_rows(const F32Frag<ND>& o, const F32Frag<ND>& dc, int g) {
  const f32x4_t x = f32_scores<ND>(o, dc);
  f32x4_t d;
#pragma unroll
  for (int r = 0; r < 4; ++r) d[r] = __shfl(x[r], 16 * g + 4 * g + r, 64);
  return d;
}

// dQ of 16 queries, and (delta not NULL) their delta for the dK/dV kernel
template <int ND, int NW, int PARTS>
__device__ __forceinline__ void f32_dq_block(const float* __restrict__ qkv, const float* __restrict__ ctx, const float* __restrict__ dctx,
                                             const float* __restrict__ lse, float* __restrict__ delta, float* __restrict__ dqkv, int s, int b,
                                             int heads, int dh, const uint8_t* __restrict__ mask, int causal, int blk, f32x4_t* part) {
  const int e = blockIdx.y, j = blockIdx.z, wave = threadIdx.x >> 6, lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
  const int q0 = blk * kF32Rows, my_q = q0 + c, qr = min(my_q, s - 1);
  const int hp = heads * dh;
  const size_t rs = (size_t)b * 3 * hp;
  const float* base = qkv + (size_t)j * 3 * hp + (size_t)e * dh;
  const float scale = rsqrtf((float)dh);
  const size_t stat = ((size_t)j * heads + e) * s + qr, out = ((size_t)qr * b + j) * hp + (size_t)e * dh;
  F32Frag<ND> q, dc;
  f32_load<ND>(q, base + (size_t)qr * rs, g, dh);
  f32_load<ND>(dc, dctx + out, g, dh);
  float D;
  {
    F32Frag<ND> o;
    f32_load<ND>(o, ctx + out, g, dh);
    D = f32_delta_column<ND>(o, dc, c);
  }
  if (delta && wave == 0 && g == 0 && my_q < s) delta[stat] = D;
  const float L = lse[stat];
  f32x4_t acc[1][ND];
#pragma unroll
  for (int t = 0; t < ND; ++t) acc[0][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const int ntiles = ((causal ? min(q0 + kF32Rows, s) : s) + kF32Rows - 1) / kF32Rows;
  const uint8_t* mrow = (!causal && mask) ? mask + ((size_t)j * s + qr) * s : nullptr;
#pragma unroll 1
  for (int pt = wave; pt < PARTS; pt += NW) {   // the wave's parts
    for (int kt = pt; kt < ntiles; kt += PARTS) {
      const int key0 = kt * kF32Rows;
      const size_t row = (size_t)min(key0 + c, s - 1) * rs;
      F32Frag<ND> k, v;
      f32_load<ND>(k, base + hp + row, g, dh);
      f32_load<ND>(v, base + 2 * hp + row, g, dh);
      const f32x4_t sc = f32_scores<ND>(k, q), dp = f32_scores<ND>(v, dc);
      f32x4_t ds;
      uint32_t vis = 0;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int key = key0 + 4 * g + r;
        const bool ok = key < s && (causal ? key <= my_q : !(mrow && mrow[key]));
        ds[r] = ok ? __expf(sc[r] * scale - L) * (dp[r] - D) * scale : 0.f;
        vis |= (uint32_t)ok << r;
      }
      f32_accumulate<ND>(acc[0], ds, base + hp, rs, key0, s, dh, causal && key0 + kF32Rows > q0, vis, lane);
    }
    if (pt + NW < PARTS) f32_set_aside<ND>(acc[0], part, wave, lane);
  }
  if constexpr (PARTS == 8) f32_join_eight<ND, NW, 1>(acc, part, 1.f, wave, lane);
  else f32_join<ND>(acc[0], part, wave, lane);
  if (wave > 0 || my_q >= s) return;
  f32_store<ND>(dqkv + (size_t)my_q * rs + (size_t)j * 3 * hp + (size_t)e * dh, acc[0], g, dh);
}

// dK, dV of 16 keys.  OWN_DELTA: the queries' delta is computed here as well (ctx), not read (delta).
template <int ND, int NW, int PARTS, bool OWN_DELTA>
__device__ __forceinline__ void f32_dkv_block(const float* __restrict__ qkv, const float* __restrict__ ctx, const float* __restrict__ dctx,
                                              const float* __restrict__ lse, const float* __restrict__ delta, float* __restrict__ dqkv, int s,
                                              int b, int heads, int dh, const uint8_t* __restrict__ mask, int causal, int blk, f32x4_t* part) {
  const int e = blockIdx.y, j = blockIdx.z, wave = threadIdx.x >> 6, lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
  const int k0 = blk * kF32Rows, my_key = k0 + c, kr = min(my_key, s - 1);
  const int hp = heads * dh;
  const size_t rs = (size_t)b * 3 * hp, dors = (size_t)b * hp;
  const float* base = qkv + (size_t)j * 3 * hp + (size_t)e * dh;
  const float* dobase = dctx + (size_t)j * hp + (size_t)e * dh;
  const float scale = rsqrtf((float)dh);
  const float* lse_h = lse + ((size_t)j * heads + e) * s;
  const float* delta_h = delta + ((size_t)j * heads + e) * s;   // (read unless OWN_DELTA)
  const float* cbase = ctx + (size_t)j * hp + (size_t)e * dh;     // (read if OWN_DELTA)
  F32Frag<ND> k, v;
  f32_load<ND>(k, base + hp + (size_t)kr * rs, g, dh);
  f32_load<ND>(v, base + 2 * hp + (size_t)kr * rs, g, dh);
  f32x4_t acc[2][ND];
  f32x4_t (&dk)[ND] = acc[0], (&dv)[ND] = acc[1];
#pragma unroll
  for (int t = 0; t < ND; ++t) dk[t] = dv[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const int ntiles = (s + kF32Rows - 1) / kF32Rows;
#pragma unroll 1
  for (int pt = wave; pt < PARTS; pt += NW) {   // the wave's parts
    for (int qt = (causal ? blk : 0) + pt; qt < ntiles; qt += PARTS) {
      const int q0 = qt * kF32Rows;
      f32x4_t sc, dp, p, ds, own = {0.f, 0.f, 0.f, 0.f};
      {
        F32Frag<ND> q, dc;
        f32_load<ND>(q, base + (size_t)min(q0 + c, s - 1) * rs, g, dh);
        f32_load<ND>(dc, dobase + (size_t)min(q0 + c, s - 1) * dors, g, dh);
        if constexpr (OWN_DELTA) {
          F32Frag<ND> o;
          f32_load<ND>(o, cbase + (size_t)min(q0 + c, s - 1) * dors, g, dh);
          own = f32_delta_rows<ND>(o, dc, g);
        }
        sc = f32_scores<ND>(q, k);
        dp = f32_scores<ND>(dc, v);
      }
      uint32_t vis = 0;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int q = q0 + 4 * g + r, qq = min(q, s - 1);
        const bool ok = q < s && (!causal || q >= my_key);
        const bool hidden = !causal && mask && mask[((size_t)j * s + qq) * s + kr];
        p[r] = ok ? __expf((hidden ? kMaskFill : sc[r] * scale) - lse_h[qq]) : 0.f;
        ds[r] = ok && !hidden ? p[r] * (dp[r] - (OWN_DELTA ? own[r] : delta_h[qq])) * scale : 0.f;
        vis |= (uint32_t)ok << r;
      }
      const bool diag = causal && q0 < k0 + kF32Rows;
      f32_accumulate<ND>(dv, p, dobase, dors, q0, s, dh, diag, vis, lane);
      f32_accumulate<ND>(dk, ds, base, rs, q0, s, dh, diag, vis, lane);
    }
    if (pt + NW < PARTS) {
      f32_set_aside<ND>(dk, part, wave, lane);
      f32_set_aside<ND>(dv, part + 4 * ND * 64, wave, lane);
    }
  }
  float* out = dqkv + (size_t)my_key * rs + (size_t)j * 3 * hp + (size_t)e * dh;
  if constexpr (PARTS == 8) {
    f32_join_eight<ND, NW, 2>(acc, part, 1.f, wave, lane);
    if (my_key >= s) return;
    if (wave == 0) f32_store<ND>(out + hp, dk, g, dh);
    if (wave == 1) f32_store<ND>(out + 2 * hp, dv, g, dh);
  } else {
    const bool mine = f32_join<ND>(dk, part, wave, lane);
    if (mine && my_key < s) f32_store<ND>(out + hp, dk, g, dh);
    if (f32_join<ND>(dv, part, wave, lane) && my_key < s) f32_store<ND>(out + 2 * hp, dv, g, dh);
  }
}

constexpr int f32_dq_waves(int nd, int nw) { return nw == 8 ? 2 : nd == 2 ? 6 : nd == 4 ? 4 : nd == 6 ? 3 : nd == 8 ? 2 : 1; }   // likewise
template <int ND, int NW, int PARTS>
__global__ void __launch_bounds__(64 * NW, f32_dq_waves(ND, NW))
attn_bwd_dq_f32(const float* __restrict__ qkv, const float* __restrict__ ctx, const float* __restrict__ dctx,
                const float* __restrict__ lse, float* __restrict__ delta, float* __restrict__ dqkv, int s, int b, int heads, int dh,
                const uint8_t* __restrict__ mask, int causal) {
  __shared__ f32x4_t part[f32_places(ND, PARTS, 1)];
  // long rows first
  f32_dq_block<ND, NW, PARTS>(qkv, ctx, dctx, lse, delta, dqkv, s, b, heads, dh, mask, causal, (int)gridDim.x - 1 - (int)blockIdx.x, part);
}
template <int ND, int NW, int PARTS>
__global__ void __launch_bounds__(64 * NW)
attn_bwd_dkv_f32(const float* __restrict__ qkv, const float* __restrict__ dctx, const float* __restrict__ lse,
                 const float* __restrict__ delta, float* __restrict__ dqkv, int s, int b, int heads, int dh,
                 const uint8_t* __restrict__ mask, int causal) {
  __shared__ f32x4_t part[f32_places(ND, PARTS, 2)];
  f32_dkv_block<ND, NW, PARTS, false>(qkv, nullptr, dctx, lse, delta, dqkv, s, b, heads, dh, mask, causal, blockIdx.x, part);
}
// Both in one launch: dK/dV computes the delta of its queries itself, so that neither waits for the other.
template <int ND, int NW, int PARTS>
__global__ void __launch_bounds__(64 * NW)
attn_bwd_f32(const float* __restrict__ qkv, const float* __restrict__ ctx, const float* __restrict__ dctx, const float* __restrict__ lse,
             float* __restrict__ dqkv, int s, int b, int heads, int dh, const uint8_t* __restrict__ mask, int causal) {
  __shared__ f32x4_t part[f32_places(ND, PARTS, 2)];
  const int n = (int)gridDim.x / 2, x = (int)blockIdx.x;
  if (x < n) f32_dkv_block<ND, NW, PARTS, true>(qkv, ctx, dctx, lse, nullptr, dqkv, s, b, heads, dh, mask, causal, x, part);
  else f32_dq_block<ND, NW, PARTS>(qkv, ctx, dctx, lse, nullptr, dqkv, s, b, heads, dh, mask, causal, 2 * n - 1 - x, part);
}

// ------------------------------------------------------------------------------------------------
// bf16 MFMA kernels.  A wave owns 32 queries (forward, dQ) or 32 keys (dK/dV); the other side streams through LDS in
// tiles of 32 or 64 rows kept in memory order [row][dh].  Operands whose contraction index is the tile row (V^T, K^T,
// Q^T, dO^T) are gathered from those same tiles with transposing LDS reads, so nothing is transposed in registers
// and every tile is stored once.
// ------------------------------------------------------------------------------------------------
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4_t;

// Registers 8*ks .. 8*ks+7 of a 32x32 accumulator as a bf16 B-operand fragment.
__device__ __forceinline__ bf16x8_t pack_frag(const f32x16_t& a, int ks) {
  uint4 t = make_uint4(pack_bf16x2(a[ks * 8 + 0], a[ks * 8 + 1]), pack_bf16x2(a[ks * 8 + 2], a[ks * 8 + 3]),
                       pack_bf16x2(a[ks * 8 + 4], a[ks * 8 + 5]), pack_bf16x2(a[ks * 8 + 6], a[ks * 8 + 7]));
  return *reinterpret_cast<bf16x8_t*>(&t);
}
__device__ __forceinline__ f32x16_t zero16() {
  f32x16_t z;
#pragma unroll
  for (int r = 0; r < 16; ++r) z[r] = 0.f;
  return z;
}
// lane's 8 consecutive dh (k16 step kk) of one token row, as a B-operand fragment straight from HBM
// (`row` must be readable; `ok` false blanks the fragment)
__device__ __forceinline__ bf16x8_t frag_global(const bf16_t* row, bool ok, int kk, int half) {
  const uint4 r = *reinterpret_cast<const uint4*>(row + kk * 16 + half * 8);
  uint4 t = make_uint4(ok ? r.x : 0u, ok ? r.y : 0u, ok ? r.z : 0u, ok ? r.w : 0u);
  return *reinterpret_cast<bf16x8_t*>(&t);
}
// accumulator rows (dh) of lane's column (token) -> 8-byte stores of 4 consecutive dh
template <int NDT>
__device__ __forceinline__ void store_cols(bf16_t* out_row, const f32x16_t (&acc)[NDT], float mul, int half) {
#pragma unroll
  for (int d = 0; d < NDT; ++d)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      uint2 w;
      w.x = pack_bf16x2(acc[d][4 * g] * mul, acc[d][4 * g + 1] * mul);
      w.y = pack_bf16x2(acc[d][4 * g + 2] * mul, acc[d][4 * g + 3] * mul);
      *reinterpret_cast<uint2*>(out_row + d * 32 + 8 * g + 4 * half) = w;
    }
}

// Hidden flags of keys key .. key+3 of one mask row as the four bytes of a word (keys >= s read as 0).
__device__ __forceinline__ uint32_t mask_word(const uint8_t* __restrict__ mrow, int key, int s, bool aligned) {
  if (aligned && key < s) return *reinterpret_cast<const uint32_t*>(mrow + key);   // s % 4 == 0: key + 3 < s
  uint32_t w = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (key + i < s) w |= (uint32_t)mrow[key + i] << (8 * i);
  return w;
}

// Work assignment.  Workgroups are dealt round-robin to the 8 XCDs, each with its own L2: every block of one
// (sample, head) pair goes to the same XCD so that the pair's K and V stay in that L2, and each XCD
// takes its pairs one after the other - as long as whole rounds of 8 pairs remain.  The last heads * b mod 8 pairs
// are dealt block by block instead (block-major, so that each XCD gets the same share of every block index and
// with it of the causal triangle's work): 20 heads would otherwise leave four XCDs with three pairs and four
// with two.  Returns false for surplus ids.  `blk` counts up within a pair.
__device__ __forceinline__ bool attn_map(int id, int nblk, int heads, int b, int* blk, int* e, int* j) {
  const int xcd = id & 7, local = id >> 3;
  const int pairs = heads * b, whole = pairs >> 3, rest = pairs & 7;
  int pair;
  if (local < whole * nblk) {
    pair = xcd + 8 * (local / nblk);
    *blk = local % nblk;
  } else {
    const int g = (local - whole * nblk) * 8 + xcd;   // index into the remaining pairs' blocks, block-major
    if (g >= rest * nblk) return false;
    pair = 8 * whole + g % rest;
    *blk = g / rest;
  }
  *e = pair % heads;
  *j = pair / heads;
  return true;
}
inline long long attn_grid(long long nblk, int heads, int b) {
  const long long pairs = (long long)heads * b, whole = pairs >> 3, rest = pairs & 7;
  return 8 * (whole * nblk + (rest * nblk + 7) / 8);
}

// The same for the causal kernels on tiles from LDS, whose blocks differ in length: an XCD takes block `blk` of all its pairs
// before block blk + 1 of any, so that the longest walks start first whatever pair they belong to (pair by pair, the last
// pair's longest block starts when most others are done).  Eight block levels at a time; the last heads * b mod 8 pairs
// are dealt block by block.  Fewer than eight blocks: as above.
__device__ __forceinline__ bool attn_map_levels(int id, int nblk, int heads, int b, int* blk, int* e, int* j) {
  if (nblk < 8) return attn_map(id, nblk, heads, b, blk, e, j);
  const int xcd = id & 7, local = id >> 3;
  const int pairs = heads * b, whole = pairs >> 3, rest = pairs & 7;
  const int chunk = local / pairs, r = local % pairs;
  int pair;
  if (r < rest) {
    const int g = (chunk * rest + r) * 8 + xcd;   // index into the remaining pairs' blocks, block-major
    if (g >= rest * nblk) return false;
    pair = 8 * whole + g % rest;
    *blk = g / rest;
  } else {
    *blk = 8 * chunk + (r - rest) / whole;
    if (*blk >= nblk) return false;
    pair = xcd + 8 * ((r - rest) % whole);
  }
  *e = pair % heads;
  *j = pair / heads;
  return true;
}
inline long long attn_grid_levels(long long nblk, int heads, int b) {
  return nblk < 8 ? attn_grid(nblk, heads, b) : (long long)heads * b * (8 * ((nblk + 7) / 8));
}

// ------------------------------------------------------------------------------------------------
// Tiles of 64 rows that travel from memory straight to LDS (buffer_load ... lds), one tile ahead of the arithmetic.
// LDS image: blocks of 32 dh, [block][64 rows][64 bytes]; the 16-byte chunk c of row r sits in slot c ^ ((r >> 2) & 3),
// so that 16 rows of a fragment read and the 8 rows of a transposing read fall into different bank groups.
// ------------------------------------------------------------------------------------------------
typedef uint32_t attn_rsrc_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint32_t attn_lds_offset(const char* p) {
  return (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) void*)p);
}
// lane i's 16 bytes land at lds + 16 i.  Assembly, because the compiler makes every LDS read wait for all such loads in
// flight; s_nop 4: the descriptor may have been written by the vector ALU just before, which the compiler cannot see here.
__device__ __forceinline__ void attn_load_lds(attn_rsrc_t r, uint32_t lds, uint32_t voff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" :: "s"(lds), "v"(voff), "s"(r) : "memory", "m0");
}
// A slice is addressed from its first row with 32-bit byte offsets; they reach the end of its sixteenth row up to this pitch.
constexpr bool attn_slice_fits(uint64_t row_elements, int dh) {
  return row_elements < (1ull << 31) && 15 * row_elements * 2 + 2 * (uint64_t)dh <= 0xffffffffull;
}
typedef uint32_t attn_chunk_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) attn_chunk_t lds_chunk_t;
// A group of W waves loads a tile of KT rows; wave w takes the 16-row slices w, w + W, .. of every block.
// WIDE: any row pitch: 64-bit addresses, through registers, to the same places.
template <int DH, int W, int KT, bool WIDE> struct TileDma {
  static_assert(KT / 16 % W == 0, "every wave takes the same slices of every block");
  static constexpr int NDT = DH / 32, kBytes = KT * DH * 2;
  uint32_t off;   // the lane's chunk inside a slice's first block (WIDE: inside the lane's row)
  uint32_t lane;
  size_t rs;
  __device__ __forceinline__ void init(size_t row_elements, int lane_id) {
    rs = row_elements;
    lane = lane_id;
    off = (WIDE ? 0u : (uint32_t)((lane >> 2) * row_elements * 2)) + (((lane & 3) ^ (lane >> 4)) * 16);
  }
  // rows row0 .. row0 + KT - 1 of a head whose row 0 starts at p; rows from s on are zeros
  __device__ __forceinline__ void issue(const bf16_t* __restrict__ p, int row0, int s, uint32_t lds, int w) const {
    if constexpr (WIDE) {
#pragma unroll
      for (int g = 0; g < KT / 16 / W; ++g) {
        const int slice = w + W * g, row = row0 + 16 * slice + (int)(lane >> 2);
        const bool ok = row < s;
        const char* a = reinterpret_cast<const char*>(p + (size_t)min(row, s - 1) * rs) + off;
        const uint32_t to = lds + slice * 1024 + lane * 16;
#pragma unroll
        for (int d = 0; d < NDT; ++d) {
          attn_chunk_t t = {0u, 0u, 0u, 0u};
          if (ok) t = *reinterpret_cast<const attn_chunk_t*>(a + d * 64);
          *(lds_chunk_t*)(uintptr_t)(to + d * (KT * 64)) = t;
        }
      }
      return;
    }
#pragma unroll
    for (int g = 0; g < KT / 16 / W; ++g) {
      const int slice = w + W * g, first = row0 + 16 * slice, rows = min(s - first, 16);
      const uint64_t a = reinterpret_cast<uint64_t>(p + (size_t)first * rs);
      const attn_rsrc_t r = {(uint32_t)a, (uint32_t)(a >> 32) & 0xffffu, rows > 0 ? (uint32_t)((rows - 1) * rs * 2 + DH * 2) : 0u, 0x00020000u};
#pragma unroll
      for (int d = 0; d < NDT; ++d) attn_load_lds(r, lds + d * (KT * 64) + slice * 1024, off + d * 64);
    }
  }
};
typedef __attribute__((address_space(3))) const bf16x8_t lds_frag_t;
typedef __attribute__((address_space(3))) s16x4_t lds_tr_t;
// fragment with the tile row as the MFMA row: row sub * 32 + (lane & 31), eight dh of k16 step kk
template <int KT> struct FragDirect {
  uint32_t base[2];
  __device__ __forceinline__ void init(uint32_t tile, int l31, int half) {
#pragma unroll
    for (int p = 0; p < 2; ++p) base[p] = tile + l31 * 64 + (((2 * p + half) ^ ((l31 >> 2) & 3)) * 16);
  }
  // moved by a stage: the sum is kept in the base registers, so that everything else is in the instructions' offset fields
  __device__ __forceinline__ FragDirect at(uint32_t stage) const {
    FragDirect f{{base[0] + stage, base[1] + stage}};
    asm volatile("" : "+v"(f.base[0]), "+v"(f.base[1]));
    return f;
  }
  __device__ __forceinline__ bf16x8_t get(int sub, int kk, int tile = 0) const {
    return *(lds_frag_t*)(uintptr_t)(base[kk & 1] + (kk >> 1) * (KT * 64) + sub * 2048 + tile);
  }
};
// fragment with dh as the MFMA row (d * 32 + (lane & 31)) and tile rows as the contraction index, in the order of the 32x32
// accumulator rows that feed the other operand: rows 16 * ks + 4 * half + 0..3 and 16 * ks + 8 + 4 * half + 0..3 of
// 32-row half `sub`.  ds_read_b64_tr_b16: within 16 lanes, lane i receives element (i & 3) of the 8-byte rows addressed by
// lanes (i >> 2) + {0, 4, 8, 12}.
template <int KT> struct FragTr {
  uint32_t lo, hi;
  __device__ __forceinline__ void init(uint32_t tile, int lane) {
    const int r = lane & 15, G = lane >> 4, row = 4 * (G >> 1) + (r >> 2), c = (2 * (G & 1) + ((r & 3) >> 1)) ^ (G >> 1);
    lo = tile + row * 64 + c * 16 + (r & 1) * 8;
    hi = tile + (row + 8) * 64 + (c ^ 2) * 16 + (r & 1) * 8;
  }
  __device__ __forceinline__ FragTr at(uint32_t stage) const {
    FragTr f{lo + stage, hi + stage};
    asm volatile("" : "+v"(f.lo), "+v"(f.hi));
    return f;
  }
  __device__ __forceinline__ bf16x8_t get(int d, int sub, int ks, int tile = 0) const {
    const uint32_t o = d * (KT * 64) + sub * 2048 + ks * 1024 + tile;
    const s16x4_t a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_tr_t*)(uintptr_t)(lo + o));
    const s16x4_t b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_tr_t*)(uintptr_t)(hi + o));
    typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s16x8_t;
    const s16x8_t v = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8_t, v);
  }
};
// every request of this wave has landed, every LDS read has returned, and the same holds for the workgroup's other waves
__device__ __forceinline__ void attn_tiles_ready() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
// order of a scheduling region's MFMAs and LDS reads: the reads of the first kAhead MFMAs, then one MFMA and the reads of one
template <int MFMAS, int READS> __device__ __forceinline__ void sched_reads_ahead() {
  constexpr int kAhead = 4 < MFMAS ? 4 : MFMAS;
  __builtin_amdgcn_sched_group_barrier(0x100, kAhead * READS, 0);
#pragma unroll
  for (int i = 0; i < MFMAS; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, READS, 0);
  }
}
// MFMAs with the reads of one more and a share of VALU vector instructions behind each
template <int MFMAS, int READS, int VALU> __device__ __forceinline__ void sched_mixed() {
#pragma unroll
  for (int i = 0; i < MFMAS; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, READS, 0);
    __builtin_amdgcn_sched_group_barrier(0x402, (VALU + MFMAS - 1) / MFMAS, 0);
  }
}

// A lane's words of one general-mask tile: its query's flags of keys sub * 32 + 8 g + 4 * half .. + 3.  They are requested a
// tile ahead; take() is where the compiler waits for them: behind attn_tiles_ready, when nothing else is in flight, and before
// the next tile's requests.  A tile inside the mask row travels as 16 SUBS consecutive bytes per lane (word by word it took
// four times the address cycles, more than the tile's products: dQ of 4 x 16 heads of 64 x 512 27 us); the two lanes of a row
// then exchange every other word.
template <int SUBS> struct MaskWords {
  uint32_t next[SUBS * 4], now[SUBS][4];
  bool wide;
  __device__ __forceinline__ void load(const uint8_t* __restrict__ mrow, int key0, int s, int half) {
    typedef uint32_t words_t __attribute__((ext_vector_type(4), aligned(4)));
    wide = key0 + 32 * SUBS <= s && (s & 3) == 0;
    if (wide) {
      const words_t* p = reinterpret_cast<const words_t*>(mrow + key0 + half * (16 * SUBS));
#pragma unroll
      for (int i = 0; i < SUBS; ++i) {
        const words_t w = p[i];
#pragma unroll
        for (int k = 0; k < 4; ++k) next[4 * i + k] = w[k];
      }
    } else {
#pragma unroll
      for (int sub = 0; sub < SUBS; ++sub)
#pragma unroll
        for (int g = 0; g < 4; ++g) next[sub * 4 + g] = mask_word(mrow, key0 + sub * 32 + 8 * g + 4 * half, s, (s & 3) == 0);
    }
  }
  __device__ __forceinline__ void take() {
#pragma unroll
    for (int i = 0; i < 4 * SUBS; ++i) asm volatile("" : "+v"(next[i]));
    if (wide) {   // words 2 i, 2 i + 1 of the lower lane's and of the upper lane's bytes: even ones belong below, odd ones above
#pragma unroll
      for (int i = 0; i < 2 * SUBS; ++i) {
        const auto w = __builtin_amdgcn_permlane32_swap(next[2 * i], next[2 * i + 1], false, false);
        if constexpr (SUBS == 2) {
          now[0][i] = w[0];
          now[1][i] = w[1];
        } else {
          now[0][i] = w[0];
          now[0][2 + i] = w[1];
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4 * SUBS; ++i) now[i >> 2][i & 3] = next[i];
    }
  }
  __device__ __forceinline__ bool hidden(int sub, int r) const { return (now[sub][r >> 2] >> (8 * (r & 3))) & 0xffu; }
};
template <bool LEVELS> __device__ __forceinline__ bool attn_map_tiles(int id, int nblk, int heads, int b, int* blk, int* e, int* j) {
  if (!(LEVELS ? attn_map_levels(id, nblk, heads, b, blk, e, j) : attn_map(id, nblk, heads, b, blk, e, j))) return false;
  *blk = __builtin_amdgcn_readfirstlane(*blk);
  *e = __builtin_amdgcn_readfirstlane(*e);
  *j = __builtin_amdgcn_readfirstlane(*j);
  return true;
}

// Forward: S^T = K Q^T and O^T = V^T P^T, so that the probabilities leave the first MFMA in the register layout the second
// one takes as its B operand.  A workgroup owns 32 QW queries, 32 to a wave; K and V stream through two LDS stages of KT
// keys, requested one tile ahead, with one barrier per tile.  What bounds it: at 64 heads of 128 x 2048 the matrix cores are
// busy 35 % of the cycles and the vector ALU issues in 31 % (profiles/c4_kernel_counters.txt); the rest is the two waves of a SIMD
// waiting on each other's phases.  Hence:
//   reads of fragments run four MFMAs ahead of their use (left to the compiler, every MFMA waits for its own read);
//   the second 32 keys' exponentials are spread between the first 32 keys' products;
//   long rows start first over all pairs of an XCD (attn_map_levels): 1.5 waves run on a SIMD on average;
//   the output is rescaled only when some row's running maximum moved, the mask touches only tiles on the diagonal.
// NP = 2: two groups of QW waves take alternate tiles, with stages of their own, and their partial results are merged at the
// end: for launches with too few workgroups to fill the chip.
// us before (tiles through registers, two barriers per tile) and now, causal, s = 2048 unless given: 4 x 16 heads of 128 143 ->
// 87; 12 heads of 128 52 -> 30; 8 heads 39 -> 29, at s = 1024 21.6 -> 16.3; 20 heads of 160 98 -> 54; 32 of 64 54 -> 32; 128
// of 32 104 -> 67; without the mask 16 heads of 128 58 -> 43.
template <int DH, bool CAUSAL, int QW, int NP, int KT, bool WIDE>
__global__ void __launch_bounds__(64 * QW * NP, 2)
attn_fwd_tiles(const bf16_t* __restrict__ qkv, bf16_t* __restrict__ ctx, float* __restrict__ lse, int s, int b, int heads,
               const uint8_t* __restrict__ mask) {
  constexpr int NKK = DH / 16, NDT = DH / 32, kQ = 32 * QW, SUBS = KT / 32;
  constexpr uint32_t kTile = TileDma<DH, QW, KT, WIDE>::kBytes, kStage = 2 * kTile;
  extern __shared__ __attribute__((aligned(1024))) char smem_all[];
  const int wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), grp = NP == 1 ? 0 : wave_all / QW, wave = wave_all % QW;
  const uint32_t lds0 = attn_lds_offset(smem_all) + grp * 2 * kStage;

  const int nqb = (s + kQ - 1) / kQ;
  int qblk, e, j;
  if (!attn_map_tiles<CAUSAL && !WIDE>(blockIdx.x, nqb, heads, b, &qblk, &e, &j)) return;
  qblk = nqb - 1 - qblk;   // long rows first
  const int lane = threadIdx.x & 63, half = lane >> 5, l31 = lane & 31;
  const int hp = heads * DH;
  const size_t rs = (size_t)b * 3 * hp;
  const bf16_t* base = qkv + (size_t)j * 3 * hp + (size_t)e * DH;
  const int q_first = qblk * kQ + wave * 32;
  const int my_q = q_first + l31;
  const float c2 = rsqrtf((float)DH) * 1.4426950408889634f;  // scale * log2(e)

  const int q_last_blk = min(s, (qblk + 1) * kQ) - 1;
  const int ntiles = CAUSAL ? q_last_blk / KT + 1 : (s + KT - 1) / KT;
  TileDma<DH, QW, KT, WIDE> dma;
  dma.init(rs, lane);
  auto request = [&](int kt, uint32_t stage) {
    dma.issue(base + hp, kt * KT, s, lds0 + stage, wave);
    dma.issue(base + 2 * hp, kt * KT, s, lds0 + stage + kTile, wave);
  };
  request(grp, 0);

  bf16x8_t qf[NKK];
#pragma unroll
  for (int kk = 0; kk < NKK; ++kk) qf[kk] = frag_global(base + (size_t)min(my_q, s - 1) * rs, my_q < s, kk, half);
  FragDirect<KT> fk;
  FragTr<KT> fv;
  fk.init(lds0, l31, half);
  fv.init(lds0 + kTile, lane);
  f32x16_t o[NDT];
#pragma unroll
  for (int d = 0; d < NDT; ++d) o[d] = zero16();
  float m_run = -INFINITY, l_run = 0.f;
  const bool use_mask = !CAUSAL && mask != nullptr;
  const uint8_t* mrow = mask + ((size_t)j * s + min(my_q, s - 1)) * s;   // (read if use_mask)
  const float fill = kMaskFill * sqrtf((float)DH);   // times 1/sqrt(dh) gives the fill value
  MaskWords<SUBS> mw;
  if (use_mask) mw.load(mrow, grp * KT, s, half);

  uint32_t stage = 0;
  // all groups take the same number of steps (the barriers are the workgroup's); a group without a tile idles
  for (int kt0 = 0; kt0 < ntiles; kt0 += NP, stage ^= kStage) {
    const int kt = kt0 + grp, key0 = kt * KT;
    attn_tiles_ready();
    if (use_mask) mw.take();
    if (kt0 + NP < ntiles) {
      if (use_mask) mw.load(mrow, key0 + NP * KT, s, half);
      request(kt + NP, stage ^ kStage);
    }
    // (no query of the wave exists, or every key of the tile is in its future)
    if (kt >= ntiles || q_first >= s || (CAUSAL && key0 > q_first + 31)) continue;

    f32x16_t sacc[SUBS];
#pragma unroll
    for (int sub = 0; sub < SUBS; ++sub) sacc[sub] = zero16();
    const FragDirect<KT> fks = fk.at(stage);
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk)
#pragma unroll
      for (int sub = 0; sub < SUBS; ++sub) sacc[sub] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fks.get(sub, kk), qf[kk], sacc[sub], 0, 0, 0);
    sched_reads_ahead<SUBS * NKK, 1>();
    if (CAUSAL) {
      // causal mask (also hides keys >= s, which are > every valid query); only tiles on the diagonal need it
      if (key0 + KT - 1 > q_first) {
        const int seen = my_q - key0 - 4 * half;   // local keys above it are hidden
#pragma unroll
        for (int sub = 0; sub < SUBS; ++sub)
#pragma unroll
          for (int r = 0; r < 16; ++r) sacc[sub][r] = sub * 32 + 8 * (r >> 2) + (r & 3) > seen ? -INFINITY : sacc[sub][r];
      }
    } else {
      if (use_mask) {
#pragma unroll
        for (int sub = 0; sub < SUBS; ++sub)
#pragma unroll
          for (int r = 0; r < 16; ++r) sacc[sub][r] = mw.hidden(sub, r) ? fill : sacc[sub][r];
      }
      if (key0 + KT > s) {   // keys past the end of the sequence do not exist
#pragma unroll
        for (int sub = 0; sub < SUBS; ++sub)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int key = key0 + sub * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
            sacc[sub][r] = key >= s ? -INFINITY : sacc[sub][r];
          }
      }
    }
    float mx = m_run;
#pragma unroll
    for (int sub = 0; sub < SUBS; ++sub)
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sacc[sub][r]);
    const LaneHalves mh = lane_halves(mx);
    mx = fmaxf(mh.lo, mh.hi);
    if (__any(mx > m_run)) {   // some row's maximum moved: rescale what has been accumulated
      const float corr = __builtin_amdgcn_exp2f((m_run - mx) * c2);
      m_run = mx;
      l_run *= corr;
#pragma unroll
      for (int d = 0; d < NDT; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[d][r] *= corr;
    }
    const float mc = mx * c2;
    bf16x8_t pf[SUBS][2], vr[2][NDT];
    auto weights = [&](int sub) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        sacc[sub][r] = __builtin_amdgcn_exp2f(sacc[sub][r] * c2 - mc);
        l_run += sacc[sub][r];
      }
      pf[sub][0] = pack_frag(sacc[sub], 0);
      pf[sub][1] = pack_frag(sacc[sub], 1);
    };
    const FragTr<KT> fvs = fv.at(stage);
    auto read_v = [&](int u) {
#pragma unroll
      for (int d = 0; d < NDT; ++d) vr[u & 1][d] = fvs.get(d, u >> 1, u & 1);
    };
    auto multiply = [&](int u) {
#pragma unroll
      for (int d = 0; d < NDT; ++d) o[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vr[u & 1][d], pf[u >> 1][u & 1], o[d], 0, 0, 0);
    };
    read_v(0);
    weights(0);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (SUBS == 2) {   // the second half's exponentials between the first half's products
      read_v(1);
      multiply(0);
      read_v(2);
      multiply(1);
      weights(1);
      sched_mixed<2 * NDT, 2, 56>();
      __builtin_amdgcn_sched_barrier(0);
    }
    read_v(2 * SUBS - 1);
    multiply(2 * SUBS - 2);
    multiply(2 * SUBS - 1);
    __builtin_amdgcn_sched_barrier(0);
  }
  l_run += __shfl_xor(l_run, 32, 64);
  if constexpr (NP > 1) {
    // the other groups' partial results join group 0's in order: value v of lane l of wave w at part[w][v][l]
    float* part = reinterpret_cast<float*>(smem_all) + wave * ((2 + NDT * 16) * 64) + lane;
#pragma unroll 1
    for (int from = 1; from < NP; ++from) {
      __syncthreads();   // every wave is done with the tiles, the last partial result has been read
      if (grp == from) {
        part[0] = m_run;
        part[64] = l_run;
#pragma unroll
        for (int d = 0; d < NDT; ++d)
#pragma unroll
          for (int r = 0; r < 16; ++r) part[(2 + d * 16 + r) * 64] = o[d][r];
      }
      __syncthreads();
      if (grp == 0) {
        const float m1 = part[0], l1 = part[64];
        const float m = fmaxf(m_run, m1);   // group 0 always has tile 0, whose key 0 every query sees: m_run is finite
        const float a0 = __builtin_amdgcn_exp2f((m_run - m) * c2), a1 = __builtin_amdgcn_exp2f((m1 - m) * c2);
        l_run = l_run * a0 + l1 * a1;
        m_run = m;
#pragma unroll
        for (int d = 0; d < NDT; ++d)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[d][r] = o[d][r] * a0 + part[(2 + d * 16 + r) * 64] * a1;
      }
    }
    if (grp > 0) return;
  }
  if (my_q < s) {
    store_cols<NDT>(ctx + ((size_t)my_q * b + j) * hp + (size_t)e * DH, o, 1.f / l_run, half);
    if (half == 0) lse[((size_t)j * heads + e) * s + my_q] = m_run * rsqrtf((float)DH) + __logf(l_run);
  }
}

// ------------------------------------------------------------------------------------------------
// bf16 MFMA backward.  P is recomputed from the stashed log-sum-exp; two kernels so that no result
// needs atomics: one owns 64 queries and produces dQ, one owns 64 keys and produces dK and dV.
//   dP = dO V^T, dS = P o (dP - delta), dQ = dS K / sqrt(dh), dK = dS^T Q / sqrt(dh), dV = P^T dO
// ------------------------------------------------------------------------------------------------
// delta = sum_d dctx * ctx of 32 rows, one to a lane and its neighbour 32 lanes on: the diagonal of ctx dctx^T, summed in the order of dP
// in the kernels below (with one visible key dP - D is exactly zero).  `row`: the lane's row of ctx, readable.
template <int DH>
__device__ __forceinline__ float attn_delta_of(const bf16_t* __restrict__ row, const bf16x8_t (&dof)[DH / 16], bool valid, int lane) {
  const int half = lane >> 5, l31 = lane & 31;
  f32x16_t x = zero16();
#pragma unroll
  for (int kk = 0; kk < DH / 16; ++kk) x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_global(row, valid, kk, half), dof[kk], x, 0, 0, 0);
  // row l31 of column l31: register (l31 & 3) + 4 * (l31 >> 3) of the lane of half (l31 >> 2) & 1
  float mine = x[0];
#pragma unroll
  for (int r = 1; r < 16; ++r) mine = (l31 & 3) + 4 * (l31 >> 3) == r ? x[r] : mine;
  return __shfl(mine, ((l31 >> 2) & 1) * 32 + l31, 64);
}

// dQ of 32 QW queries, as the forward kernel walks them: K and V stream through two LDS stages of KT keys (K is read twice,
// as rows for S and transposed for dQ).  NP groups (1, 2 or 4) take tiles in turn and their sums are added at the end.  A wave
// holds Q, dO and dQ and fits two to a SIMD (tiles on their way through registers had left one), so that one's
// exponentials run under the other's products.  Error against 64 bits unchanged.
// us before and now, causal, s = 2048 unless given: 4 x 16 heads of 128 216 -> 106; 12 heads of 128 61 -> 38; 8 heads 48 -> 34, at
// s = 1024 27 -> 20; 20 heads of 160 121 -> 56; 32 of 64 62 -> 36; 128 of 32 112 -> 76; 16 of 128 without the mask 147 -> 61; 4 x 16
// heads of 64 x 512 under a general mask 23 -> 16.
// READ: delta comes from memory.
template <int DH, bool CAUSAL, int QW, int NP, int KT, bool WIDE, bool READ>
__device__ __forceinline__ void attn_dq_block(const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ ctx, const bf16_t* __restrict__ dctx,
                                              const float* __restrict__ lse, float* __restrict__ delta, bf16_t* __restrict__ dqkv, int s, int b,
                                              int heads, const uint8_t* __restrict__ mask, int id, char* smem_all) {
  constexpr int NKK = DH / 16, NDT = DH / 32, kQ = 32 * QW, SUBS = KT / 32;
  constexpr uint32_t kTile = TileDma<DH, QW, KT, WIDE>::kBytes, kStage = 2 * kTile;
  const int wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), grp = NP == 1 ? 0 : wave_all / QW, wave = wave_all % QW;
  const uint32_t lds0 = attn_lds_offset(smem_all) + grp * 2 * kStage;

  const int nqb = (s + kQ - 1) / kQ;
  int qblk, e, j;
  if (!attn_map_tiles<CAUSAL && !WIDE>(id, nqb, heads, b, &qblk, &e, &j)) return;
  qblk = nqb - 1 - qblk;   // long rows first
  const int lane = threadIdx.x & 63, half = lane >> 5, l31 = lane & 31;
  const int hp = heads * DH;
  const size_t rs = (size_t)b * 3 * hp;
  const bf16_t* base = qkv + (size_t)j * 3 * hp + (size_t)e * DH;
  const int q_first = qblk * kQ + wave * 32;
  const int my_q = q_first + l31;
  const bool valid = my_q < s;
  const float scale = rsqrtf((float)DH), c2 = scale * 1.4426950408889634f;
  const size_t stat = ((size_t)j * heads + e) * s + my_q;

  const int q_last_blk = min(s, (qblk + 1) * kQ) - 1;
  const int ntiles = CAUSAL ? q_last_blk / KT + 1 : (s + KT - 1) / KT;
  TileDma<DH, QW, KT, WIDE> dma;
  dma.init(rs, lane);
  auto request = [&](int kt, uint32_t stage) {
    dma.issue(base + hp, kt * KT, s, lds0 + stage, wave);
    dma.issue(base + 2 * hp, kt * KT, s, lds0 + stage + kTile, wave);
  };
  request(grp, 0);

  const float L2 = valid ? lse[stat] * 1.4426950408889634f : 0.f;
  bf16x8_t qf[NKK], dof[NKK];
  const size_t out_row = ((size_t)min(my_q, s - 1) * b + j) * hp + (size_t)e * DH;
#pragma unroll
  for (int kk = 0; kk < NKK; ++kk) {
    qf[kk] = frag_global(base + (size_t)min(my_q, s - 1) * rs, valid, kk, half);
    dof[kk] = frag_global(dctx + out_row, valid, kk, half);
  }
  float D;
  if constexpr (READ) {
    D = valid ? delta[stat] : 0.f;
  } else {
    D = attn_delta_of<DH>(ctx + out_row, dof, valid, lane);
    if (grp == 0 && half == 0 && valid) delta[stat] = D;
  }
  FragDirect<KT> fk, fv;
  FragTr<KT> ft;
  fk.init(lds0, l31, half);
  fv.init(lds0 + kTile, l31, half);
  ft.init(lds0, lane);
  f32x16_t acc[NDT];
#pragma unroll
  for (int d = 0; d < NDT; ++d) acc[d] = zero16();
  const bool use_mask = !CAUSAL && mask != nullptr;
  const uint8_t* mrow = mask + ((size_t)j * s + min(my_q, s - 1)) * s;   // (read if use_mask)
  MaskWords<SUBS> mw;
  if (use_mask) mw.load(mrow, grp * KT, s, half);

  uint32_t stage = 0;
  // all groups take the same number of steps (the barriers are the workgroup's); a group without a tile idles
  for (int kt0 = 0; kt0 < ntiles; kt0 += NP, stage ^= kStage) {
    const int kt = kt0 + grp, key0 = kt * KT;
    attn_tiles_ready();
    if (use_mask) mw.take();
    if (kt0 + NP < ntiles) {
      if (use_mask) mw.load(mrow, key0 + NP * KT, s, half);
      request(kt + NP, stage ^ kStage);
    }
    // (no query of the wave exists, or every key of the tile is in its future)
    if (kt >= ntiles || q_first >= s || (CAUSAL && key0 > q_first + 31)) continue;

    const FragDirect<KT> fks = fk.at(stage), fvs = fv.at(stage);
    const FragTr<KT> fts = ft.at(stage);
    // some score of the tile is hidden (under the causal mask only in tiles on the diagonal)
    const bool hide = CAUSAL ? key0 + KT - 1 > q_first : use_mask || key0 + KT > s;
#pragma unroll
    for (int sub = 0; sub < SUBS; ++sub) {
      f32x16_t sacc = zero16(), dp = zero16();
#pragma unroll
      for (int kk = 0; kk < NKK; ++kk) {
        sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fks.get(sub, kk), qf[kk], sacc, 0, 0, 0);
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fvs.get(sub, kk), dof[kk], dp, 0, 0, 0);
      }
      sched_reads_ahead<2 * NKK, 1>();
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = 0; r < 16; ++r) sacc[r] = __builtin_amdgcn_exp2f(sacc[r] * c2 - L2) * (dp[r] - D);
      if (hide) {
        // without the causal mask a hidden score is the constant fill: its probability counts (through D) but it passes no
        // gradient; keys past the end do not exist (an empty row's lse is so low that their exp2 would overflow)
        if (CAUSAL || key0 + KT > s) {
          const int seen = (CAUSAL ? my_q : s - 1) - key0 - sub * 32 - 4 * half;   // local keys above it are hidden
#pragma unroll
          for (int r = 0; r < 16; ++r) sacc[r] = 8 * (r >> 2) + (r & 3) > seen ? 0.f : sacc[r];
        }
        if (use_mask) {
#pragma unroll
          for (int r = 0; r < 16; ++r) sacc[r] = mw.hidden(sub, r) ? 0.f : sacc[r];
        }
      }
      const bf16x8_t dsf[2] = {pack_frag(sacc, 0), pack_frag(sacc, 1)};
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int d = 0; d < NDT; ++d) acc[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fts.get(d, sub, ks), dsf[ks], acc[d], 0, 0, 0);
      sched_reads_ahead<2 * NDT, 2>();
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  if constexpr (NP > 1) {
    // the other groups' sums join group 0's in order: register r of lane l of wave w at sum[w][r][l]
    float* sum = reinterpret_cast<float*>(smem_all) + wave * (NDT * 16 * 64) + lane;
#pragma unroll 1
    for (int from = 1; from < NP; ++from) {
      __syncthreads();   // every wave is done with the tiles, the last sums have been read
      if (grp == from) {
#pragma unroll
        for (int d = 0; d < NDT; ++d)
#pragma unroll
          for (int r = 0; r < 16; ++r) sum[(d * 16 + r) * 64] = acc[d][r];
      }
      __syncthreads();
      if (grp == 0) {
#pragma unroll
        for (int d = 0; d < NDT; ++d)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[d][r] += sum[(d * 16 + r) * 64];
      }
    }
    if (grp > 0) return;
  }
  if (valid) store_cols<NDT>(dqkv + (size_t)my_q * rs + (size_t)j * 3 * hp + (size_t)e * DH, acc, scale, half);
}
// (it also writes delta, which the dK/dV kernel, launched next, reads: in a launch of its own that took 8 to 61 us)
template <int DH, bool CAUSAL, int QW, int NP, int KT, bool WIDE>
__global__ void __launch_bounds__(64 * QW * NP, 2)
attn_bwd_dq_tiles(const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ ctx, const bf16_t* __restrict__ dctx,
                  const float* __restrict__ lse, float* __restrict__ delta, bf16_t* __restrict__ dqkv, int s, int b, int heads,
                  const uint8_t* __restrict__ mask) {
  extern __shared__ __attribute__((aligned(1024))) char smem_all[];
  attn_dq_block<DH, CAUSAL, QW, NP, KT, WIDE, false>(qkv, ctx, dctx, lse, delta, dqkv, s, b, heads, mask, blockIdx.x, smem_all);
}

// The hidden flags of a tile of KEYS keys x QT queries on their way to LDS as one bit each, [key][query]: a lane reads the bits of
// its key at once.  A thread turns 8 queries x 4 keys: eight words of four keys, whose nonzero bytes' flags are shifted
// into one byte per key.
template <int THREADS, int KEYS, int QT> struct MaskBits {
  static constexpr int kRow = QT / 8, kBytes = KEYS * kRow, NB = (KEYS / 4) * kRow;   // NB: blocks, at most one per thread
  static_assert(NB <= THREADS);
  uint32_t v[8];
  __device__ __forceinline__ void load(const uint8_t* __restrict__ mask_j, int q0, int key0, int s, bool aligned, int tid) {
    if (tid >= NB) return;
    const int key = key0 + 4 * (tid % (KEYS / 4)), q = q0 + 8 * (tid / (KEYS / 4));
#pragma unroll
    for (int r = 0; r < 8; ++r) v[r] = mask_word(mask_j + (size_t)min(q + r, s - 1) * s, key, s, aligned);
  }
  __device__ __forceinline__ void store(char* lds, int tid) const {
    if (tid >= NB) return;
    uint32_t bits = 0;
#pragma unroll
    for (int r = 0; r < 8; ++r) bits = (bits >> 1) | ((((v[r] & 0x7f7f7f7fu) + 0x7f7f7f7fu) | v[r]) & 0x80808080u);
    const int key = 4 * (tid % (KEYS / 4)), q8 = tid / (KEYS / 4);
#pragma unroll
    for (int k = 0; k < 4; ++k) lds[(key + k) * kRow + q8] = (char)(bits >> (8 * k));
  }
};

// dK, dV of 32 KW keys; Q and dO stream through two LDS stages of QT queries, requested one tile ahead, with one barrier per tile,
// and are read twice each: as rows for S = Q K^T and dP = dO V^T, transposed for dK and dV.  The queries' lse and delta (and the
// general mask) travel in registers and are written to the next stage behind the arithmetic.
// SPLIT: KW waves compute S, dP and dK and KW waves S and dV: S twice is a quarter more matrix work, but both results of heads of
// 160 do not fit the 256 registers that leave two waves on a SIMD (50 to 90 spilled), and short walks are cut once more.
// What bounds it: every product reads its own fragment from LDS, which at full rate takes as long as the products, and
// the two waves of a SIMD wait on each other's phases: 35 % of the matrix rate at 64 heads of 128 x 2048 (the same file).
// Heads of 128 with both results in a wave spill: without the causal mask 32 registers (92 bytes of scratch a lane) in (4, 1, 64) and
// 20 in tiles of 32, with it up to 3.  Where the launcher takes them they are still the faster forms (its table).
// us for this kernel before (tiles through registers, two barriers per tile, one wave per SIMD where both results were in
// one wave) and now, causal, s = 2048: 4 x 16 heads of 128 316 -> 157, 12 heads 83 -> 54, 20 heads of 160 219 -> 96, 128 of 32 180 -> 101;
// 16 heads of 64 x 333 11.2 -> 9.9; 4 x 16 heads of 64 x 512 under a general mask 36 -> 23.
template <int DH, bool CAUSAL, int KW, int NP, int QT, bool SPLIT> struct DkvGeom {
  static constexpr int kWaves = SPLIT ? 2 * KW : KW, kThreads = 64 * kWaves;   // of a group
  static constexpr int kTile = QT * DH * 2, kStats = 2 * kTile, kMask = kStats + 2 * QT * (int)sizeof(float);
  static constexpr int stage_bytes(bool masked) {   // kept a multiple of 128 bytes
    return ((masked ? kMask + MaskBits<kThreads, 32 * KW, QT>::kBytes : kMask) + 127) / 128 * 128;
  }
  static constexpr int kSums = NP > 1 ? KW * 2 * (DH / 2) * 64 * (int)sizeof(float) : 0;
  static constexpr int lds_bytes(bool masked) { return NP * 2 * stage_bytes(masked) > kSums ? NP * 2 * stage_bytes(masked) : kSums; }
};
template <int DH, bool CAUSAL, int KW, int NP, int QT, bool SPLIT, bool WIDE>
__device__ __forceinline__ void attn_dkv_block(const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ dctx, const float* __restrict__ lse,
                                               const float* __restrict__ delta, bf16_t* __restrict__ dqkv, int s, int b, int heads,
                                               const uint8_t* __restrict__ mask, int id, char* smem_all) {
  using Geom = DkvGeom<DH, CAUSAL, KW, NP, QT, SPLIT>;
  constexpr int NKK = DH / 16, NDT = DH / 32, kKeys = 32 * KW, SUBS = QT / 32, GW = Geom::kWaves, kTile = Geom::kTile;
  constexpr int NR = SPLIT ? 1 : 2;   // results of a wave
  const bool use_mask = !CAUSAL && mask != nullptr;
  const uint32_t stage_bytes = Geom::stage_bytes(!CAUSAL && use_mask);
  const int wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), grp = NP == 1 ? 0 : wave_all / GW, wave = wave_all % GW;
  const int kw = wave % KW, tid = threadIdx.x & (Geom::kThreads - 1);
  static_assert((Geom::kThreads & (Geom::kThreads - 1)) == 0 && QT <= Geom::kThreads);
  char* smem = smem_all + grp * 2 * stage_bytes;
  const uint32_t lds0 = attn_lds_offset(smem);

  const int nkb = (s + kKeys - 1) / kKeys;
  int kblk, e, j;   // the first key blocks see the most queries and start first
  if (!attn_map_tiles<CAUSAL && !WIDE>(id, nkb, heads, b, &kblk, &e, &j)) return;
  static_assert(!SPLIT || KW == 2);
  // which half of a group takes dK alternates, so that every SIMD gets both
  const bool want_dk = !SPLIT || ((wave / KW) ^ (NP == 2 ? grp : id >> 8)) & 1;
  const int lane = threadIdx.x & 63, half = lane >> 5, l31 = lane & 31;
  const int hp = heads * DH;
  const size_t rs = (size_t)b * 3 * hp, dors = (size_t)b * hp;
  const bf16_t* base = qkv + (size_t)j * 3 * hp + (size_t)e * DH;
  const bf16_t* dobase = dctx + (size_t)j * hp + (size_t)e * DH;
  const int key_first = kblk * kKeys + kw * 32;
  const int my_key = key_first + l31;
  const bool valid = my_key < s;
  const float scale = rsqrtf((float)DH), c2 = scale * 1.4426950408889634f;
  const float fill = kMaskFill * sqrtf((float)DH);
  const float* lse_h = lse + ((size_t)j * heads + e) * s;
  const float* delta_h = delta + ((size_t)j * heads + e) * s;
  const uint8_t* mask_j = mask + (size_t)j * s * s;   // (read if use_mask)
  const bool aligned = (s & 3) == 0;

  // every wave loads a share of both tiles, or one half of the waves Q and the other dO
  constexpr int kSlices = QT / 16, DW = GW > kSlices ? kSlices : GW;
  static_assert(GW <= 2 * kSlices);
  TileDma<DH, DW, QT, WIDE> dma_q, dma_do;
  dma_q.init(rs, lane);
  dma_do.init(dors, lane);
  auto request = [&](int qt, uint32_t at) {
    if (GW == DW || wave < DW) dma_q.issue(base, qt * QT, s, lds0 + at, wave % DW);
    if (GW == DW || wave >= DW) dma_do.issue(dobase, qt * QT, s, lds0 + at + kTile, wave % DW);
  };
  float lse_r = 0.f, delta_r = 0.f;
  MaskBits<Geom::kThreads, kKeys, QT> mb;
  auto fetch = [&](int qt) {
    const int q = qt * QT + tid;
    if (tid < QT) {
      lse_r = q < s ? lse_h[q] * 1.4426950408889634f : INFINITY;   // p is zero past the end
      delta_r = q < s ? delta_h[q] : 0.f;
    }
    if (use_mask) mb.load(mask_j, qt * QT, kblk * kKeys, s, aligned, tid);
  };
  auto put = [&](uint32_t at) {
    if (tid < QT) {
      float* st = reinterpret_cast<float*>(smem + at + Geom::kStats);
      st[tid] = lse_r;
      st[QT + tid] = delta_r;
    }
    if (use_mask) mb.store(smem + at + Geom::kMask, tid);
  };
  const int nqt = (s + QT - 1) / QT, qt_first = CAUSAL ? kblk * kKeys / QT : 0;
  if (qt_first + grp < nqt) {
    request(qt_first + grp, 0);
    fetch(qt_first + grp);
    put(0);
  }
  bf16x8_t kf[NKK], vf[NKK];
#pragma unroll
  for (int kk = 0; kk < NKK; ++kk) {
    kf[kk] = frag_global(base + (size_t)min(my_key, s - 1) * rs + hp, valid, kk, half);
    vf[kk] = frag_global(base + (size_t)min(my_key, s - 1) * rs + 2 * hp, valid, kk, half);
  }
  FragDirect<QT> f0;
  FragTr<QT> t0;
  f0.init(lds0, l31, half);
  t0.init(lds0, lane);
  f32x16_t acc[NR][NDT];   // dV and dK, or one of them
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int d = 0; d < NDT; ++d) acc[r][d] = zero16();

  uint32_t stage = 0;
  // all groups take the same number of steps (the barriers are the workgroup's); a group without a tile idles
  for (int qt0 = qt_first; qt0 < nqt; qt0 += NP, stage ^= stage_bytes) {
    const int qt = qt0 + grp, q0 = qt * QT;
    attn_tiles_ready();
    const bool more = qt + NP < nqt;
    if (more) {
      fetch(qt + NP);
      request(qt + NP, stage ^ stage_bytes);
    }
    // (skipped if no key of the wave exists, or every query of the tile precedes its keys)
    if (qt < nqt && key_first < s && !(CAUSAL && q0 + QT - 1 < key_first)) {
      const FragDirect<QT> fs = f0.at(stage);
      const FragTr<QT> ts = t0.at(stage);
      const char* stats = smem + stage + Geom::kStats;
      const bool diag = CAUSAL && q0 < key_first + 31;   // some query of the tile precedes some key of this wave
#pragma unroll
      for (int sub = 0; sub < SUBS; ++sub) {
        f32x16_t sacc = zero16(), dp = zero16();
        if (!SPLIT || want_dk) {
#pragma unroll
          for (int kk = 0; kk < NKK; ++kk) {
            sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fs.get(sub, kk), kf[kk], sacc, 0, 0, 0);
            dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fs.get(sub, kk, kTile), vf[kk], dp, 0, 0, 0);
          }
          sched_reads_ahead<2 * NKK, 1>();
        } else {
#pragma unroll
          for (int kk = 0; kk < NKK; ++kk) sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fs.get(sub, kk), kf[kk], sacc, 0, 0, 0);
          sched_reads_ahead<NKK, 1>();
        }
        __builtin_amdgcn_sched_barrier(0);
        // hidden scores in branches of their own: few tiles have any, and selects in every tile were a third of the vector instructions
        uint32_t mw = 0;   // bit 8 g + i: query 8 g + 4 half + i of this half of the tile is hidden from my_key
        if (use_mask) {
          mw = *reinterpret_cast<const uint32_t*>(smem + stage + Geom::kMask + (kw * 32 + l31) * (QT / 8) + sub * 4) >> (4 * half);
#pragma unroll
          for (int r = 0; r < 16; ++r) sacc[r] = (mw >> (8 * (r >> 2) + (r & 3))) & 1u ? fill : sacc[r];
        }
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int ql = sub * 32 + 8 * g + 4 * half;   // local index of the first of 4 consecutive queries
          const f32x4_t Ls = *reinterpret_cast<const f32x4_t*>(stats + ql * 4), Ds = *reinterpret_cast<const f32x4_t*>(stats + (QT + ql) * 4);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int r = 4 * g + i;
            const float p = __builtin_amdgcn_exp2f(sacc[r] * c2 - Ls[i]);
            sacc[r] = p;
            dp[r] = p * (dp[r] - Ds[i]);
          }
        }
        if (use_mask) {   // no gradient through a hidden score
#pragma unroll
          for (int r = 0; r < 16; ++r) dp[r] = (mw >> (8 * (r >> 2) + (r & 3))) & 1u ? 0.f : dp[r];
        }
        if (diag) {
          const int before = my_key - q0 - sub * 32 - 4 * half;   // local queries below it precede my_key
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const bool gone = 8 * (r >> 2) + (r & 3) < before;
            sacc[r] = gone ? 0.f : sacc[r];
            dp[r] = gone ? 0.f : dp[r];
          }
        }
        const bf16x8_t pf[2] = {pack_frag(sacc, 0), pack_frag(sacc, 1)}, dsf[2] = {pack_frag(dp, 0), pack_frag(dp, 1)};
        if constexpr (SPLIT) {
          // Q^T or dO^T; P or dS
          const uint32_t tile = want_dk ? 0 : kTile;
          const FragTr<QT> tw{ts.lo + tile, ts.hi + tile};
#pragma unroll
          for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int d = 0; d < NDT; ++d) acc[0][d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tw.get(d, sub, ks), want_dk ? dsf[ks] : pf[ks], acc[0][d], 0, 0, 0);
          sched_reads_ahead<2 * NDT, 2>();
        } else {
#pragma unroll
          for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int d = 0; d < NDT; ++d) {
              acc[0][d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ts.get(d, sub, ks, kTile), pf[ks], acc[0][d], 0, 0, 0);
              acc[1][d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ts.get(d, sub, ks), dsf[ks], acc[1][d], 0, 0, 0);
            }
          sched_reads_ahead<4 * NDT, 2>();
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (more) put(stage ^ stage_bytes);
  }
  if constexpr (NP > 1) {
    // the second group's sums join the first's: register r of lane l of the wave with keys kw (and one result) at sum[..][r][l]
    float* sum = reinterpret_cast<float*>(smem_all) + (SPLIT ? (want_dk ? KW : 0) + kw : 2 * kw) * (NDT * 16 * 64) + lane;
    __syncthreads();   // every wave is done with the tiles
    if (grp == 1) {
#pragma unroll
      for (int x = 0; x < NR; ++x)
#pragma unroll
        for (int d = 0; d < NDT; ++d)
#pragma unroll
          for (int r = 0; r < 16; ++r) sum[((x * NDT + d) * 16 + r) * 64] = acc[x][d][r];
    }
    __syncthreads();
    if (grp == 1) return;
#pragma unroll
    for (int x = 0; x < NR; ++x)
#pragma unroll
      for (int d = 0; d < NDT; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[x][d][r] += sum[((x * NDT + d) * 16 + r) * 64];
  }
  if (valid) {
    bf16_t* out = dqkv + (size_t)my_key * rs + (size_t)j * 3 * hp + (size_t)e * DH;
    if constexpr (SPLIT) {
      store_cols<NDT>(out + (want_dk ? hp : 2 * hp), acc[0], want_dk ? scale : 1.f, half);
    } else {
      store_cols<NDT>(out + 2 * hp, acc[0], 1.f, half);
      store_cols<NDT>(out + hp, acc[1], scale, half);
    }
  }
}
// Causal heads of 64 in tiles of 32: 168 registers instead of 171 (three spilled) leave three waves on a SIMD (whole backward of 32 heads x 2048 98 ->
// 89 us, 24 heads 75, 76, 60 x 777 40.5, 38.8; in tiles of 64 30 heads x 4 x 777 83 -> 86, and without the causal mask it spills).
template <int DH, bool CAUSAL, int KW, int NP, int QT, bool SPLIT, bool WIDE>
__global__ void __launch_bounds__(64 * KW * (SPLIT ? 2 : 1) * NP, WIDE ? 1 : CAUSAL && DH == 64 && QT == 32 ? 3 : 2)
attn_bwd_dkv_tiles(const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ dctx, const float* __restrict__ lse,
                   const float* __restrict__ delta, bf16_t* __restrict__ dqkv, int s, int b, int heads,
                   const uint8_t* __restrict__ mask) {
  extern __shared__ __attribute__((aligned(1024))) char smem_all[];
  attn_dkv_block<DH, CAUSAL, KW, NP, QT, SPLIT, WIDE>(qkv, dctx, lse, delta, dqkv, s, b, heads, mask, blockIdx.x, smem_all);
}

// delta in a launch of its own, in front of dQ and dK/dV side by side (3 us where those are: few workgroups)
template <int DH>
__global__ void __launch_bounds__(256)
attn_delta_kernel(const bf16_t* __restrict__ ctx, const bf16_t* __restrict__ dctx, float* __restrict__ delta, int s, int b, int heads) {
  const int lane = threadIdx.x & 63, half = lane >> 5, l31 = lane & 31, nblk = (s + 31) / 32;
  const int unit = blockIdx.x * 4 + (threadIdx.x >> 6);   // 32 rows of a (sample, head)
  if (unit >= nblk * heads * b) return;
  const int blk = unit % nblk, pair = unit / nblk, e = pair % heads, j = pair / heads, row = blk * 32 + l31;
  const bool valid = row < s;
  const size_t at = ((size_t)min(row, s - 1) * b + j) * heads * DH + (size_t)e * DH;
  bf16x8_t dof[DH / 16];
#pragma unroll
  for (int kk = 0; kk < DH / 16; ++kk) dof[kk] = frag_global(dctx + at, valid, kk, half);
  const float D = attn_delta_of<DH>(ctx + at, dof, valid, lane);
  if (half == 0 && valid) delta[((size_t)j * heads + e) * s + row] = D;
}
// dQ (64 queries to a workgroup) and dK/dV (64 keys) side by side, for few workgroups, where each alone leaves much of the chip idle and
// takes as long as its longest walk.  Eight workgroups of one and eight of the other in turn, so that both kernels' long
// walks start first.  Times of both ways stand at the launcher.
template <int DH, bool CAUSAL, int NPK, int QT, bool SPLIT>
__global__ void __launch_bounds__(128 * NPK * (SPLIT ? 2 : 1), 2)
attn_bwd_pair_tiles(const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ dctx, const float* __restrict__ lse,
                    float* __restrict__ delta, bf16_t* __restrict__ dqkv, int s, int b, int heads, const uint8_t* __restrict__ mask) {
  constexpr int NPQ = NPK * (SPLIT ? 2 : 1);   // dQ's groups of waves: both kernels' workgroups have the same size
  extern __shared__ __attribute__((aligned(1024))) char smem_all[];
  const int id = (blockIdx.x >> 4) * 8 + (blockIdx.x & 7);
  if (!(blockIdx.x & 8)) attn_dkv_block<DH, CAUSAL, 2, NPK, QT, SPLIT, false>(qkv, dctx, lse, delta, dqkv, s, b, heads, mask, id, smem_all);
  else attn_dq_block<DH, CAUSAL, 2, NPQ, 32, false, true>(qkv, nullptr, dctx, lse, delta, dqkv, s, b, heads, mask, id, smem_all);
}

// ------------------------------------------------------------------------------------------------
// host launchers
// ------------------------------------------------------------------------------------------------
bool attn_dh_supported(int dtype, int dh) {
  if (dh <= 0 || dh % 8 != 0) return false;
  if (dtype == PTDP_F32) return dh <= kMaxF32Dh;
  return dh == 32 || dh == 64 || dh == 96 || dh == 128 || dh == 160;
}

template <int DH, bool CAUSAL, int QW, int NP, int KT, bool WIDE = false>
static int attn_fwd_tiles_np(const bf16_t* qkv, bf16_t* ctx, float* lse, int s, int b, int heads, const uint8_t* mask, hipStream_t stream) {
  constexpr int tiles = NP * 4 * TileDma<DH, QW, KT, WIDE>::kBytes, part = NP > 1 ? QW * (2 + DH / 2) * 64 * (int)sizeof(float) : 0;
  constexpr int smem = tiles > part ? tiles : part;
  static once_flag_t done[kMaxDevices];
  if (set_dynamic_smem(reinterpret_cast<const void*>(attn_fwd_tiles<DH, CAUSAL, QW, NP, KT, WIDE>), smem, done) != PTDP_OK) return PTDP_E_HIP;
  const int nblk = (s + 32 * QW - 1) / (32 * QW);
  const dim3 grid(CAUSAL && !WIDE ? attn_grid_levels(nblk, heads, b) : attn_grid(nblk, heads, b));
  hipLaunchKernelGGL((attn_fwd_tiles<DH, CAUSAL, QW, NP, KT, WIDE>), grid, dim3(64 * QW * NP), smem, stream, qkv, ctx, lse, s, b, heads, mask);
  return PTDP_OK;
}

static inline double attn_flops(int s, int b, int heads, int dh) { return 4.0 * b * heads * (double)s * s * dh; }

static int attn_compute_units() {
  static std::atomic<int> cached[kMaxDevices];   // per device, looked up once
  const int d = device_slot();
  if (d >= 0 && cached[d].load(std::memory_order_relaxed) > 0) return cached[d].load(std::memory_order_relaxed);
  int dev = 0, cu = 256;
  if (hipGetDevice(&dev) == hipSuccess) {
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0) cu = v;
  }
  if (d >= 0) cached[d].store(cu, std::memory_order_relaxed);
  return cu;
}
// The form of a kernel that a call takes.  w: a workgroup's queries (dK/dV: keys) / 32; groups: how many groups of waves share its
// walk; tile: rows per tile; split: one result per wave (dK/dV).
// wide: the row pitch b * 3 * heads * dh is too large for slices with 32-bit offsets (attn_slice_fits), or so many workgroups of
// the form that a launch cannot number their threads: tiles with 64-bit addresses, workgroups of two waves.
// us with tiles through registers as these calls had them before 32-bit offsets and so (63 rows and less): 24576 samples x 16 heads of
// 128, causal, 16 rows forward 2640, 2430, backward 10870, 8930; 40 rows 5390, 5790 and 22000, 22200.
struct AttnForm {
  int w, groups, tile;
  bool split, wide;
};
static AttnForm attn_wide_or(AttnForm f, AttnForm wide, bool causal, int s, int b, int heads, int dh) {
  const uint64_t pairs = (uint64_t)b * heads;
  const int nblk = (s + 32 * f.w - 1) / (32 * f.w), threads = 64 * f.w * (f.split ? 2 : 1) * f.groups;
  if (pairs >= (1ull << 31) || !attn_slice_fits(pairs * 3 * dh, dh)) return wide;
  const long long blocks = causal ? attn_grid_levels(nblk, heads, b) : attn_grid(nblk, heads, b);
  return blocks < (1ll << 32) / threads ? f : wide;
}
// Forward.  Long walks (seven blocks of 64 rows and more) are split in two while one group per workgroup would leave the chip's
// 2048 wave slots half empty, with 64 queries per workgroup as long as about every compute unit gets one (heads of 64 and less:
// two fit), else with 128, for heads of 96 and 128 up to two blocks of 64 per compute unit unless a long causal walk is to be cut.
// us for (2, 2, 64), (4, 2, 64), (4, 1, 64): 8 heads of 128 x 2048 28.5, 34, 41; 12 heads 30, 36, 43; 16 heads without the mask
// 58, 41, 47, 20 heads 101, 77, 66; 32 heads of 64 35, 32, 35; 64 heads of 128 151, 102, 87.  Heads of 160: two groups' stages of
// 64 keys would take all LDS, so tiles of 32: (2, 2, 32), (4, 1, 64): 20 heads 54, 57.
// Short walks are not worth a merge once every compute unit has work, and stages of 64 keys then keep workgroups off the chip:
//   one block: (2, 1, 32).  us for it, (2, 2, 64), (4, 2, 64), (4, 1, 64): 1024 heads of 128 x 64 15.2, 26.3, 28.3, 16.1; of 64
//     7.2, 9.9, 10.8, 7.0; 64 heads of 64 4.5, 4.5, 4.6, 4.5;
//   three: 128 queries would leave three waves idle in half of the workgroups, or two, which only very many heads hide.
//     (2, 1, 32), (4, 1, 64): 4096 heads of 32 x 129 44, 57, of 128 153, 173; 672 heads of 128 x 164 without the mask 0.87 of the time;
//   up to six: (4, 1, 64) and (2, 2, 64), (4, 2, 64): 64 heads of 128 x 320 10.3, -, 14.7, without the mask 12.0, -, 17.9.
// A general mask whose rows are not a multiple of four bytes is read byte by byte, which with one tile of 32 keys ahead hides
// better: (2, 2, 32) and (2, 2, 64), (4, 2, 64), (4, 1, 64): 32 heads of 96 x 577 36, 53, 36, 48; 256 of 64 x 1030 454, 598, 490, 590.
static AttnForm attn_fwd_form(int dh, bool causal, bool masked, int s, int b, int heads) {
  const int n = (s + 63) / 64;
  const long long blocks64 = (long long)n * heads * b, ncu = attn_compute_units();
  const bool bytes = masked && (s & 3), one_wave_left = s % 128 > 0 && s % 128 <= 32;
  const AttnForm small = {2, 1, 32, false, false}, split32 = {2, 2, 32, false, false}, split64 = {2, 2, 64, false, false};
  const AttnForm split128 = {4, 2, 64, false, false};
  AttnForm f = {4, 1, 64, false, false};
  if (dh > 128) {
    if (blocks64 <= 4 * ncu) f = split32;
  } else if (bytes && n <= 2 && (blocks64 <= 2 * ncu || (dh <= 64 && s > 96))) {
    f = split32;
  } else if (n == 1) {
    f = small;
  } else if (bytes && n >= 3 && (n <= 5 || blocks64 > ncu)) {
    f = blocks64 > 2 * ncu && ((dh >= 64 && n == 3) || (dh == 128 && n <= 6)) ? small : split32;
  } else if (blocks64 <= (dh <= 64 ? n <= 3 ? ncu * 3 / 2 : ncu * 2 : causal && n > 6 ? ncu * 3 / 2 : ncu)) {
    f = split64;
  } else if (n > 6 && blocks64 <= (dh > 64 && (!causal || n <= 16) ? 2 : 4) * ncu) {
    f = split128;
  } else if (n == 3 && (one_wave_left || (blocks64 > 3 * ncu && blocks64 <= 10 * ncu))) {
    f = small;
  }
  return attn_wide_or(f, {2, 1, 32, false, true}, causal, s, b, heads, dh);
}
template <int DH, bool CAUSAL>
static int attn_fwd_mfma_t(const bf16_t* qkv, bf16_t* ctx, float* lse, int s, int b, int heads, const uint8_t* mask,
                           hipStream_t stream) {
  const AttnForm f = attn_fwd_form(DH, CAUSAL, !CAUSAL && mask != nullptr, s, b, heads);
  if (f.wide) return attn_fwd_tiles_np<DH, CAUSAL, 2, 1, 32, true>(qkv, ctx, lse, s, b, heads, mask, stream);
  if (f.w == 4 && f.groups == 1) return attn_fwd_tiles_np<DH, CAUSAL, 4, 1, 64>(qkv, ctx, lse, s, b, heads, mask, stream);
  if constexpr (DH > 128) {
    return attn_fwd_tiles_np<DH, CAUSAL, 2, 2, 32>(qkv, ctx, lse, s, b, heads, mask, stream);
  } else {
    if (f.groups == 1) return attn_fwd_tiles_np<DH, CAUSAL, 2, 1, 32>(qkv, ctx, lse, s, b, heads, mask, stream);
    if (f.tile == 32) return attn_fwd_tiles_np<DH, CAUSAL, 2, 2, 32>(qkv, ctx, lse, s, b, heads, mask, stream);
    if (f.w == 2) return attn_fwd_tiles_np<DH, CAUSAL, 2, 2, 64>(qkv, ctx, lse, s, b, heads, mask, stream);
    return attn_fwd_tiles_np<DH, CAUSAL, 4, 2, 64>(qkv, ctx, lse, s, b, heads, mask, stream);
  }
}

// a launch numbers its threads with 32 bits: the form of the smallest workgroups (wide) has to fit
static bool attn_sizes_fit(int s, int b, int heads) {
  const uint64_t pairs = (uint64_t)b * heads;
  return pairs < (1ull << 31) && attn_grid((s + 63) / 64, heads, b) < (1ll << 32) / 128;
}

// steps of 16 dh, rounded up to one of the built forms
#define PTDP_F32_DISPATCH(dh, CALL) \
  do {                              \
    if ((dh) <= 32) CALL(2);        \
    else if ((dh) <= 64) CALL(4);   \
    else if ((dh) <= 96) CALL(6);   \
    else if ((dh) <= 128) CALL(8);  \
    else if ((dh) <= 160) CALL(10); \
    else CALL(16);                  \
  } while (0)

template <int ND, int NW, int PARTS>
static void attn_fwd_f32_nw(const float* qkv, float* ctx, float* lse, int s, int b, int heads, int dh, const uint8_t* mask, int causal,
                            hipStream_t stream) {
  hipLaunchKernelGGL((attn_fwd_f32<ND, NW, PARTS>), dim3((s + kF32Rows - 1) / kF32Rows, heads, b), dim3(64 * NW), 0, stream, qkv, ctx, lse, s, b, heads, dh,
                     mask, causal);
}
// Eight waves for more than four tiles of 16 keys while the workgroups leave the chip's wave slots empty (heads beyond 128 take too
// many registers).  us with four and with eight waves, causal: 64 workgroups of dh 64 x 128 9.1, 8.1, x 256 14.5, 11.3; 256 x 256 15.1, 11.6; 512 x
// 512 47, 33; 1024 107, 108; dh 128: 256 x 256 41, 29, 512 91, 95; 48 rows (three tiles) 6.3, 7.1.  (Four waves with four parts: that four waves make
// the eight parts of a longer walk costs them, in the forward, 1024 workgroups of 32 x 66 7.0 -> 7.5, 32 x 256 18.2 -> 18.4, 64 x 128 20.6 -> 21.1,
// 96 x 100 26.6 -> 27.9, 64 x 512 58.6 -> 56.9; backward -4 to +4 %.)
template <int ND>
static void attn_fwd_f32_t(const float* qkv, float* ctx, float* lse, int s, int b, int heads, int dh, const uint8_t* mask, int causal,
                           hipStream_t stream) {
  if constexpr (ND <= 8) {
    const long long groups = (long long)((s + kF32Rows - 1) / kF32Rows) * heads * b, ncu = attn_compute_units();
    if (s > 4 * kF32Rows) {
      if (groups <= (ND <= 6 ? 2 : 1) * ncu) return attn_fwd_f32_nw<ND, 8, 8>(qkv, ctx, lse, s, b, heads, dh, mask, causal, stream);
      return attn_fwd_f32_nw<ND, 4, 8>(qkv, ctx, lse, s, b, heads, dh, mask, causal, stream);
    }
  }
  attn_fwd_f32_nw<ND, 4, 4>(qkv, ctx, lse, s, b, heads, dh, mask, causal, stream);
}

// Without the causal mask every row is a full row: count the whole s x s square as executed too.
int launch_attn_fwd(int dtype, const void* qkv, void* ctx, float* lse, int s, int b, int heads, int dh,
                    const uint8_t* mask, int causal, hipStream_t stream) {
  if (s == 0 || b == 0 || heads == 0) return PTDP_OK;
  if (!attn_dh_supported(dtype, dh) || (dtype == PTDP_BF16 && !attn_sizes_fit(s, b, heads))) return PTDP_E_UNSUPPORTED;
  Launch L(PTDP_K_ATTN_FWD, attn_flops(s, b, heads, dh), stream);
  int rc = PTDP_OK;
  if (dtype == PTDP_F32) {
#define PTDP_ATTN_FWD32(ND) attn_fwd_f32_t<ND>((const float*)qkv, (float*)ctx, lse, s, b, heads, dh, mask, causal, stream)
    PTDP_F32_DISPATCH(dh, PTDP_ATTN_FWD32);
#undef PTDP_ATTN_FWD32
  } else {
    const bf16_t* q = (const bf16_t*)qkv;
    bf16_t* c = (bf16_t*)ctx;
#define PTDP_ATTN_FWD(D) \
  rc = causal ? attn_fwd_mfma_t<D, true>(q, c, lse, s, b, heads, mask, stream) \
              : attn_fwd_mfma_t<D, false>(q, c, lse, s, b, heads, mask, stream)
    if (dh == 32) PTDP_ATTN_FWD(32);
    else if (dh == 96) PTDP_ATTN_FWD(96);
    else if (dh == 64) PTDP_ATTN_FWD(64);
    else if (dh == 128) PTDP_ATTN_FWD(128);
    else PTDP_ATTN_FWD(160);
#undef PTDP_ATTN_FWD
  }
  if (rc != PTDP_OK) return rc;
  return L.status();
}

// Backward.  dQ and dK/dV run in one launch while both fit the chip side by side (more, and the delta computed once per block of keys
// and the larger of the two kernels' registers for both cost more than the second launch; heads beyond 160 spill), in workgroups
// of eight waves where the walk has more than four tiles and that leaves room.  us, causal, for two launches of four waves, two of
// eight, one of four, one of eight; n workgroups of 16 rows:
//   n = 6 of dh 64 x 48 15.8, 17.9, 9.0, 10.9;  64 of 32 x 128 15.9, -, 9.3, 8.0, of 64 x 128 25.8, 22.5, 15.9, 13.7 (a layer of 256 tokens 124.4 -> 114.7 with one of four),
//   of 64 x 256 42, 34, 27.8, 21.4, of 96 x 256 62, 49, 41, 31;  128 of 64 x 256 -, 34.5, 28.2, 21.7;  256 of 32 x 256 25, 20.3, 20.4, 17.2, of 64 x 128 26.9, 23.2, 23.7,
//   26.3, x 256 45, 35.5, 41.4, 41.8, of 96 x 256 66, 51, 61, 66, of 128 x 256 87, -, 120, -;  448 of 64 x 100 31, 36, 33.7, -;  512 of 32 x 512 62, 47.8, 55, 55, of 64 x
//   512 112, 105, 144, -, x 1024 202, 186, 215, -;  1344 of 64 x 333 147, 165.  Without the mask the same but for 512 and more of 32.
struct F32Bwd {
  bool together;
  int waves;
};
static F32Bwd f32_bwd_form(int dh, int causal, int s, long long groups) {
  const long long ncu = attn_compute_units();
  if (dh > 96) return {dh <= 160 && groups <= ncu / 2, 4};
  if (groups <= (dh <= 32 ? ncu : ncu / 2)) return {true, s > 4 * kF32Rows ? 8 : 4};
  if (s >= 256 && groups <= 2 * ncu) return {false, 8};
  return {groups <= (dh <= 32 && causal ? 2 * ncu : ncu), 4};
}
template <int ND, int NW, int PARTS>
static void attn_bwd_f32_nw(bool together, const float* qkv, const float* ctx, const float* lse, const float* dctx, float* dqkv, float* delta,
                            int s, int b, int heads, int dh, const uint8_t* mask, int causal, hipStream_t stream) {
  const dim3 grid((s + kF32Rows - 1) / kF32Rows, heads, b), block(64 * NW);
  if constexpr (ND <= 10) {
    if (together) {
      hipLaunchKernelGGL((attn_bwd_f32<ND, NW, PARTS>), dim3(2 * grid.x, heads, b), block, 0, stream, qkv, ctx, dctx, lse, dqkv, s, b, heads, dh, mask, causal);
      return;
    }
  }
  hipLaunchKernelGGL((attn_bwd_dq_f32<ND, NW, PARTS>), grid, block, 0, stream, qkv, ctx, dctx, lse, delta, dqkv, s, b, heads, dh, mask, causal);
  hipLaunchKernelGGL((attn_bwd_dkv_f32<ND, NW, PARTS>), grid, block, 0, stream, qkv, dctx, lse, (const float*)delta, dqkv, s, b, heads, dh, mask, causal);
}
template <int ND>
static void attn_bwd_f32_t(const float* qkv, const float* ctx, const float* lse, const float* dctx, float* dqkv, float* delta, int s,
                           int b, int heads, int dh, const uint8_t* mask, int causal, hipStream_t stream) {
  const F32Bwd f = f32_bwd_form(dh, causal, s, (long long)((s + kF32Rows - 1) / kF32Rows) * heads * b);
  if constexpr (ND <= 6) {
    if (f.waves == 8) return attn_bwd_f32_nw<ND, 8, 8>(f.together, qkv, ctx, lse, dctx, dqkv, delta, s, b, heads, dh, mask, causal, stream);
    if (s > 4 * kF32Rows) return attn_bwd_f32_nw<ND, 4, 8>(f.together, qkv, ctx, lse, dctx, dqkv, delta, s, b, heads, dh, mask, causal, stream);
  }
  attn_bwd_f32_nw<ND, 4, 4>(f.together, qkv, ctx, lse, dctx, dqkv, delta, s, b, heads, dh, mask, causal, stream);
}

template <int DH, bool CAUSAL, int QW, int NP, int KT, bool WIDE = false>
static int attn_bwd_dq_tiles_np(const bf16_t* qkv, const bf16_t* ctx, const bf16_t* dctx, const float* lse, float* delta, bf16_t* dqkv,
                                int s, int b, int heads, const uint8_t* mask, hipStream_t stream) {
  constexpr int tiles = NP * 4 * TileDma<DH, QW, KT, WIDE>::kBytes, sums = NP > 1 ? QW * (DH / 2) * 64 * (int)sizeof(float) : 0;
  constexpr int smem = tiles > sums ? tiles : sums;
  static once_flag_t done[kMaxDevices];
  if (set_dynamic_smem(reinterpret_cast<const void*>(attn_bwd_dq_tiles<DH, CAUSAL, QW, NP, KT, WIDE>), smem, done) != PTDP_OK) return PTDP_E_HIP;
  const int nblk = (s + 32 * QW - 1) / (32 * QW);
  const dim3 grid(CAUSAL && !WIDE ? attn_grid_levels(nblk, heads, b) : attn_grid(nblk, heads, b));
  hipLaunchKernelGGL((attn_bwd_dq_tiles<DH, CAUSAL, QW, NP, KT, WIDE>), grid, dim3(64 * QW * NP), smem, stream, qkv, ctx, dctx, lse, delta,
                     dqkv, s, b, heads, mask);
  return PTDP_OK;
}

// Which form: as for the forward kernel.  us for (2, 2, 32), (2, 2, 64), (4, 2, 64), (4, 1, 64): 8 heads of 128 x 2048 34, 33, 43, 49; 16
// heads 42, 46, 50, 53; 24 heads 52, 69, 54, 58; 32 heads 68, 87, 65, 64; 64 heads 122, 172, 129, 106; 32 heads of 64 36, 42, 40, 44;
// 128 heads of 32 94, 102, 87, 76; 20 and 40 heads of 160 (first and last) 56, 69 and 101, 88; 16 heads of 128 without the mask 61,
// 80, 56, 60.
// One block of 64 rows, or three (all causal calls, where the last one is one wave's, and heads of up to 64 unless very many):
// workgroups of 128 rows would be half empty.
// us for the whole backward with (2, 1, 32), (4, 1, 64): 4096 heads of 32 x 129, causal, 154, 183; of 128 x 129 692, 788; 1024 of 64 x 64
// 27.7, 29.8.
static bool attn_bwd_small(int dh, bool causal, int s, long long blocks64, long long ncu) {
  const int n = (s + 63) / 64;
  return dh <= 128 && ((n == 1 && blocks64 > 2 * ncu) || (n == 3 && blocks64 > (causal && dh == 64 ? 2 : 3) * ncu &&
                                                                      (causal || (s % 128 > 0 && s % 128 <= 32) || (dh <= 64 && blocks64 <= 10 * ncu))));
}
// Heads of 32 under a mask read byte by byte stay in two groups: 512 heads x 333 196, (4, 1, 64) 232.
static AttnForm attn_dq_form(int dh, bool causal, bool masked, int s, int b, int heads) {
  const int n = (s + 63) / 64;
  const long long blocks64 = (long long)n * heads * b, ncu = attn_compute_units();
  AttnForm f = {2, 2, 32, false, false};
  if (attn_bwd_small(dh, causal, s, blocks64, ncu)) f = {2, 1, 32, false, false};
  else if (blocks64 > (dh > 64 || (causal && n <= 6) ? 3 : 4) * ncu && !(dh == 32 && masked && (s & 3))) f = {4, 1, 64, false, false};
  return attn_wide_or(f, {2, 1, 32, false, true}, causal, s, b, heads, dh);
}
template <int DH, bool CAUSAL>
static int attn_bwd_dq_t(const bf16_t* qkv, const bf16_t* ctx, const bf16_t* dctx, const float* lse, float* delta, bf16_t* dqkv, int s,
                         int b, int heads, const uint8_t* mask, hipStream_t stream) {
  const AttnForm f = attn_dq_form(DH, CAUSAL, !CAUSAL && mask != nullptr, s, b, heads);
  if (f.wide) return attn_bwd_dq_tiles_np<DH, CAUSAL, 2, 1, 32, true>(qkv, ctx, dctx, lse, delta, dqkv, s, b, heads, mask, stream);
  if constexpr (DH <= 128)
    if (f.w == 2 && f.groups == 1) return attn_bwd_dq_tiles_np<DH, CAUSAL, 2, 1, 32>(qkv, ctx, dctx, lse, delta, dqkv, s, b, heads, mask, stream);
  if (f.groups == 1) return attn_bwd_dq_tiles_np<DH, CAUSAL, 4, 1, 64>(qkv, ctx, dctx, lse, delta, dqkv, s, b, heads, mask, stream);
  return attn_bwd_dq_tiles_np<DH, CAUSAL, 2, 2, 32>(qkv, ctx, dctx, lse, delta, dqkv, s, b, heads, mask, stream);
}

template <int DH, bool CAUSAL, int KW, int NP, int QT, bool SPLIT, bool WIDE = false>
static int attn_bwd_dkv_tiles_np(const bf16_t* qkv, const bf16_t* dctx, const float* lse, const float* delta, bf16_t* dqkv, int s, int b,
                                 int heads, const uint8_t* mask, hipStream_t stream) {
  using Geom = DkvGeom<DH, CAUSAL, KW, NP, QT, SPLIT>;
  static once_flag_t done[kMaxDevices];
  const auto kernel = attn_bwd_dkv_tiles<DH, CAUSAL, KW, NP, QT, SPLIT, WIDE>;
  if (set_dynamic_smem(reinterpret_cast<const void*>(kernel), Geom::lds_bytes(!CAUSAL), done) != PTDP_OK) return PTDP_E_HIP;
  const int nblk = (s + 32 * KW - 1) / (32 * KW);
  const dim3 grid(CAUSAL && !WIDE ? attn_grid_levels(nblk, heads, b) : attn_grid(nblk, heads, b));
  hipLaunchKernelGGL(kernel, grid, dim3(Geom::kThreads * NP), Geom::lds_bytes(!CAUSAL && mask != nullptr), stream, qkv, dctx, lse, delta, dqkv,
                     s, b, heads, mask);
  return PTDP_OK;
}
// Which form.  us for the whole backward (measured with hidden scores selected in every tile: all forms 6-10 % slower than now)
// with (4, 1, 64), (2, 2, 32), (2, 2, 64) and, split by result, (2, 1, 32), (2, 2, 32), (2, 2, 64):
//   heads x s     dh 128 8 x 2048 146, 104, 103, 118, 95, 92; 12 x 2048 155, 116, 111, 130, 106, 103; 24 x 2048 186, 148, 186, 154, 177, 175;
//                 32 x 2048 215, 188, 236, 196, 225, 224; 64 x 2048 327, 344, 444, 350, 422, 415; without the mask 16 x 2048 211, 181, 260,
//                 188, 206, 201, 64 x 2048 572, 613, 932, 620, 727, 709
//                 dh 160 (no room for the last; both results spill) 16 x 1001 147, 96, -, 76, 66; 20 x 2048 323, 260, -, 169, 180
//                 dh 96 8 x 1024 59, 45, 43; 20 x 2048 127, 102, 122; 64 x 2048 246, 257, 322; 64 x 1024 under a general mask 144, 154, 188
//                 dh 64 16 x 333 25, 19.6, 19.2; 64 x 512 under a general mask 44, 40, 38; 32 x 2048 122, 101, 110; 64 x 2048 equal
//                 dh 32 32 x 512 23, 18.3, 17.7; 32 x 2048 88, 70, 68; 128 x 2048 212, 225, 223
// Few blocks per head, as for dQ: (2, 1, 64) for heads of up to 64, (2, 1, 32) for others.  us for the whole backward with (2, 1, 64),
// (2, 1, 32), (4, 1, 64), (2, 2, 32): causal 4096 heads of 64 x 129 329, 329, 402, 360; 1024 of 64 x 64 27.0, 27.7, 29.1, 31.1; 4096 of 128 x 129
// 682, 584, 789, 663; 256 of 64 x 200 31.2, 30.9, 30.0, 36.1.
static AttnForm attn_dkv_form(int dh, bool causal, int s, int b, int heads) {
  const int n = (s + 63) / 64;
  const long long blocks64 = (long long)n * heads * b, ncu = attn_compute_units();
  AttnForm f = {2, 2, 32, false, false};
  if (dh > 128) f = {2, blocks64 <= 2 * ncu ? 2 : 1, 32, true, false};
  else if (attn_bwd_small(dh, causal, s, blocks64, ncu)) f = {2, 1, dh <= 64 ? 64 : 32, false, false};
  else if (blocks64 > (causal && n > 6 ? 6 : 3) * ncu) f = {4, 1, 64, false, false};
  else if (dh == 128 ? !causal && blocks64 <= ncu * 3 / 2 : dh == 96 || (dh == 32 && causal) ? false : blocks64 <= 2 * ncu) f = {2, 2, 64, dh == 128, false};
  return attn_wide_or(f, {2, 1, 32, false, true}, causal, s, b, heads, dh);
}
template <int DH, bool CAUSAL>
static int attn_bwd_dkv_t(const bf16_t* qkv, const bf16_t* dctx, const float* lse, const float* delta, bf16_t* dqkv, int s, int b, int heads,
                          const uint8_t* mask, hipStream_t stream) {
  const AttnForm f = attn_dkv_form(DH, CAUSAL, s, b, heads);
  if (f.wide) return attn_bwd_dkv_tiles_np<DH, CAUSAL, 2, 1, 32, false, true>(qkv, dctx, lse, delta, dqkv, s, b, heads, mask, stream);
  if constexpr (DH > 128) {
    if (f.groups == 2) return attn_bwd_dkv_tiles_np<DH, CAUSAL, 2, 2, 32, true>(qkv, dctx, lse, delta, dqkv, s, b, heads, mask, stream);
    return attn_bwd_dkv_tiles_np<DH, CAUSAL, 2, 1, 32, true>(qkv, dctx, lse, delta, dqkv, s, b, heads, mask, stream);
  } else {
    if (f.w == 2 && f.groups == 1)
      return attn_bwd_dkv_tiles_np<DH, CAUSAL, 2, 1, DH <= 64 ? 64 : 32, false>(qkv, dctx, lse, delta, dqkv, s, b, heads, mask, stream);
    if (f.w == 4) return attn_bwd_dkv_tiles_np<DH, CAUSAL, 4, 1, 64, false>(qkv, dctx, lse, delta, dqkv, s, b, heads, mask, stream);
    if constexpr (DH == 64 || (DH != 96 && !CAUSAL))
      if (f.tile == 64) return attn_bwd_dkv_tiles_np<DH, CAUSAL, 2, 2, 64, DH == 128>(qkv, dctx, lse, delta, dqkv, s, b, heads, mask, stream);
    return attn_bwd_dkv_tiles_np<DH, CAUSAL, 2, 2, 32, false>(qkv, dctx, lse, delta, dqkv, s, b, heads, mask, stream);
  }
}
// dQ and dK/dV side by side in one launch, behind one for delta (k_tile = 0: one after the other).  dQ: 64 queries, k_groups (split: twice as
// many) groups of waves, tiles of 32; dK/dV: 64 keys, k_groups groups, tiles of k_tile, split by result or not.  Time of the whole
// backward over that of the two kernels in turn, causal / without a mask, at blocks of 64 rows = 128, 256, 384, 512:
//   dh 32 (2, 64) s = 512 .73 .78 .83 .89 / .73 .84 .83 1.04, 2048 .62 .66 .67 .73 / .64 .77 .76 1.01;   64 the same, 512 .72 .77 .97 1.06 / .73 .88 1.01 1.13,
//   1024 .66 .73 .81 .96 / .67 .86 .95 1.07, 2048 .62 .67 .69 .85 / .63 .84 .96 1.07;   96 (2, 64) 512 .74 .96 1.13 1.38 / .76 1.12 1.14 1.35, (2, 32) 512 .76 .83 .97
//   1.04 / .78 .96 .97 1.06, 2048 .67 .74 .76 .89 / .69 .91 .99 1.05;   128 (2, 64, split) 512 .74 .99 1.07 1.33 / .73 1.18, 1024 .69 .86 / .69 1.15, 2048 .65 .77 / .66
//   1.12, (1, 32, split) 200 .75 .95 .82 1.07 / .72 .91 .85 1.01, 512 .81 .88 .89 1.01 / .80 1.01 .89 1.10, 2048 .88 .94 .94 .97 / .90 1.09 1.06 1.21, (2, 32) 1024 .81 .86 .85
//   .91, 2048 .80 .86 .85 .84;   160 (2, 32, split) 512 .72 .97 1.08 / .73 1.16, 2048 .62 .76 1.03 / .67 1.19, (1, 32, split) 200 .74 .93 .80 .86 / .73 .89 .81 .89,
//   512 .76 .84 .90 .93 / .79 .96 .89 .98, 2048 .79 .87 .92 1.02 / .84 1.07 1.04 1.11.  Heads of 64 x 512, general mask: as without.
// Registers: (2, 32) of 128, causal, takes all 256 and spills three (16 bytes a lane), as dK/dV does in a launch of its own; no other spills.
struct AttnPair {
  int k_groups, k_tile;
  bool split;
};
static AttnPair attn_pair_form(int dh, bool causal, bool masked, int s, int b, int heads) {
  const int n = (s + 63) / 64;
  const long long blocks64 = (long long)n * heads * b, ncu = attn_compute_units();
  const bool half = blocks64 <= ncu / 2, one = blocks64 <= ncu, more = blocks64 <= ncu * 3 / 2, two = blocks64 <= 2 * ncu;
  const AttnPair none = {0, 0, false};
  if (dh <= 64) {
    const bool take = one || (dh == 32 ? more || (causal && two) : causal && ((n >= 8 && more) || (n >= 16 && two)));
    return take ? AttnPair{2, 64, false} : none;
  }
  if (dh == 96) return half ? AttnPair{2, 64, false} : one || (causal && n >= 8 && more) ? AttnPair{2, 32, false} : none;
  const AttnPair split1 = {1, 32, true}, split2 = {2, dh == 128 ? 64 : 32, true}, whole = {2, 32, false};
  const bool long_walk = causal && n >= 16;
  if (half) return n <= 4 ? split1 : split2;
  if (one && long_walk) return split2;
  if (dh == 128 && long_walk) return two ? whole : none;
  return more && (causal || (n <= 5 && !masked)) ? split1 : none;
}
void attn_form_query(int kernel, int causal, int masked, int s, int b, int heads, int dh, int* rows, int* groups, int* tile, int* wide) {
  AttnForm f = kernel == PTDP_ATTN_KERNEL_FWD ? attn_fwd_form(dh, causal != 0, !causal && masked, s, b, heads)
               : kernel == PTDP_ATTN_KERNEL_DQ ? attn_dq_form(dh, causal != 0, !causal && masked, s, b, heads) : attn_dkv_form(dh, causal != 0, s, b, heads);
  const AttnPair p = attn_pair_form(dh, causal != 0, !causal && masked, s, b, heads);
  if (kernel != PTDP_ATTN_KERNEL_FWD && p.k_tile > 0) {
    f = kernel == PTDP_ATTN_KERNEL_DQ ? AttnForm{2, p.split ? 2 * p.k_groups : p.k_groups, 32, false, false} : AttnForm{2, p.k_groups, p.k_tile, p.split, false};
  }
  *rows = 32 * f.w;
  *groups = f.groups;
  *tile = f.tile;
  *wide = f.wide;
}
void attn_bwd_launch_query(int causal, int masked, int s, int b, int heads, int dh, int* together, int* split) {
  const AttnPair p = attn_pair_form(dh, causal != 0, !causal && masked, s, b, heads);
  *together = p.k_tile > 0;
  *split = p.k_tile > 0 ? p.split : attn_dkv_form(dh, causal != 0, s, b, heads).split;
}
template <int DH, bool CAUSAL, int NPK, int QT, bool SPLIT>
static int attn_bwd_pair(const bf16_t* qkv, const bf16_t* ctx, const float* lse, const bf16_t* dctx, bf16_t* dqkv, float* delta, int s, int b,
                         int heads, const uint8_t* mask, hipStream_t stream) {
  using Geom = DkvGeom<DH, CAUSAL, 2, NPK, QT, SPLIT>;
  constexpr int NPQ = NPK * (SPLIT ? 2 : 1), tiles = NPQ * 4 * TileDma<DH, 2, 32, false>::kBytes, sums = DH * 64 * (int)sizeof(float);
  constexpr int dq_smem = tiles > sums ? tiles : sums;
  auto larger = [](int x) { return x > dq_smem ? x : dq_smem; };
  static once_flag_t done[kMaxDevices];
  const auto kernel = attn_bwd_pair_tiles<DH, CAUSAL, NPK, QT, SPLIT>;
  if (set_dynamic_smem(reinterpret_cast<const void*>(kernel), larger(Geom::lds_bytes(!CAUSAL)), done) != PTDP_OK) return PTDP_E_HIP;
  const int nblk = (s + 63) / 64;
  const unsigned units = (unsigned)((s + 31) / 32) * heads * b;
  hipLaunchKernelGGL(attn_delta_kernel<DH>, dim3((units + 3) / 4), dim3(256), 0, stream, ctx, dctx, delta, s, b, heads);
  const long long grid = CAUSAL ? attn_grid_levels(nblk, heads, b) : attn_grid(nblk, heads, b);
  hipLaunchKernelGGL(kernel, dim3(2 * grid), dim3(128 * NPQ), larger(Geom::lds_bytes(!CAUSAL && mask != nullptr)), stream, qkv, dctx, lse, delta, dqkv,
                     s, b, heads, mask);
  return PTDP_OK;
}
template <int DH, bool CAUSAL>
static int attn_bwd_mfma_t(const bf16_t* qkv, const bf16_t* ctx, const float* lse, const bf16_t* dctx, bf16_t* dqkv,
                           float* delta, int s, int b, int heads, const uint8_t* mask, hipStream_t stream) {
  const AttnPair p = attn_pair_form(DH, CAUSAL, !CAUSAL && mask != nullptr, s, b, heads);
  if constexpr (DH <= 96) {
    if (p.k_tile == 64) return attn_bwd_pair<DH, CAUSAL, 2, 64, false>(qkv, ctx, lse, dctx, dqkv, delta, s, b, heads, mask, stream);
    if constexpr (DH == 96)
      if (p.k_tile == 32) return attn_bwd_pair<DH, CAUSAL, 2, 32, false>(qkv, ctx, lse, dctx, dqkv, delta, s, b, heads, mask, stream);
  } else {
    if (p.split && p.k_groups == 2) return attn_bwd_pair<DH, CAUSAL, 2, DH == 128 ? 64 : 32, true>(qkv, ctx, lse, dctx, dqkv, delta, s, b, heads, mask, stream);
    if (p.split) return attn_bwd_pair<DH, CAUSAL, 1, 32, true>(qkv, ctx, lse, dctx, dqkv, delta, s, b, heads, mask, stream);
    if constexpr (DH == 128 && CAUSAL)
      if (p.k_groups == 2) return attn_bwd_pair<DH, CAUSAL, 2, 32, false>(qkv, ctx, lse, dctx, dqkv, delta, s, b, heads, mask, stream);
  }
  const int rc = attn_bwd_dq_t<DH, CAUSAL>(qkv, ctx, dctx, lse, delta, dqkv, s, b, heads, mask, stream);   // first: it writes delta
  if (rc != PTDP_OK) return rc;
  return attn_bwd_dkv_t<DH, CAUSAL>(qkv, dctx, lse, delta, dqkv, s, b, heads, mask, stream);
}

int launch_attn_bwd(int dtype, const void* qkv, const void* ctx, const float* lse, const void* dctx, void* dqkv,
                    float* delta, int s, int b, int heads, int dh, const uint8_t* mask, int causal, hipStream_t stream) {
  if (s == 0 || b == 0 || heads == 0) return PTDP_OK;
  if (!attn_dh_supported(dtype, dh) || (dtype == PTDP_BF16 && !attn_sizes_fit(s, b, heads))) return PTDP_E_UNSUPPORTED;
  Launch L(PTDP_K_ATTN_BWD, 2.0 * attn_flops(s, b, heads, dh), stream);
  int rc = PTDP_OK;
  if (dtype == PTDP_F32) {
#define PTDP_ATTN_BWD32(ND) \
  attn_bwd_f32_t<ND>((const float*)qkv, (const float*)ctx, lse, (const float*)dctx, (float*)dqkv, delta, s, b, heads, dh, mask, causal, stream)
    PTDP_F32_DISPATCH(dh, PTDP_ATTN_BWD32);
#undef PTDP_ATTN_BWD32
  } else {
    const bf16_t* q = (const bf16_t*)qkv;
    const bf16_t* c = (const bf16_t*)ctx;
    const bf16_t* d = (const bf16_t*)dctx;
    bf16_t* o = (bf16_t*)dqkv;
#define PTDP_ATTN_BWD(D) \
  rc = causal ? attn_bwd_mfma_t<D, true>(q, c, lse, d, o, delta, s, b, heads, mask, stream) \
              : attn_bwd_mfma_t<D, false>(q, c, lse, d, o, delta, s, b, heads, mask, stream)
    if (dh == 32) PTDP_ATTN_BWD(32);
    else if (dh == 96) PTDP_ATTN_BWD(96);
    else if (dh == 64) PTDP_ATTN_BWD(64);
    else if (dh == 128) PTDP_ATTN_BWD(128);
    else PTDP_ATTN_BWD(160);
#undef PTDP_ATTN_BWD
  }
  if (rc != PTDP_OK) return rc;
  return L.status();
}

}  // namespace ptdp
