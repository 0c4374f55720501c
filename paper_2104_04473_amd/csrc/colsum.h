// Second stage of the column sums (bias and LayerNorm parameter gradients): in a launch of its own or as workgroups of another one.
#pragma once
#include "common.h"

namespace ptdp {

// out[c] += sum over parts of part[p][c]  (second stage of every column sum; fixed order).
// A workgroup owns 64 columns; each of its sixteen waves adds a sixteenth of the parts with eight loads of either sum in
// flight, and the first wave adds the sixteen sums in order.  Bound by the latency of that chain of loads for narrow
// layers (with four waves of four loads, 256 parts took 22 us at any width; now 5) and by reading the partial sums
// for wide ones (h 25600: 44 -> 36 us).
// The parts left over behind whole groups of loads are requested together as well, at places that exist, and what is too much is
// not added: a branch for each made them a chain of up to seven trips to memory (two layers of 512, 666 tokens 262.2 -> 260.0 us, with the
// rows' early requests in layernorm_bwd_sums_kernel; two groups of eight in flight: 260.3, fp32 layer 256 wide 103.0 -> 103.5).
// Fewer than sixteen waves take several sixteenths each, one after the other: the same sums in the same order.
constexpr int kFinishWaves = 16, kFinishLoads = 8, kFinishRed = 2 * kFinishWaves * 64;
// the next kFinishLoads (WHOLE) or n > 0 parts; p is the same for the whole wave, c the lane's column
template <bool TWO, bool WHOLE>
__device__ __forceinline__ void colsum_finish_step(const float* __restrict__ p, int c, int n, int stride, int width, float (&sa)[kFinishLoads],
                                                   float (&sb)[kFinishLoads]) {
  float va[kFinishLoads], vb[kFinishLoads];
#pragma unroll
  for (int u = 0; u < kFinishLoads; ++u) {
    const float* row = p + (size_t)(WHOLE ? u : min(u, n - 1)) * stride;
    va[u] = row[c];
    vb[u] = TWO ? row[width + c] : 0.f;
  }
#pragma unroll
  for (int u = 0; u < kFinishLoads; ++u) {
    sa[u] += WHOLE || u < n ? va[u] : 0.f;
    sb[u] += WHOLE || u < n ? vb[u] : 0.f;
  }
}
template <bool TWO>
__device__ __forceinline__ void colsum_finish_part(const float* __restrict__ p, int c, int n, int stride, int width, float& a, float& b) {
  float sa[kFinishLoads], sb[kFinishLoads];
#pragma unroll
  for (int u = 0; u < kFinishLoads; ++u) sa[u] = sb[u] = 0.f;
  for (; n >= kFinishLoads; n -= kFinishLoads, p += (size_t)kFinishLoads * stride) colsum_finish_step<TWO, true>(p, c, n, stride, width, sa, sb);
  if (n > 0) colsum_finish_step<TWO, false>(p, c, n, stride, width, sa, sb);
  a = ((sa[0] + sa[1]) + (sa[2] + sa[3])) + ((sa[4] + sa[5]) + (sa[6] + sa[7]));
  b = ((sb[0] + sb[1]) + (sb[2] + sb[3])) + ((sb[4] + sb[5]) + (sb[6] + sb[7]));
}
// waves: of the workgroup; red: kFinishRed floats of LDS
__device__ __forceinline__ void colsum_finish_block(const ColsumJob& j, int blk, int waves, float* red) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = blk * 64 + lane;
  const int per = (j.nparts + kFinishWaves - 1) / kFinishWaves;
#pragma unroll 1
  for (int q = wave; q < kFinishWaves; q += waves) {
    const int p0 = q * per, n = min(j.nparts, p0 + per) - p0;
    float a = 0.f, b = 0.f;
    if (c < j.width && n > 0) {
      if (j.out1) colsum_finish_part<true>(j.part + (size_t)p0 * j.stride, c, n, j.stride, j.width, a, b);
      else colsum_finish_part<false>(j.part + (size_t)p0 * j.stride, c, n, j.stride, j.width, a, b);
    }
    red[q * 64 + lane] = a;
    red[(kFinishWaves + q) * 64 + lane] = b;
  }
  __syncthreads();
  // wave 0 finishes the first sum, wave 1 the second
  for (int o = wave; o < 2; o += waves) {
    float* out = o == 0 ? j.out0 : j.out1;
    if (!out || c >= j.width) continue;
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < kFinishWaves; ++w) t += red[(o * kFinishWaves + w) * 64 + lane];
    out[c] += t;
  }
}

// several finishes in one launch: job j owns workgroups first[j] .. first[j+1]-1
struct ColsumBatchArgs {
  ColsumJob job[kMaxColsumJobs];
  int first[kMaxColsumJobs + 1];
  int n;
};
__device__ __forceinline__ void colsum_finish_id(const ColsumBatchArgs& a, int id, int waves, float* red) {
  ColsumJob j = a.job[0];   // constant indices only: the arguments stay in scalar registers
  int first = 0;
#pragma unroll
  for (int q = 1; q < kMaxColsumJobs; ++q)
    if (q < a.n && id >= a.first[q]) {
      j = a.job[q];
      first = a.first[q];
    }
  colsum_finish_block(j, id - first, waves, red);
}
// *bytes += what the jobs read
inline ColsumBatchArgs colsum_batch_args(const ColsumBatch& batch, double* bytes) {
  ColsumBatchArgs a;
  a.n = batch.n;
  int at = 0;
  for (int j = 0; j < kMaxColsumJobs; ++j) {
    a.job[j] = batch.job[j < batch.n ? j : 0];   // unused slots repeat job 0 (never selected)
    a.first[j] = at;
    if (j < batch.n) {
      at += (batch.job[j].width + 63) / 64;
      *bytes += (double)batch.job[j].nparts * batch.job[j].stride * sizeof(float);
    }
  }
  a.first[kMaxColsumJobs] = at;
  return a;
}

}  // namespace ptdp
