// GeLU and its derivative (exact and tanh form), shared by the element-wise kernels and the GEMMs' output stages.
#pragma once
#include "common.h"

namespace ptdp {

// Standard normal CDF Phi(z) and density phi(z) from one exponential: with x = |z| / sqrt(2),
// erfc(x) = t (a1 + t (a2 + t (a3 + t (a4 + t a5)))) exp(-x^2), t = 1 / (1 + p x) (Abramowitz & Stegun 7.1.26,
// absolute error below 1.5e-7), taken on the side that needs no cancellation.  These kernels are bound by their
// arithmetic, not by memory (41 vector instructions per element before, against 16 bytes moved per 8 elements), so
// the constants are folded (the coefficients carry erfc's factor 0.5, the exponent -log2(e)/2) and the reciprocal is
// the hardware's 1-ulp one instead of a correctly rounded division (ten instructions): its error is a tenth of the
// formula's own.
__device__ __forceinline__ float normal_cdf_pdf(float z, float* pdf) {
  const float e = __builtin_amdgcn_exp2f(z * z * -0.7213475204444817f);   // exp(-z^2 / 2)
  const float t = __builtin_amdgcn_rcpf(fmaf(fabsf(z), 0.3275911f * 0.7071067811865476f, 1.f));
  const float poly = t * (0.127414796f + t * (-0.142248368f + t * (0.7107068705f + t * (-0.7265760135f + t * 0.5307027145f))));
  const float tail = poly * e;   // 0.5 erfc(|z| / sqrt(2))
  *pdf = e * 0.3989422804014327f;
  return z < 0.f ? tail : 1.f - tail;
}
// tanh(u) = 1 - 2 / (1 + exp(2u)) with the hardware's exponential and reciprocal (absolute error ~1e-7; exp
// overflowing to infinity gives exactly 1, underflowing to zero exactly -1)
__device__ __forceinline__ float fast_tanh(float u) {
  return 1.f - 2.f * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(u * 2.8853900817779268f));
}
template <int MODE> __device__ __forceinline__ float gelu_f(float z) {
  if (MODE == PTDP_GELU_TANH) {
    const float c = 0.7978845608028654f;
    return 0.5f * z * (1.f + fast_tanh(c * (z + 0.044715f * z * z * z)));
  }
  float pdf;
  return z * normal_cdf_pdf(z, &pdf);
}
template <int MODE> __device__ __forceinline__ float gelu_grad_f(float z) {
  if (MODE == PTDP_GELU_TANH) {
    const float c = 0.7978845608028654f;
    const float th = fast_tanh(c * (z + 0.044715f * z * z * z));
    return 0.5f * (1.f + th) + 0.5f * z * (1.f - th * th) * c * (1.f + 3.f * 0.044715f * z * z);
  }
  float pdf;
  const float cdf = normal_cdf_pdf(z, &pdf);
  return cdf + z * pdf;
}

}  // namespace ptdp
