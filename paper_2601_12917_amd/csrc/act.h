// erf-GELU in fp32 for the epilogues of the products.
#pragma once
#include <hip/hip_runtime.h>

namespace zgr {

// x Phi(x) = max(x, 0) - |x| / 2 erfc(|x| / sqrt 2), with erfc(|x| / sqrt 2) = exp2(q(|x|)): q is a degree-10 minimax fit of log2 erfc on [0, 6], weighted by
// what it moves in the result (1.5e-10 at most); beyond 6 the second term, below 6e-9, is left out.  Nothing cancels, so the result is closer
// than 0.5 x (1 + erff(x / sqrt 2)), whose sum does (8 standard deviations on either side of zero, against fp64: largest error 2.4e-7 and 4.5e-7, rms 4.3e-8 and 5.7e-8,
// largest relative error below 1 1.7e-7 and 2.2e-7), and it has no branches: erff takes both of its sides in most waves, some sixty
// instructions a value, which a block of four waves with 64 values a lane has nothing to hide behind (24 us a round of blocks).
// NaN stays NaN, inf stays inf, -inf gives NaN, as the other form does.
__device__ __forceinline__ float gelu_f32(float x) {
  const float a = fminf(fabsf(x), 6.0f);
  float q = -5.265487601491259e-08f;
  q = __builtin_fmaf(q, a, 1.3207697975303745e-06f);
  q = __builtin_fmaf(q, a, -1.4652984646090772e-05f);
  q = __builtin_fmaf(q, a, 9.205499372910708e-05f);
  q = __builtin_fmaf(q, a, -0.0003172860888298601f);
  q = __builtin_fmaf(q, a, 5.163852983969264e-05f);
  q = __builtin_fmaf(q, a, 0.006909135263413191f);
  q = __builtin_fmaf(q, a, -0.05242925509810448f);
  q = __builtin_fmaf(q, a, -0.45922115445137024f);
  q = __builtin_fmaf(q, a, -1.1511045694351196f);
  q = __builtin_fmaf(q, a, 2.5855193541701738e-08f);
  const float t = 0.5f * a * __builtin_amdgcn_exp2f(q);
  return (x > 0.f ? x : x * 0.f) - (fabsf(x) < 6.0f ? t : 0.f);
}

}  // namespace zgr
