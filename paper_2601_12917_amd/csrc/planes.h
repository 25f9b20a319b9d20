// fp32 products on the bf16 matrix instructions.  An fp32 number is the sum of three bf16 numbers exactly: its mantissa cut into pieces of
// eight bits ("planes").  The product of two bf16 numbers is exact in fp32, so with a bf16 factor three such products are the whole product,
// and that of two fp32 numbers is the sum of nine, of which the three smallest are left out.  The sums are the instruction's, in fp32.  Six bf16
// instructions take 0.38 of the time of the fp32 ones they replace, three 0.19.
// Two fp32 factors: planes are cut by rounding.  Plane 1 of a number in [1, 2) is then at most 2^-8 and plane 2 at most 2^-17, what is left out at most
// 2^-24 of the product, and its sign is anyone's.  (Cut by truncation it is up to 2^-21, always with the sign of the product: sums of positive products came
// out 2^-24.5 too small, and where the sum has grown so large that a step's share of the smaller planes is under half its last place, all of that share was
// lost: 2048 x 2048 x 2048 factors of [1, 2) were off by 48 2^-24 of the norm, 4096 x 1024 x 8192 by 269; the fp32 instruction 11 and 23.)
// With a bf16 factor: the first plane by truncation, under which it doesn't overflow, the second by rounding, so that the third's signs mix (the sums of 8191 positive
// products of 2048 x 4096 were off by 90 2^-24 with both truncated; the fp32 instruction 23).
// Off from fp64 no further than the fp32 instructions, whose every fourth (16x16x4) or second (32x32x2) term is
// followed by a rounding of the sum, here every thirty-second (sixteenth) of each plane (figures where it is used).
// An infinite factor has NaN in its second plane, one that rounds up to infinity (above 3.39e38) in its third; sums that come out not finite have to be
// taken again by the fp32 instructions.  The instruction takes a subnormal plane as zero: entries are exact to 2^-126, so numbers below 2^-103
// lose their last plane (factors of 2^-115 times factors of 2^100: off by 37 2^-24).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace zgr {

typedef float planes_f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t planes_u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 planes_bf16x8 __attribute__((ext_vector_type(8)));

// Eight terms of one row (or column) as bf16 operands of the matrix instruction, the largest plane first.
template <int N> struct PlanesOf { static constexpr int n = N; planes_u32x4 p[N]; };

__device__ __forceinline__ uint32_t high_halves(uint32_t x1, uint32_t x0) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_perm(x1, x0, 0x07060302u);
#else
  return (x1 & 0xFFFF0000u) | (x0 >> 16);
#endif
}
__device__ __forceinline__ uint32_t low_halves(uint32_t x1, uint32_t x0) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_perm(x1, x0, 0x05040100u);
#else
  return (x1 << 16) | (x0 & 0xFFFFu);
#endif
}
typedef float planes_f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 planes_bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t round_pair(float x0, float x1) { return __builtin_bit_cast(uint32_t, __builtin_convertvector(planes_f32x2{x0, x1}, planes_bf16x2)); }
__device__ __forceinline__ float low_float(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float high_float(uint32_t u) { return __uint_as_float(u & 0xFFFF0000u); }
// words 1 and 2 of the planes: what is left of the first, rounded, and of that
__device__ __forceinline__ void cut_rest(float r0, float r1, int w, PlanesOf<3>& o) {
  const uint32_t v = round_pair(r0, r1);
  o.p[1][w] = v;
  o.p[2][w] = high_halves(__float_as_uint(r1 - high_float(v)), __float_as_uint(r0 - low_float(v)));
}
// words w of the planes: terms 2 w and 2 w + 1.  For products with a bf16 factor: the first plane by truncation
__device__ __forceinline__ void cut_pair(float x0, float x1, int w, PlanesOf<3>& o) {
  const uint32_t u0 = __float_as_uint(x0), u1 = __float_as_uint(x1);
  o.p[0][w] = high_halves(u1, u0);
  cut_rest(x0 - high_float(u0), x1 - high_float(u1), w, o);
}
// for products of two fp32 factors: by rounding
__device__ __forceinline__ void cut_pair_rounded(float x0, float x1, int w, PlanesOf<3>& o) {
  const uint32_t u = round_pair(x0, x1);
  o.p[0][w] = u;
  cut_rest(x0 - low_float(u), x1 - high_float(u), w, o);
}

// The terms of a product of two factors with NA and NB planes, the smallest first: f(x, y) for plane x of the first factor and y of the second.
template <int NA, int NB, typename F> __device__ __forceinline__ void for_terms(F f) {
#pragma unroll
  for (int order = NA + NB - 2; order >= 0; --order)
#pragma unroll
    for (int x = NA - 1; x >= 0; --x) {
      const int y = order - x;
      if (order <= 2 && y >= 0 && y < NB) f(x, y);
    }
}

}  // namespace zgr
