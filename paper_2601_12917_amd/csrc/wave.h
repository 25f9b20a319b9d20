// Sums and maxima over the 64 lanes of a wave, in every lane, without LDS: the steps of a butterfly (lane ^ 32, 16, 8, 4, 2, 1) on the exchanges that vector
// instructions can make, so the terms meet in the butterfly's order.  Step 4 takes the lane four further on in its row of 16: after step 8 that one holds
// what lane ^ 4 does.  Through LDS (__shfl_xor) a step takes some 100 cycles of latency and a wave has nothing to hide them behind: six steps
// 0.3 us, which a LayerNorm does twice and its rule in the backward pass four times.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace zgr {

#if defined(__HIP_DEVICE_COMPILE__)
typedef uint32_t wave_u32x2 __attribute__((ext_vector_type(2)));
// f of the lane's value and of the value in lane ^ 32
template <typename F> __device__ __forceinline__ float wave_step32(float v, F f) {
  const wave_u32x2 r = __builtin_bit_cast(wave_u32x2, __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false));
  return f(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
template <typename F> __device__ __forceinline__ float wave_step16(float v, F f) {
  const wave_u32x2 r = __builtin_bit_cast(wave_u32x2, __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false));
  return f(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
template <int CTRL, typename F> __device__ __forceinline__ float wave_step(float v, F f) {
  return f(v, __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), CTRL, 0xF, 0xF, true)));
}
template <typename F> __device__ __forceinline__ float wave_all(float v, F f) {
  v = wave_step32(v, f);
  v = wave_step16(v, f);
  v = wave_step<0x128>(v, f);      // row_ror:8
  v = wave_step<0x124>(v, f);      // row_ror:4
  v = wave_step<0x4E>(v, f);       // quad_perm [2, 3, 0, 1]
  return wave_step<0xB1>(v, f);    // quad_perm [1, 0, 3, 2]
}
__device__ __forceinline__ float wave_sum(float v) { return wave_all(v, [](float x, float y) { return x + y; }); }
__device__ __forceinline__ float wave_max(float v) { return wave_all(v, [](float x, float y) { return fmaxf(x, y); }); }
#else
__device__ __forceinline__ float wave_sum(float v) { return v; }      // the host's pass over device code
__device__ __forceinline__ float wave_max(float v) { return v; }
#endif

}  // namespace zgr
