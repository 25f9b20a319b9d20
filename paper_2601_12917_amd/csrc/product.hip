// C = epilogue(alpha A B + bias) with fp32 products and sums on the matrix cores, for operands as they lie: fp32 or bf16,
// contiguous along the summed index or along the other one, any sizes.  These are the backward products of fp32 models, of bf16
// models whose token count is no multiple of 64 (the gradients of a block's weights only where the count is long: forward.hip
// takes the others on planes of dy, api.hip's plane_tokens), the five products per head of the attention rule, and the projections of fp32 models that are too
// small for forward.hip's tiles to fill the chip.
//
// Two fp32 operands take the fp32 instruction (v_mfma_f32_16x16x4_f32); with a bf16 operand the products are taken on v_mfma_f32_16x16x32_bf16 (planes.h),
// three of which do the work of eight of the others in three sixteenths of their time: 1024 x 4096 x 231 (the gradient of a weight) 37 us -> 16,
// 231 x 1024 x 4096 (of its input) 25 -> 18, against fp64 off by 8e-8 and 1.7e-7 of the norm (1.4e-7 and 2.1e-7 with the fp32 instruction).
// A wave owns a 64 x 64 piece of C and loads its operands from global memory straight into the instruction's layout: lane
// (i = lane % 16, kg = lane / 16) supplies element i of the free index and kg of the summed one.  A step takes 16 terms,
// k = k0 + 4 kg + s in instruction s (32 terms with planes, k = k0 + 16 u + 4 kg + s as term 4 u + s of the lane's eight).  An operand that is contiguous along k gives a lane four terms of one row per load (tile t: rows
// 16 t + i); one that is contiguous along its other index gives it four rows of one term (tile t: rows 4 i + t).  So every load
// is four elements wide whichever way the operand lies, and nothing passes through LDS but the partial sums of waves that
// share a piece.
// What bounds two fp32 operands is the fp32 matrix rate (157 TFLOP/s): 64 instructions of 32 cycles per step against 8 loads.  The loop holds nothing
// else: addresses are a scalar base plus a lane offset that stays the same (a vector instruction would queue behind the matrix
// instructions of the SIMD's other waves).  The LDS-tiled vector kernel this replaces reached 5 TFLOP/s on 231 tokens of a
// 1024-wide model, where its grid left most of the chip idle (54 of the pass's 60 ms; the whole pass now takes 10).
#include "product.h"
#include "forward.h"
#include "act.h"
#include "planes.h"

namespace zgr {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
struct bf16_t { uint16_t bits; };

__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(bf16_t x) { return __uint_as_float((uint32_t)x.bits << 16); }

__device__ __forceinline__ int uniform(int v) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_readfirstlane(v);
#else
  return v;
#endif
}
// nothing is scheduled across this point
__device__ __forceinline__ void in_this_order() {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_sched_barrier(0);
#endif
}

// Four consecutive elements `byte` + `more` bytes (< 2^32, `more` a scalar) past a scalar base, as loaded.
template <typename T> struct Raw4;
template <> struct Raw4<float> {
  f32x4 v;
  __device__ __forceinline__ void load(const float* base, uint32_t byte, uint32_t more = 0) {
#if defined(__HIP_DEVICE_COMPILE__)
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, 0xFFFFFFFFu, 0x00020000);
    v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, byte, more, 0));
#endif
  }
  __device__ __forceinline__ void set(int q, float x) { v[q] = x; }
  __device__ __forceinline__ f32x4 widen() const { return v; }
};
template <> struct Raw4<bf16_t> {
  u32x2 v;
  __device__ __forceinline__ void load(const bf16_t* base, uint32_t byte, uint32_t more = 0) {
#if defined(__HIP_DEVICE_COMPILE__)
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(base), 0, 0xFFFFFFFFu, 0x00020000);
    v = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(rs, byte, more, 0));
#endif
  }
  __device__ __forceinline__ void set(int q, float x) {          // x came out of bf16
    const uint32_t h = __float_as_uint(x) >> 16;
    v[q >> 1] = (q & 1) ? (v[q >> 1] & 0xFFFFu) | (h << 16) : h;
  }
  __device__ __forceinline__ f32x4 widen() const {
    return f32x4{__uint_as_float(v[0] << 16), __uint_as_float(v[0] & 0xFFFF0000u), __uint_as_float(v[1] << 16), __uint_as_float(v[1] & 0xFFFF0000u)};
  }
};

template <typename T> struct PlanesFor;
template <> struct PlanesFor<float> { typedef PlanesOf<3> type; };
template <> struct PlanesFor<bf16_t> { typedef PlanesOf<1> type; };
template <typename T> using Planes = typename PlanesFor<T>::type;
constexpr uint32_t kOnes = 0x3F803F80u;      // two bf16 ones

// The planes of the TT tiles of an operand.  ALONG_K: loads 2 t and 2 t + 1 brought tile t's terms; otherwise load e brought term e of four tiles.
template <bool ALONG_K, int TT> __device__ __forceinline__ void cut(const Raw4<float>* r, Planes<float>* o) {
#pragma unroll
  for (int t = 0; t < TT; ++t)
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      if (ALONG_K) cut_pair(r[2 * t + (w >> 1)].v[2 * (w & 1)], r[2 * t + (w >> 1)].v[2 * (w & 1) + 1], w, o[t]);
      else         cut_pair(r[2 * w].v[t], r[2 * w + 1].v[t], w, o[t]);
    }
}
template <bool ALONG_K, int TT> __device__ __forceinline__ void cut(const Raw4<bf16_t>* r, Planes<bf16_t>* o) {
#pragma unroll
  for (int t = 0; t < TT; ++t)
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      if (ALONG_K)    o[t].p[0][w] = r[2 * t + (w >> 1)].v[w & 1];
      else if (t & 1) o[t].p[0][w] = high_halves(r[2 * w + 1].v[t >> 1], r[2 * w].v[t >> 1]);
      else            o[t].p[0][w] = low_halves(r[2 * w + 1].v[t >> 1], r[2 * w].v[t >> 1]);
    }
}
__device__ __forceinline__ f32x4 mfma_planes(planes_u32x4 a, planes_u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(planes_bf16x8, a), __builtin_bit_cast(planes_bf16x8, b), c, 0, 0, 0);
}

constexpr int kStep = 16, kStep32 = 32, kWaves = 2048;
struct Yes { static constexpr bool value = true; };
struct No { static constexpr bool value = false; };

struct KernelArgs {
  const void* A; const void* B; float* C; float* a_sums;
  int64_t lda, ldb, ldc;
  int M, N, K;
  float alpha;
  int epilogue; const float* bias;
  int split;                 // waves that share a piece of C, each taking every split-th step: 1 (a block is 2 x 2 pieces), 4 or 8 (one piece)
  int k_part;                // terms of one part of the sum: part z of a batch writes its result at C + z c_part (a_sums + z M)
  int64_t c_part;
  int parts, zdiv;           // a block's z: batch z / parts, part z % parts
  int64_t bias_outer;
  int64_t a_outer, a_inner, b_outer, b_inner, c_outer, c_inner;
};

__device__ __forceinline__ void finish(float* c, float v, int epilogue, const float* bias, int j) {
  if (bias) v += bias[j];
  switch (epilogue) {                                            // uniform
    case EPI_GELU:  *c = gelu_f32(v); break;
    case EPI_RELU:  *c = fmaxf(v, 0.f); break;
    case EPI_RESID: *c += v; break;
    default:        *c = v; break;
  }
}

// NEAR: the byte offsets of a step fit 32 bits, an operand contiguous along its free index has at least four entries of it, and bf16
// operands lie on 4 bytes; the other form loads element by element.
template <typename TA, typename TB, bool AK, bool BK, bool NEAR, int TT>
__global__ void __launch_bounds__(512, 2) product_kernel(KernelArgs p) {
  static_assert(TT == 4 || (AK && BK), "an operand contiguous along its free index brings four tiles per load");
  constexpr int kTile = 16 * TT, TILES = TT * TT;
  constexpr bool PLANES = NEAR && (Planes<TA>::n == 1 || Planes<TB>::n == 1);
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int lane = threadIdx.x & 63, wave = uniform((int)threadIdx.x >> 6), il = lane & 15, kg = lane >> 4;
  const TA* A = reinterpret_cast<const TA*>(p.A);
  const TB* B = reinterpret_cast<const TB*>(p.B);
  float* C = p.C;
  const int zb = uniform((int)blockIdx.z / p.parts), z = (int)blockIdx.z - zb * p.parts;
  const int zo = uniform(zb / p.zdiv), zi = zb - zo * p.zdiv;
  A += zo * p.a_outer + zi * p.a_inner;
  B += zo * p.b_outer + zi * p.b_inner;
  C += zo * p.c_outer + zi * p.c_inner + z * p.c_part;
  const float* const bias = p.bias ? p.bias + zo * p.bias_outer : nullptr;
  const int k_begin = z * p.k_part, k_end = p.K < k_begin + p.k_part ? p.K : k_begin + p.k_part;
  const bool alone = p.split == 1;
  const int tm = alone ? (int)blockIdx.y * 2 + (wave >> 1) : (int)blockIdx.y, tn = alone ? (int)blockIdx.x * 2 + (wave & 1) : (int)blockIdx.x;
  const int i0 = tm * kTile, j0 = tn * kTile;
  if (alone && (i0 >= p.M || j0 >= p.N)) return;                 // no barrier follows for such a block
  const int share = alone ? 0 : wave;
  // Rows past the end: an operand contiguous along k repeats its last row, the other kind takes its last four entries instead;
  // what comes of them is not stored.
  auto first_i = [&](int q) { const int i = i0 + 4 * q; return NEAR && i > p.M - 4 ? p.M - 4 : i; };
  auto first_j = [&](int q) { const int j = j0 + 4 * q; return NEAR && j > p.N - 4 ? p.N - 4 : j; };
  auto row_i = [&](int t, int q) { const int i = AK ? i0 + 16 * t + q : first_i(q) + t; return i < p.M ? i : p.M - 1; };
  auto row_j = [&](int t, int q) { const int j = BK ? j0 + 16 * t + q : first_j(q) + t; return j < p.N ? j : p.N - 1; };
  constexpr int LA = AK ? 2 * TT : 8, LB = BK ? 2 * TT : 8;      // loads per step
  constexpr int OA = AK ? TT : 8, OB = BK ? TT : 8;              // lane offsets
  uint32_t ao[OA], bo[OB];
#pragma unroll
  for (int t = 0; t < OA; ++t)
    ao[t] = (uint32_t)sizeof(TA) * (AK ? (uint32_t)(row_i(t, il) - i0) * (uint32_t)p.lda + 4u * kg : (uint32_t)(16 * (t >> 2) + 4 * kg + (t & 3)) * (uint32_t)p.lda + (uint32_t)first_i(il));
#pragma unroll
  for (int t = 0; t < OB; ++t)
    bo[t] = (uint32_t)sizeof(TB) * (BK ? (uint32_t)(row_j(t, il) - j0) * (uint32_t)p.ldb + 4u * kg : (uint32_t)(16 * (t >> 2) + 4 * kg + (t & 3)) * (uint32_t)p.ldb + (uint32_t)first_j(il));
  const TA* a_base = AK ? A + (int64_t)i0 * p.lda : A;
  const TB* b_base = BK ? B + (int64_t)j0 * p.ldb : B;
  auto a_at = [&](int i, int k) { return to_f32(AK ? A[(int64_t)i * p.lda + k] : A[(int64_t)k * p.lda + i]); };
  auto b_at = [&](int j, int k) { return to_f32(BK ? B[(int64_t)j * p.ldb + k] : B[(int64_t)k * p.ldb + j]); };
  f32x4 acc[TT][TT], sums[TT];
#pragma unroll
  for (int t = 0; t < TT; ++t) {
    sums[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int n = 0; n < TT; ++n) acc[t][n] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const bool want_sums = !AK && p.a_sums && tn == 0;
  // Two fp32 operands (and what can't be loaded four wide): the fp32 instructions, sixteen terms a step.
  constexpr int EA = AK ? TT : 4, EB = BK ? TT : 4;
  struct Operands { Raw4<TA> a[EA]; Raw4<TB> b[EB]; };
  auto fetch = [&](int k0, Operands& o) {
    if constexpr (NEAR) {
      const TA* ak = a_base + (AK ? (int64_t)k0 : k0 * p.lda);
      const TB* bk = b_base + (BK ? (int64_t)k0 : k0 * p.ldb);
#pragma unroll
      for (int t = 0; t < EA; ++t) o.a[t].load(ak, ao[t]);
#pragma unroll
      for (int t = 0; t < EB; ++t) o.b[t].load(bk, bo[t]);
    }
  };
  // x[t] holds what load t brought: tile t, terms s (contiguous along k) or term t, tiles s
  auto multiply4 = [&](const f32x4 (&a)[EA], const f32x4 (&b)[EB], auto with_sums) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int t = 0; t < TT; ++t) {
        const float av = AK ? a[t][s] : a[s][t];
#pragma unroll
        for (int n = 0; n < TT; ++n) acc[t][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, BK ? b[n][s] : b[s][n], acc[t][n], 0, 0, 0);
        if (decltype(with_sums)::value) sums[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, 1.0f, sums[t], 0, 0, 0);
      }
  };
  auto loop = [&](auto with_sums) {
    auto multiply = [&](const Operands& o) {
      f32x4 a[EA], b[EB];
#pragma unroll
      for (int t = 0; t < EA; ++t) a[t] = o.a[t].widen();
#pragma unroll
      for (int t = 0; t < EB; ++t) b[t] = o.b[t].widen();
      multiply4(a, b, with_sums);
    };
    const int stride = p.split * kStep, full = k_begin + (k_end - k_begin) / kStep * kStep;
    int k0 = k_begin + share * kStep;
    const int steps = NEAR ? uniform(k0 < full ? (full - k0 + stride - 1) / stride : 0) : 0;
    if (steps > 0) {
      Operands o0, o1;
      auto step = [&](int i) { return k0 + (i < steps ? i : steps - 1) * stride; };      // behind the last step it is read again
      int i = 0;
      if (steps & 1) { fetch(k0, o0); multiply(o0); i = 1; }
      fetch(step(i), o0);
      for (; i < steps; i += 2) {
        fetch(step(i + 1), o1);
        in_this_order();
        multiply(o0);
        in_this_order();
        fetch(step(i + 2), o0);
        in_this_order();
        multiply(o1);
        in_this_order();
      }
      k0 += steps * stride;
    }
    // the terms left over (the wave whose turn it is; every step in the element-by-element form): zeros past the end
    for (; k0 < k_end; k0 += stride) {
      f32x4 a[EA], b[EB];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
#pragma unroll
        for (int t = 0; t < EA; ++t) { const int k = k0 + 4 * kg + (AK ? s : t); a[t][s] = k < k_end ? a_at(row_i(AK ? t : s, il), k) : 0.f; }
#pragma unroll
        for (int t = 0; t < EB; ++t) { const int k = k0 + 4 * kg + (BK ? s : t); b[t][s] = k < k_end ? b_at(row_j(BK ? t : s, il), k) : 0.f; }
      }
      multiply4(a, b, with_sums);
    }
  };
  // Those of the wave's shares again, entry by entry (sums of the next form that are not finite).
  auto loop_again = [&](auto with_sums) {
    for (int k0 = k_begin + share * kStep32; k0 < k_end; k0 += p.split * kStep32)
#pragma unroll 1
      for (int ks = k0; ks < k0 + kStep32 && ks < k_end; ks += 16) {
        float a[4][TT], b[4][TT];                                // zeros past the end
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int t = 0; t < TT; ++t) {
            const int k = ks + 4 * kg + q;
            a[q][t] = k < k_end ? a_at(row_i(t, il), k) : 0.f;
            b[q][t] = k < k_end ? b_at(row_j(t, il), k) : 0.f;
          }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int t = 0; t < TT; ++t) {
#pragma unroll
            for (int n = 0; n < TT; ++n) acc[t][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[q][t], b[q][n], acc[t][n], 0, 0, 0);
            if (decltype(with_sums)::value) sums[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[q][t], 1.0f, sums[t], 0, 0, 0);
          }
      }
  };
  // The bf16 instructions on the operands' planes.
  auto loop_planes = [&](auto with_sums) {
    Raw4<TA> ra[LA];
    Raw4<TB> rb[LB];
    Planes<TA> pa[TT];
    Planes<TB> pb[TT];
    auto fetch_a = [&](int k0) {
      const TA* ak = a_base + (AK ? (int64_t)k0 : k0 * p.lda);
#pragma unroll
      for (int t = 0; t < LA; ++t) ra[t].load(ak, ao[AK ? t >> 1 : t], AK ? 16u * (t & 1) * sizeof(TA) : 0u);
    };
    auto fetch_b = [&](int k0) {
      const TB* bk = b_base + (BK ? (int64_t)k0 : k0 * p.ldb);
#pragma unroll
      for (int t = 0; t < LB; ++t) rb[t].load(bk, bo[BK ? t >> 1 : t], BK ? 16u * (t & 1) * sizeof(TB) : 0u);
    };
    auto multiply = [&]() {
      for_terms<Planes<TA>::n, Planes<TB>::n>([&](int x, int y) {
#pragma unroll
        for (int t = 0; t < TT; ++t)
#pragma unroll
          for (int n = 0; n < TT; ++n) acc[t][n] = mfma_planes(pa[t].p[x], pb[n].p[y], acc[t][n]);
      });
      if (decltype(with_sums)::value)
#pragma unroll
        for (int x = Planes<TA>::n - 1; x >= 0; --x)
#pragma unroll
          for (int t = 0; t < TT; ++t) sums[t] = mfma_planes(pa[t].p[x], planes_u32x4{kOnes, kOnes, kOnes, kOnes}, sums[t]);
    };
    const int stride = p.split * kStep32, full = k_begin + (k_end - k_begin) / kStep32 * kStep32;
    int k0 = k_begin + share * kStep32;
    const int steps = uniform(k0 < full ? (full - k0 + stride - 1) / stride : 0);
    if (steps > 0) {
      fetch_a(k0);
      fetch_b(k0);
      for (int i = 0; i < steps; ++i) {
        const int next = k0 + (i + 1 < steps ? i + 1 : i) * stride;      // behind the last step it is read again
        cut<AK, TT>(ra, pa);
        in_this_order();
        fetch_a(next);
        in_this_order();
        cut<BK, TT>(rb, pb);
        in_this_order();
        fetch_b(next);
        in_this_order();
        multiply();
      }
      k0 += steps * stride;
    }
    if (k0 < k_end) {                                            // the terms left over (the wave whose turn it is): zeros past the end
      auto k_of = [&](int e) { return k0 + 16 * (e >> 2) + 4 * kg + (e & 3); };
#pragma unroll
      for (int t = 0; t < LA; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) { const int k = AK ? k_of(4 * (t & 1) + q) : k_of(t); ra[t].set(q, k < k_end ? a_at(row_i(AK ? t >> 1 : q, il), k) : 0.f); }
#pragma unroll
      for (int t = 0; t < LB; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) { const int k = BK ? k_of(4 * (t & 1) + q) : k_of(t); rb[t].set(q, k < k_end ? b_at(row_j(BK ? t >> 1 : q, il), k) : 0.f); }
      cut<AK, TT>(ra, pa);
      cut<BK, TT>(rb, pb);
      multiply();
    }
  };
  auto sum_up = [&](auto with_sums) {
    if constexpr (!PLANES) {
      loop(with_sums);
    } else {
      loop_planes(with_sums);
      if (Planes<TA>::n * Planes<TB>::n == 1) return;
      // An infinite operand has NaN in its second plane, and times another operand's zero planes it makes NaN of what fp32 products leave
      // infinite.  Such sums are not finite either way: they are taken again by the fp32 instructions.
      float zero = 0.f;
#pragma unroll
      for (int t = 0; t < TT; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
#pragma unroll
          for (int n = 0; n < TT; ++n) zero = __builtin_fmaf(acc[t][n][v], 0.f, zero);
          zero = __builtin_fmaf(sums[t][v], 0.f, zero);
        }
      if (!__ballot(!(zero == 0.f))) return;
#pragma unroll
      for (int t = 0; t < TT; ++t) {
        sums[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int n = 0; n < TT; ++n) acc[t][n] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      loop_again(with_sums);
    }
  };
  if constexpr (!AK) { if (want_sums) sum_up(Yes{}); else sum_up(No{}); }
  else sum_up(No{});
  // waves that share the piece add up in a fixed order (8: 0+4, 1+5, 2+6, 3+7; then 0+2, 1+3; then 0+1)
  const bool four = TT == 4 && p.split == 4;                     // summed when they are stored, below
  if (!alone && !four) {
    for (int half = p.split >> 1; half >= 1; half >>= 1) {
      __syncthreads();
      if (wave >= half && wave < 2 * half)
#pragma unroll
        for (int t = 0; t < TT; ++t)
#pragma unroll
          for (int n = 0; n < TT; ++n) *reinterpret_cast<f32x4*>(lds + (((wave - half) * TILES + t * TT + n) * 64 + lane) * 4) = acc[t][n];
      __syncthreads();
      if (wave < half)
#pragma unroll
        for (int t = 0; t < TT; ++t)
#pragma unroll
          for (int n = 0; n < TT; ++n) acc[t][n] += *reinterpret_cast<const f32x4*>(lds + ((wave * TILES + t * TT + n) * 64 + lane) * 4);
      if (want_sums) {                                           // uniform over the block
        __syncthreads();
        if (wave >= half && wave < 2 * half)
#pragma unroll
          for (int t = 0; t < TT; ++t) *reinterpret_cast<f32x4*>(lds + (((wave - half) * TT + t) * 64 + lane) * 4) = sums[t];
        __syncthreads();
        if (wave < half)
#pragma unroll
          for (int t = 0; t < TT; ++t) sums[t] += *reinterpret_cast<const f32x4*>(lds + ((wave * TT + t) * 64 + lane) * 4);
      }
    }
  }
  // lane (il, kg) holds column il of a tile and its rows 4 kg + v.  A lane that took entries before its own stores its own only.
  auto store_sums = [&](int t, const f32x4& sum) {
    if (il == 0)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = first_i(4 * kg + v) + t;
        if (i >= i0 + 4 * (4 * kg + v) && i < p.M) p.a_sums[(int64_t)z * p.M + i] = sum[v];
      }
  };
  if (want_sums && !four && share == 0)
#pragma unroll
    for (int t = 0; t < TT; ++t) store_sums(t, sums[t]);
  // Rows 4 kg + v0 .. 4 kg + v0 + count - 1 of the tiles (t, 0 .. TT - 1).  A whole piece without an epilogue takes no condition per
  // entry, and 16-byte stores where a lane's columns are consecutive.
  const float alpha = p.alpha;
  const bool plain = !bias && (p.epilogue == EPI_STORE || p.epilogue == EPI_F32) && i0 + kTile <= p.M && j0 + kTile <= p.N;
  auto row_of = [&](int t, int v) { return AK ? i0 + 16 * t + 4 * kg + v : first_i(4 * kg + v) + t; };
  auto store = [&](int t, int v, const float (&x)[TT]) {
    const int i = row_of(t, v);
    if (plain) {
      float* c = C + (int64_t)i * p.ldc + j0;
      if constexpr (BK) {
#pragma unroll
        for (int n = 0; n < TT; ++n) c[16 * n + il] = alpha * x[n];
      } else {
        typedef f32x4 __attribute__((aligned(4))) f32x4_u;
        *reinterpret_cast<f32x4_u*>(c + 4 * il) = f32x4{alpha * x[0], alpha * x[1], alpha * x[2], alpha * x[3]};
      }
      return;
    }
    if (i >= p.M || (!AK && i < i0 + 4 * (4 * kg + v))) return;
#pragma unroll
    for (int n = 0; n < TT; ++n) {
      const int j = BK ? j0 + 16 * n + il : first_j(il) + n;
      if (j < p.N && (BK || j >= j0 + 4 * il)) finish(C + (int64_t)i * p.ldc + j, alpha * x[n], p.epilogue, bias, j);
    }
  };
  if (alone) {
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        float x[TT];
#pragma unroll
        for (int n = 0; n < TT; ++n) x[n] = acc[t][n][v];
        store(t, v, x);
      }
  } else if (four) {
    // four waves: all partial sums side by side in LDS, wave t adds up and stores the 16 rows of tiles (t, 0 .. 3)
    auto part = [&](int w, int n) -> f32x4& { return *reinterpret_cast<f32x4*>(lds + ((w * TILES + n) * 64 + lane) * 4); };
    auto added = [&](int n) { return (part(0, n) + part(1, n)) + (part(2, n) + part(3, n)); };
    if (want_sums) {                                             // uniform over the block
#pragma unroll
      for (int t = 0; t < TT; ++t) part(wave, t) = sums[t];
      __syncthreads();
      store_sums(wave, added(wave));
      __syncthreads();
    }
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
      for (int n = 0; n < TT; ++n) part(wave, t * TT + n) = acc[t][n];
    __syncthreads();
    f32x4 r[TT];
#pragma unroll
    for (int n = 0; n < TT; ++n) r[n] = added(wave * TT + n);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      float x[TT];
#pragma unroll
      for (int n = 0; n < TT; ++n) x[n] = r[n][v];
      store(wave, v, x);
    }
  } else {                                                       // the waves share out the rows
    __syncthreads();
    if (wave == 0)
#pragma unroll
      for (int t = 0; t < TT; ++t)
#pragma unroll
        for (int n = 0; n < TT; ++n) *reinterpret_cast<f32x4*>(lds + ((t * TT + n) * 64 + lane) * 4) = acc[t][n];
    __syncthreads();
    const int count = 4 * TT / p.split;
    for (int r = wave * count; r < (wave + 1) * count; ++r) {
      float x[TT];
#pragma unroll
      for (int n = 0; n < TT; ++n) x[n] = lds[(((r >> 2) * TT + n) * 64 + lane) * 4 + (r & 3)];
      store(r >> 2, r & 3, x);
    }
  }
}

// C[i][j] = epilogue(alpha (part 0 + part 1 + ...)[i][j] + bias[j]), a_sums likewise without alpha: the parts in their order; a row of blocks per batch
__global__ void __launch_bounds__(256) product_sum_kernel(const float* __restrict__ part, int parts, int64_t n, int N, float* __restrict__ C, int64_t ldc, float alpha,
                                                          const float* __restrict__ sum_part, int M, float* __restrict__ a_sums, int epilogue, const float* __restrict__ bias, int64_t c_outer, int64_t bias_outer) {
  part += (int64_t)blockIdx.y * parts * n;
  C += (int64_t)blockIdx.y * c_outer;
  if (bias) bias += (int64_t)blockIdx.y * bias_outer;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n + (a_sums ? M : 0); e += (int64_t)gridDim.x * 256) {
    const float* src = e < n ? part + e : sum_part + (e - n);
    const int64_t stride = e < n ? n : M;
    float v = 0.f;
#pragma unroll 4
    for (int z = 0; z < parts; ++z) v += src[(int64_t)z * stride];
    if (e < n) finish(C + e / N * ldc + e % N, alpha * v, epilogue, bias, (int)(e % N)); else a_sums[e - n] = v;
  }
}

template <typename TA, typename TB, bool AK, bool BK, int TT = 4>
hipError_t launch_t(const KernelArgs& k, bool near, dim3 grid, hipStream_t s) {
  const unsigned threads = k.split == 8 ? 512 : 256;
  const size_t lds = k.split == 1 ? 0 : (size_t)(TT == 4 && k.split == 4 ? 4 : k.split / 2) * TT * TT * 64 * 16;       // 64 KB at most
  if (near) hipLaunchKernelGGL((product_kernel<TA, TB, AK, BK, true, TT>), grid, dim3(threads), lds, s, k);
  else      hipLaunchKernelGGL((product_kernel<TA, TB, AK, BK, false, TT>), grid, dim3(threads), lds, s, k);
  return hipGetLastError();
}

// Whether an operand's step can be loaded four elements wide with 32-bit offsets (see product_kernel).
bool near_operand(const void* p, int dtype, bool along_k, int64_t ld, int n, int64_t outer, int64_t inner) {
  const int64_t es = dtype == 1 ? 2 : 4;
  if ((along_k ? 64 : 32) * ld * es + (along_k ? 64 : (int64_t)n * es) >= ((int64_t)1 << 32)) return false;
  if (!along_k && n < 4) return false;
  if (dtype == 1 && (((uintptr_t)p & 3) || (ld & 1) || (outer & 1) || (inner & 1) || (!along_k && (n & 1)))) return false;
  return true;
}

}  // namespace

hipError_t launch_product(const ProductArgs& p, hipStream_t s) {
  if (p.M < 1 || p.N < 1 || p.batches < 1) return hipSuccess;
  if (p.K < 0 || p.batches > 65535 || p.zdiv < 1 || (p.a_sums && (p.a_k || p.a_dtype != 0 || p.batches != 1))) return hipErrorInvalidValue;
  if (p.parts_left && (p.batches != 1 || p.row_blocks != 1 || p.alpha != 1.0f || p.epilogue != EPI_STORE || p.bias || p.a_sums || p.ldc != p.N)) return hipErrorInvalidValue;
  if (p.models < 1 || p.batches % p.models || p.row_blocks < 1 || p.M % p.row_blocks || (p.row_blocks > 1 && (p.batches != 1 || p.a_k))) return hipErrorInvalidValue;
  const int rows = p.M / p.row_blocks;
  const int64_t tiles = (((int64_t)rows + 63) / 64) * (((int64_t)p.N + 63) / 64) * (p.batches / p.models);
  const int steps = (p.K + kStep - 1) / kStep;
  // Two fp32 operands.  Two waves per SIMD hide each other's loads (one: 10.35 ms for the backward pass of a 24-block, 1024-wide encoder on 231
  // tokens, two: 10.06).  With fewer pieces than that four waves share each, or eight where blocks of four would leave CUs with one (385 x 768 x 768:
  // 20.4 us with eight, 385 x 3072 x 768: 36 with four, 40 with eight).  Where that is still too few the sum is split over
  // blocks as well, each share at least eight steps (385 x 768 x 3072: 55 us undivided, 33 in three parts).
  // With planes a share of the sum takes a third of the time and adding up costs the same: four waves a piece, and half the blocks
  // (231 x 1024 x 4096: 20 us with eight, 18 with four waves and four parts; 231 x 4096 x 1024: 24 in two parts, 16 undivided).  (A reader that adds the parts up is
  // no reason for more of them: eight of that first product 16 us, four 13.)
  const bool planes = p.a_dtype == 1 || p.b_dtype == 1;
  int split = tiles >= kWaves || steps < 4 ? 1 : (planes || tiles >= 320 || steps < 32 ? 4 : 8);
  int parts = 1;
  const bool few = p.batches == p.models && p.zdiv == 1;      // one product, or that of two models
  if (few && p.scratch && split > 1) {
    int64_t z = (planes ? kWaves / 2 : kWaves) / (tiles * split);
    const int64_t room = (int64_t)(p.scratch_floats / ((size_t)rows * ((size_t)p.N + 1) * (size_t)p.batches));
    if (z > steps / (8 * split)) z = steps / (8 * split);
    if (z > room) z = room;
    if (z > 1) parts = (int)z;
  }
  if (p.row_blocks > 1 && parts > 1 && (size_t)parts * p.M * ((size_t)p.N + 1) > p.scratch_floats) {      // no room for all blocks' parts: one after the other
    ProductArgs q = p;
    q.M = rows; q.row_blocks = 1;
    for (int b = 0; b < p.row_blocks; ++b) {
      q.A = reinterpret_cast<const char*>(p.A) + (size_t)b * rows * (p.a_dtype == 1 ? 2 : 4);
      q.C = p.C + (int64_t)b * rows * p.ldc;
      q.a_sums = p.a_sums ? p.a_sums + (int64_t)b * rows : nullptr;
      const hipError_t e = launch_product(q, s);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  // What is left with few pieces and an undivided sum takes 32 x 32 pieces, four times the blocks (512 x 128 x 512: 8.0 us against 16.6,
  // 385 x 768 x 768: 15.9 against 20.4; at 252 pieces, 385 x 2304 x 768, they are slower: 28 against 22).
  const bool small = p.a_k && p.b_k && p.a_dtype == 0 && p.b_dtype == 0 && few && tiles <= 128 && parts == 1;
  if (small && split > 1) split = 4;
  const int tile = small ? 32 : 64;
  const int64_t tm = ((int64_t)p.M + tile - 1) / tile, tn = ((int64_t)p.N + tile - 1) / tile;
  if (tm > 65535) return hipErrorInvalidValue;
  KernelArgs k{};
  k.A = p.A; k.B = p.B; k.lda = p.lda; k.ldb = p.ldb; k.M = p.M; k.N = p.N; k.K = p.K; k.split = split;
  k.parts = parts; k.zdiv = p.zdiv; k.bias_outer = p.bias_outer;
  k.a_outer = p.a_outer; k.a_inner = p.a_inner; k.b_outer = p.b_outer; k.b_inner = p.b_inner; k.c_outer = p.c_outer; k.c_inner = p.c_inner;
  k.k_part = (steps + parts - 1) / parts * kStep;
  k.k_part = (k.k_part + kStep32 - 1) / kStep32 * kStep32;
  if (k.k_part < 1) k.k_part = 1;
  const int64_t n = (int64_t)p.M * p.N;
  float* sum_part = p.scratch + (int64_t)parts * p.batches * n;
  if (parts > 1) { k.C = p.scratch; k.ldc = p.N; k.alpha = 1.0f; k.epilogue = EPI_STORE; k.c_part = n; k.c_outer = parts * n; k.c_inner = 0; k.a_sums = p.a_sums ? sum_part : nullptr; }
  else           { k.C = p.C; k.ldc = p.ldc; k.alpha = p.alpha; k.epilogue = p.epilogue; k.bias = p.bias; k.a_sums = p.a_sums; }
  const bool near = near_operand(p.A, p.a_dtype, p.a_k, p.lda, p.M, p.a_outer, p.a_inner) && near_operand(p.B, p.b_dtype, p.b_k, p.ldb, p.N, p.b_outer, p.b_inner);
  const dim3 grid((unsigned)(split == 1 ? (tn + 1) / 2 : tn), (unsigned)(split == 1 ? (tm + 1) / 2 : tm), (unsigned)(p.batches * parts));
  hipError_t e = hipErrorInvalidValue;
  const int form = (p.a_dtype << 3) | (p.b_dtype << 2) | ((p.a_k ? 1 : 0) << 1) | (p.b_k ? 1 : 0);
  switch (form) {
    case 0b0010: e = launch_t<float, float, true, false>(k, near, grid, s); break;
    case 0b0110: e = launch_t<float, bf16_t, true, false>(k, near, grid, s); break;
    case 0b0000: e = launch_t<float, float, false, false>(k, near, grid, s); break;
    case 0b0100: e = launch_t<float, bf16_t, false, false>(k, near, grid, s); break;
    case 0b0011: e = small ? launch_t<float, float, true, true, 2>(k, near, grid, s) : launch_t<float, float, true, true>(k, near, grid, s); break;
    case 0b0111: e = launch_t<float, bf16_t, true, true>(k, near, grid, s); break;
    case 0b1111: e = launch_t<bf16_t, bf16_t, true, true>(k, near, grid, s); break;
    default: break;
  }
  if (p.parts_left) *p.parts_left = parts;
  if (e != hipSuccess || parts == 1 || p.parts_left) return e;
  const int64_t total = n + (p.a_sums ? p.M : 0);
  hipLaunchKernelGGL(product_sum_kernel, dim3((unsigned)(total / 256 + 1 < 2048 ? total / 256 + 1 : 2048), (unsigned)p.batches), dim3(256), 0, s, p.scratch, parts, n, p.N, p.C, p.ldc, p.alpha, sum_part, p.M, p.a_sums, p.epilogue, p.bias, p.c_outer, p.bias_outer);
  return hipGetLastError();
}

}  // namespace zgr
