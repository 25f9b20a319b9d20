// Forward pass L(W; x) for the two loss evaluations of the ZGR step (Sec. 3.2,
// Eq. (11); Sec. 3.1 workflow step 6): pre-LayerNorm transformer blocks with
// softmax attention and erf-GELU feed-forward, next-token cross-entropy through
// the tied embedding (decoder) or a classification head on the first token
// (encoder), and the least-squares loss of a single linear layer.
//
// Storage type T of weights and GEMM inputs is fp32 or bf16; accumulation, the
// residual stream, LayerNorm, softmax and the loss are fp32, the final mean fp64.
#include "forward.h"
#include "act.h"
#include "planes.h"
#include "wave.h"
#include "product.h"
#include <algorithm>
#include <atomic>

namespace zgr {

namespace {

struct bf16_t { uint16_t bits; };
__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(bf16_t x) { return __uint_as_float((uint32_t)x.bits << 16); }
__device__ __forceinline__ void from_f32(float x, float& o) { o = x; }
__device__ __forceinline__ void from_f32(float x, bf16_t& o) {     // round to nearest, ties to even (v_cvt_pk_bf16_f32)
  const __bf16 h = static_cast<__bf16>(x);
  o.bits = __builtin_bit_cast(uint16_t, h);
}

// block of 256 threads: reduce across the 4 waves through LDS
__device__ __forceinline__ float block_sum(float v, float* red) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return red[0] + red[1] + red[2] + red[3];
}
__device__ __forceinline__ float block_max(float v, float* red) {
  v = wave_max(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}

// A parameter of the model a row belongs to: with two models (Twin) the second one's parameters lie w bytes behind the first's.
template <typename T> __device__ __forceinline__ const T* of_model(const T* p, bool second, int64_t w) {
  return reinterpret_cast<const T*>(reinterpret_cast<const unsigned char*>(p) + (second ? w : 0));
}
__device__ __forceinline__ int uniform_of(int v) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_readfirstlane(v);
#else
  return v;
#endif
}

// ------------------------------------------------------------------ embedding
// With targets the rows' next tokens as well (those of one model): row m = b seq + t predicts tok[m + 1] for t < seq - 1, -1 otherwise.
template <typename T>
__global__ void __launch_bounds__(256) embed_kernel(const int32_t* __restrict__ tok, const T* __restrict__ E, const T* __restrict__ Pe,
                                                    float* __restrict__ x, int M, int seq, int d, int vocab, int64_t w, int32_t* __restrict__ targets) {
  const int m = blockIdx.x, mt = m < M ? m : m - M;
  if (targets && threadIdx.x == 0 && m < M) {
    int t = -1;
    if (m % seq < seq - 1) { t = tok[m + 1]; t = t < 0 ? 0 : (t >= vocab ? vocab - 1 : t); }   // the embedding's clamp
    targets[m] = t;
  }
  int t = tok[mt];
  t = t < 0 ? 0 : (t >= vocab ? vocab - 1 : t);
  const T* e = of_model(E, m >= M, w) + (size_t)t * d;
  const T* p = of_model(Pe, m >= M, w) + (size_t)(mt % seq) * d;
  for (int i = threadIdx.x; i < d; i += 256) x[(size_t)m * d + i] = to_f32(e[i]) + to_f32(p[i]);
}

// ------------------------------------------------------------------ LayerNorm (one block per row)
template <typename T>
__global__ void __launch_bounds__(256) layernorm_kernel(const float* x, const T* __restrict__ g, const T* __restrict__ b,
                                                        T* __restrict__ out, int d, float eps, float* xout, int M, int64_t w) {
  __shared__ float red[4];
  g = of_model(g, (int)blockIdx.x >= M, w); b = of_model(b, (int)blockIdx.x >= M, w);
  const float* row = x + (size_t)blockIdx.x * d;
  float s = 0.f;
  for (int i = threadIdx.x; i < d; i += 256) s += row[i];
  const float mu = block_sum(s, red) / d;
  float v = 0.f;
  for (int i = threadIdx.x; i < d; i += 256) { const float t = row[i] - mu; v += t * t; }
  const float rstd = 1.0f / sqrtf(block_sum(v, red) / d + eps);
  T* o = out + (size_t)blockIdx.x * d;
  float* xo = xout ? xout + (size_t)blockIdx.x * d : nullptr;      // may be the row itself: an element is read, then written, by one thread
  for (int i = threadIdx.x; i < d; i += 256) {
    const float y = (row[i] - mu) * rstd * to_f32(g[i]) + to_f32(b[i]);
    from_f32(y, o[i]);
    if (xo) xo[i] = y;
  }
}

// Row held in registers (d % 4 == 0, d <= 8192): one read of x, float4 loads, packed stores.
template <typename T>
__global__ void __launch_bounds__(256) layernorm_reg_kernel(const float* x, const T* __restrict__ g, const T* __restrict__ b,
                                                            T* __restrict__ out, int d, float eps, float* xout, int M, int64_t w) {
  __shared__ float red[4];
  g = of_model(g, (int)blockIdx.x >= M, w); b = of_model(b, (int)blockIdx.x >= M, w);
  constexpr int MAXV = 8;
  const float4* row = reinterpret_cast<const float4*>(x + (size_t)blockIdx.x * d);
  const int nv = d >> 2;
  float4 v[MAXV];
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < MAXV; ++j) {
    const int i = threadIdx.x + 256 * j;
    v[j] = i < nv ? row[i] : make_float4(0.f, 0.f, 0.f, 0.f);
    s += (v[j].x + v[j].y) + (v[j].z + v[j].w);
  }
  const float mu = block_sum(s, red) / d;
  float q = 0.f;
#pragma unroll
  for (int j = 0; j < MAXV; ++j) {
    const int i = threadIdx.x + 256 * j;
    if (i < nv) {
      const float a0 = v[j].x - mu, a1 = v[j].y - mu, a2 = v[j].z - mu, a3 = v[j].w - mu;
      q += (a0 * a0 + a1 * a1) + (a2 * a2 + a3 * a3);
    }
  }
  const float rstd = 1.0f / sqrtf(block_sum(q, red) / d + eps);
  T* o = out + (size_t)blockIdx.x * d;
#pragma unroll
  for (int j = 0; j < MAXV; ++j) {
    const int i = threadIdx.x + 256 * j;
    if (i < nv) {
      struct alignas(sizeof(T) * 4) V4 { T e[4]; };
      const V4 gg = *reinterpret_cast<const V4*>(g + 4 * i), bb = *reinterpret_cast<const V4*>(b + 4 * i);
      V4 r;
      const float4 y = make_float4((v[j].x - mu) * rstd * to_f32(gg.e[0]) + to_f32(bb.e[0]), (v[j].y - mu) * rstd * to_f32(gg.e[1]) + to_f32(bb.e[1]),
                                   (v[j].z - mu) * rstd * to_f32(gg.e[2]) + to_f32(bb.e[2]), (v[j].w - mu) * rstd * to_f32(gg.e[3]) + to_f32(bb.e[3]));
      from_f32(y.x, r.e[0]); from_f32(y.y, r.e[1]); from_f32(y.z, r.e[2]); from_f32(y.w, r.e[3]);
      *reinterpret_cast<V4*>(o + 4 * i) = r;
      if (xout) reinterpret_cast<float4*>(xout + (size_t)blockIdx.x * d)[i] = y;      // the row is in registers: xout may be x
    }
  }
}

// One wave per row (d % 4 == 0, d <= 2048): the row sits in eight float4 per lane, eight 16-byte loads in flight per lane,
// and both reductions stay inside the wave: no LDS, no workgroup barrier.  Four rows per block.
template <typename T>
__global__ void __launch_bounds__(256) layernorm_wave_kernel(const float* x, const T* __restrict__ g, const T* __restrict__ b,
                                                             T* __restrict__ out, int rows, int d, float eps, float* xout, int M, int64_t w) {
  constexpr int MAXV = 8;
  const int lane = threadIdx.x & 63;
  const int row_i = uniform_of(blockIdx.x * 4 + (threadIdx.x >> 6));
  if (row_i >= rows) return;                                       // whole waves leave: no barrier below
  g = of_model(g, row_i >= M, w); b = of_model(b, row_i >= M, w);
  const float4* row = reinterpret_cast<const float4*>(x + (size_t)row_i * d);
  const int nv = d >> 2;
  float4 v[MAXV];
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < MAXV; ++j) {
    const int i = lane + 64 * j;
    v[j] = i < nv ? row[i] : make_float4(0.f, 0.f, 0.f, 0.f);
    s += (v[j].x + v[j].y) + (v[j].z + v[j].w);
  }
  const float mu = wave_sum(s) / d;
  float q = 0.f;
#pragma unroll
  for (int j = 0; j < MAXV; ++j) {
    const int i = lane + 64 * j;
    if (i < nv) {
      const float a0 = v[j].x - mu, a1 = v[j].y - mu, a2 = v[j].z - mu, a3 = v[j].w - mu;
      q += (a0 * a0 + a1 * a1) + (a2 * a2 + a3 * a3);
    }
  }
  const float rstd = 1.0f / sqrtf(wave_sum(q) / d + eps);
  T* o = out + (size_t)row_i * d;
#pragma unroll
  for (int j = 0; j < MAXV; ++j) {
    const int i = lane + 64 * j;
    if (i < nv) {
      struct alignas(sizeof(T) * 4) V4 { T e[4]; };
      const V4 gg = *reinterpret_cast<const V4*>(g + 4 * i), bb = *reinterpret_cast<const V4*>(b + 4 * i);
      V4 r;
      const float4 y = make_float4((v[j].x - mu) * rstd * to_f32(gg.e[0]) + to_f32(bb.e[0]), (v[j].y - mu) * rstd * to_f32(gg.e[1]) + to_f32(bb.e[1]),
                                   (v[j].z - mu) * rstd * to_f32(gg.e[2]) + to_f32(bb.e[2]), (v[j].w - mu) * rstd * to_f32(gg.e[3]) + to_f32(bb.e[3]));
      from_f32(y.x, r.e[0]); from_f32(y.y, r.e[1]); from_f32(y.z, r.e[2]); from_f32(y.w, r.e[3]);
      *reinterpret_cast<V4*>(o + 4 * i) = r;
      if (xout) reinterpret_cast<float4*>(xout + (size_t)row_i * d)[i] = y;          // the row is in registers: xout may be x
    }
  }
}

// ------------------------------------------------------------------ GEMM  C = A W^T (+bias) with epilogues
// A [M,K] and W [N,K] are K-contiguous.
//   EPI_STORE: out T [M,N] = acc + bias
//   EPI_GELU : out T [M,N] = gelu(acc + bias);  EPI_RELU: out T [M,N] = max(acc + bias, 0)
//   EPI_RESID: xres fp32 [M,N] += acc + bias
//   EPI_F32  : outf fp32 [M,N] = acc + bias (bias may be null)
struct GemmEpi { int mode; void* out; const void* bias; const float* resid; };      // resid: what EPI_RESID adds to (out, or another place)
// The values are waited for here, once.  In front of stores under a condition each the compiler waits anew inside every one of them, which then
// sits out the store before it: 16 round trips to memory for a fragment at the ragged edge (the loss of a prompt of 33 tokens, 125M parameters, 24 such
// launches: 721 us, now 691; the fp32 step on 5 x 77 tokens 3.07 ms, now 2.93).
__device__ __forceinline__ void arrived(float (&v)[16]) {
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
  for (int i = 0; i < 16; ++i) asm volatile("" : "+v"(v[i]));
#endif
}
// Bytes from the first model's operands to the second's (Twin); which of the two a block works on is a dimension of the grid.
struct GemmTwin { int64_t a, w, out, bias, tlogit; };
// The tile of a block (and, returned, its model; -1: none).  Consecutive block ids go round-robin to the 8 XCDs, each with its own L2 and about 32
// blocks in flight.  Every XCD gets an equal run of the tiles, which go through each model in bands of four rows of tiles, column by column, so that the
// blocks resident in one L2 share 4 row panels of A and 8 of W.  (Whole super-tiles of 4 x 8 dealt out to the XCDs left half of them idle where there
// are few: 16 x 6 tiles are four of them.  2 x 2048 x 768 x 768 and x 3072 with the residual: 47.6 us -> 26.7 on average, 2 x 4096 x 6144 x 2048:
// 216 -> 173.)
__device__ __forceinline__ int place_of_block(int total) {
  const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3, q = total >> 3, rem = total & 7;
  return local >= q + (xcd < rem ? 1 : 0) ? -1 : xcd * q + (xcd < rem ? xcd : rem) + local;
}
__device__ __forceinline__ void tile_at(int place, int tiles_m, int tiles_n, int& tm, int& tn) {
  constexpr int GM = 4;
  const int band = place / (GM * tiles_n), at = place - band * (GM * tiles_n);
  const int rows = tiles_m - band * GM < GM ? tiles_m - band * GM : GM;
  tn = at / rows;
  tm = band * GM + (at - tn * rows);
}
__device__ __forceinline__ int tile_of_block(int tiles_m, int tiles_n, int models, int& tm, int& tn) {
  const int per_model = tiles_m * tiles_n, place = place_of_block(per_model * models);
  if (place < 0) return -1;
  const int model = place / per_model;
  tile_at(place - model * per_model, tiles_m, tiles_n, tm, tn);
  return model;
}
template <typename T> __device__ __forceinline__ const T* ahead(const T* p, int64_t bytes) {
  return p ? reinterpret_cast<const T*>(reinterpret_cast<const unsigned char*>(p) + bytes) : p;
}
template <typename T> __device__ __forceinline__ T* ahead(T* p, int64_t bytes) {
  return p ? reinterpret_cast<T*>(reinterpret_cast<unsigned char*>(p) + bytes) : p;
}

template <typename T>
__device__ __forceinline__ void epilogue_store(const GemmEpi& ep, int m, int n, int N, float v) {
  if (ep.bias) v += to_f32(reinterpret_cast<const T*>(ep.bias)[n]);
  const size_t o = (size_t)m * N + n;
  switch (ep.mode) {
    case EPI_STORE: from_f32(v, reinterpret_cast<T*>(ep.out)[o]); break;
    case EPI_GELU:  from_f32(gelu_f32(v), reinterpret_cast<T*>(ep.out)[o]); break;
    case EPI_RELU:  from_f32(fmaxf(v, 0.f), reinterpret_cast<T*>(ep.out)[o]); break;
    case EPI_RESID: reinterpret_cast<float*>(ep.out)[o] = ep.resid[o] + v; break;
    default:        reinterpret_cast<float*>(ep.out)[o] = v; break;
  }
}

// fp32 path: 64x64 tile, BK = 16, each thread 4x4 outputs; any M, N, K.
__global__ void __launch_bounds__(256) gemm_f32_kernel(const float* __restrict__ A, const float* __restrict__ W, int M, int N, int K, GemmEpi ep, GemmTwin tw) {
  A = ahead(A, blockIdx.z * tw.a); W = ahead(W, blockIdx.z * tw.w); ep.out = ahead(ep.out, blockIdx.z * tw.out); ep.resid = ahead(ep.resid, blockIdx.z * tw.out); ep.bias = ahead(ep.bias, blockIdx.z * tw.bias);
  __shared__ float As[16][64 + 4], Ws[16][64 + 4];
  const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  float acc[4][4] = {};
  for (int k0 = 0; k0 < K; k0 += 16) {
    for (int i = threadIdx.x; i < 64 * 16; i += 256) {
      const int r = i >> 4, kk = i & 15;
      As[kk][r] = (m0 + r < M && k0 + kk < K) ? A[(size_t)(m0 + r) * K + k0 + kk] : 0.f;
      Ws[kk][r] = (n0 + r < N && k0 + kk < K) ? W[(size_t)(n0 + r) * K + k0 + kk] : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      float a[4], w[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) { a[i] = As[kk][ty * 4 + i]; w[i] = Ws[kk][tx * 4 + i]; }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_fmaf(a[i], w[j], acc[i][j]);
    }
    __syncthreads();
  }
  for (int i = 0; i < 4; ++i)
    for (int j = 0; j < 4; ++j) {
      const int m = m0 + ty * 4 + i, n = n0 + tx * 4 + j;
      if (m < M && n < N) epilogue_store<float>(ep, m, n, N, acc[i][j]);
    }
}

// fp32 path on the matrix cores: v_mfma_f32_32x32x2_f32.  Block tile 64 F x 64 F (F = 1 or 2), BK = 16, four waves
// in 2 x 2, each owning F x F accumulator fragments of 32 x 32.  An fp32 MFMA keeps the matrix pipe busy for 64
// cycles with two floats per lane, so the operands are no bottleneck: the next k-tile travels global -> registers
// while the current one is multiplied and is written to the other LDS buffer afterwards, one barrier per k-tile.
// Four consecutive lanes fetch the 64 contiguous bytes a row contributes to a k-tile.  LDS keeps the rows as they
// are, [row][16 + 4 pad]; the contraction index is split so that a lane's eight values of a k-tile are contiguous
// (the half-wave h takes k = 8 h .. 8 h + 7, in both operands alike): two 16-byte reads per fragment and k-tile,
// conflict-free at a row stride of 20 floats.
// Any M, N; K % 4 == 0 and 16-byte aligned rows (the 64 x 64 kernel above takes what is left).
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// At least two waves per SIMD, i.e. at most 256 registers per lane: the accumulators then live in ordinary vector registers,
// which the MFMA reads and writes directly.  (Allowed 512, the compiler multiplies in the accumulation registers, carries
// the sums round the loop in vector registers and moves all 64 of them back and forth in every k-tile.)
template <int F, int BK>
__global__ void __launch_bounds__(256, 2) gemm_f32_mfma_kernel(const float* __restrict__ A, const float* __restrict__ W, int M, int N, int K, GemmEpi ep, GemmTwin tw) {
  A = ahead(A, blockIdx.z * tw.a); W = ahead(W, blockIdx.z * tw.w); ep.out = ahead(ep.out, blockIdx.z * tw.out); ep.resid = ahead(ep.resid, blockIdx.z * tw.out); ep.bias = ahead(ep.bias, blockIdx.z * tw.bias);
  constexpr int BT = 64 * F, LD = BK + 4, KQ = BK / 4, NV = BT * KQ / 256, HK = BK / 2;
  __shared__ __attribute__((aligned(16))) float As[2][BT][LD], Ws[2][BT][LD];
  const int m0 = blockIdx.y * BT, n0 = blockIdx.x * BT;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, half = lane >> 5;
  const int wm = (wave >> 1) * 32 * F, wn = (wave & 1) * 32 * F;
  // a thread moves NV float4 of each operand per k-tile: row r = idx / KQ, k columns 4 (idx % KQ) .. + 3.  Rows past the
  // matrix are read from its last row (their products are never stored), so only the last, partial k-tile needs a mask.
  float4 ra[NV], rw[NV];
  const float* pa[NV];
  const float* pw[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int idx = tid + 256 * i, r = idx / KQ, kq = idx % KQ;
    pa[i] = A + (size_t)min(m0 + r, M - 1) * K + 4 * kq;
    pw[i] = W + (size_t)min(n0 + r, N - 1) * K + 4 * kq;
  }
  auto fetch = [&](int k0) {
    if (k0 + BK <= K) {
#pragma unroll
      for (int i = 0; i < NV; ++i) { ra[i] = *reinterpret_cast<const float4*>(pa[i] + k0); rw[i] = *reinterpret_cast<const float4*>(pw[i] + k0); }
    } else {
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const bool kin = k0 + 4 * ((tid + 256 * i) % KQ) < K;
        ra[i] = kin ? *reinterpret_cast<const float4*>(pa[i] + k0) : make_float4(0.f, 0.f, 0.f, 0.f);
        rw[i] = kin ? *reinterpret_cast<const float4*>(pw[i] + k0) : make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
  };
  auto stage = [&](int buf) {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int idx = tid + 256 * i, r = idx / KQ, kq = idx % KQ;
      *reinterpret_cast<float4*>(&As[buf][r][4 * kq]) = ra[i];
      *reinterpret_cast<float4*>(&Ws[buf][r][4 * kq]) = rw[i];
    }
  };
  f32x16 acc[F][F];
#pragma unroll
  for (int f = 0; f < F; ++f)
#pragma unroll
    for (int g = 0; g < F; ++g)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[f][g][v] = 0.f;
  // fragments of one k-tile: a lane's HK values of each of its F + F fragment rows
  auto read_frags = [&](int buf, float (&a)[F][HK], float (&w)[F][HK]) {
#pragma unroll
    for (int f = 0; f < F; ++f)
#pragma unroll
      for (int q = 0; q < HK / 4; ++q) {
        const float4 av = *reinterpret_cast<const float4*>(&As[buf][wm + 32 * f + l32][HK * half + 4 * q]);
        const float4 wv = *reinterpret_cast<const float4*>(&Ws[buf][wn + 32 * f + l32][HK * half + 4 * q]);
        a[f][4 * q] = av.x; a[f][4 * q + 1] = av.y; a[f][4 * q + 2] = av.z; a[f][4 * q + 3] = av.w;
        w[f][4 * q] = wv.x; w[f][4 * q + 1] = wv.y; w[f][4 * q + 2] = wv.z; w[f][4 * q + 3] = wv.w;
      }
  };
  auto multiply = [&](const float (&a)[F][HK], const float (&w)[F][HK], int ks0, int ks1) {
#pragma unroll
    for (int ks = ks0; ks < ks1; ++ks)
#pragma unroll
      for (int f = 0; f < F; ++f)
#pragma unroll
        for (int g = 0; g < F; ++g) acc[f][g] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[f][ks], w[g][ks], acc[f][g], 0, 0, 0);
  };
  // Three k-tiles are in flight: t in fragment registers (being multiplied), t + 1 in LDS (its fragments are read between
  // the two halves of t's MFMAs), t + 2 on its way from global memory (written to the buffer of t, which every wave left
  // before the previous barrier, behind t's MFMAs).  Everything but the MFMAs is issued in their shadow.
  const int ktiles = (K + BK - 1) / BK;
  float fa[2][F][HK], fw[2][F][HK];
  fetch(0);
  stage(0);
  if (ktiles > 1) fetch(BK);
  __syncthreads();
  read_frags(0, fa[0], fw[0]);
  if (ktiles > 1) stage(1);
  __syncthreads();
  auto step = [&](int kt, float (&ca)[F][HK], float (&cw)[F][HK], float (&na)[F][HK], float (&nw)[F][HK]) {
    if (kt + 2 < ktiles) fetch((kt + 2) * BK);
    multiply(ca, cw, 0, HK / 2);
    if (kt + 1 < ktiles) read_frags((kt + 1) & 1, na, nw);
    multiply(ca, cw, HK / 2, HK);
    if (kt + 2 < ktiles) stage(kt & 1);
    __syncthreads();
  };
  // The same step without its conditions, for k-tiles whose successors t + 1 and t + 2 exist and need no mask: one basic block,
  // in which the scheduler is told to put the global fetches between the first half's MFMAs and the fragment reads between the
  // second half's (a fetch or read blocks the wave's issue for tens of cycles; behind an MFMA of 64 cycles that costs nothing).
  auto fast_step = [&](int kt, float (&ca)[F][HK], float (&cw)[F][HK], float (&na)[F][HK], float (&nw)[F][HK]) {
#pragma unroll
    for (int i = 0; i < NV; ++i) { ra[i] = *reinterpret_cast<const float4*>(pa[i] + (kt + 2) * BK); rw[i] = *reinterpret_cast<const float4*>(pw[i] + (kt + 2) * BK); }
    multiply(ca, cw, 0, HK / 2);
    read_frags((kt + 1) & 1, na, nw);
    multiply(ca, cw, HK / 2, HK);
    stage(kt & 1);
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int MF = F * F * HK / 2;                    // MFMAs per half
#pragma unroll
    for (int i = 0; i < 2 * NV; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, MF / (2 * NV), 0);     // MFMA
      __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);                 // one global fetch
    }
#pragma unroll
    for (int i = 0; i < F * HK / 2; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, MF / (F * HK / 2), 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                 // one fragment read
    }
#endif
    __syncthreads();
  };
  const int kfull = K / BK;                               // k-tiles that need no mask
  int kt = 0;
  for (; kt + 3 < kfull; kt += 2) {
    fast_step(kt, fa[0], fw[0], fa[1], fw[1]);
    fast_step(kt + 1, fa[1], fw[1], fa[0], fw[0]);
  }
  for (; kt < ktiles; kt += 2) {
    step(kt, fa[0], fw[0], fa[1], fw[1]);
    if (kt + 1 < ktiles) step(kt + 1, fa[1], fw[1], fa[0], fw[0]);
  }
  // lane (l32, half) holds column n = l32 of a fragment and its rows 8 (v / 4) + 4 half + v % 4
#pragma unroll
  for (int f = 0; f < F; ++f)
#pragma unroll
    for (int g = 0; g < F; ++g)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int m = m0 + wm + 32 * f + 8 * (v >> 2) + 4 * half + (v & 3), n = n0 + wn + 32 * g + l32;
        if (m < M && n < N) epilogue_store<float>(ep, m, n, N, acc[f][g][v]);
      }
}

__device__ __forceinline__ void wait_vmem() {   // all outstanding global -> LDS transfers of this wave have landed
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#endif
}

template <int N> __device__ __forceinline__ void wait_vmem_upto() {   // at most N global -> LDS transfers of this wave still in flight
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
#endif
}

// Bare workgroup barrier.  __syncthreads() also fences memory, which makes the compiler drain every
// outstanding global -> LDS transfer (vmcnt(0)) and so serialises a multi-stage pipeline; the main loop
// orders its LDS traffic itself (wait_vmem_upto before the barrier, data-dependent waits on its own reads).
__device__ __forceinline__ void block_barrier() {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_s_barrier();
#endif
}

// fp32 path on the bf16 matrix instructions (planes.h).  A wave owns 64 x 64 of the result, 2 x 2 accumulator fragments of 32 x 32, and takes k-tiles of
// 32 terms.  SHARED: the block's four waves lie 2 x 2 on 128 x 128 and share the operands of every k-tile; otherwise all four own the
// same 64 x 64 and each takes every fourth k-tile, with a part of LDS of its own and no barrier in its loop.
// Operands go from global memory straight into LDS (as in the bf16 kernel below: 8 rows of 128 bytes an instruction, the 16-byte chunk c of row r in
// slot c ^ ((r / 2) % 8)).  The half-wave h takes the chunks 4 ks + 2 h and the next as its eight terms of instruction ks, in both operands alike.
// Cutting costs 5.5 vector instructions an entry, 176 per k-step against 24 matrix instructions of 32 cycles, whose shadow they just fit: eleven of the
// next step's behind each of this step's (two of them, the roundings, at half rate: 125M fp32 step 2964 us, 2940 with planes cut by truncation, planes.h).  (A 64 x 64 tile shared the usual way, 32 x 32 a wave, would cut every entry twice.)
// The product of the first planes has a set of accumulators of its own: the other five terms are at most 2^-8 of it and round in a sum as
// small, which leaves one rounding of the large sum per sixteen terms.
// The shared form has two blocks a CU and no registers for that.  Off from fp64 by 0.9e-7 of the norm at K = 768 and 1.0e-7 at 1024 (the fp32 kernels: 1.8e-7 to
// 5.0e-7, 2.9e-7 to 5.7e-7), shared 4.2e-7 at 768, 7.0e-7 at 2048 (8.1e-7), 14e-7 at 8192 (16e-7).
// What bounds it: the chip's power at large sizes (4096 x 2048 x 8192 176 TFLOP/s, 185 with planes cut by truncation, six times that on the matrix cores; the fp32 instruction 140), the wave's
// issue at small ones (2400 cycles a k-tile for 1536 of matrix instructions; 2900 with the reads and transfers in a row).
// K % 32 == 0 and 16-byte aligned rows; any M, N.
constexpr int kPlaneK = 32;
template <bool SHARED>
__global__ void __launch_bounds__(256, SHARED ? 2 : 1) gemm_planes_kernel(const float* __restrict__ A, const float* __restrict__ W, int M, int N, int K, GemmEpi ep, GemmTwin tw, int models) {
  constexpr int BT = SHARED ? 128 : 64;
  constexpr int STAGE = 2 * BT * kPlaneK * 4;                  // bytes of a k-tile: A's rows, then W's
  constexpr int LOADS = SHARED ? 8 : 16;                       // transfers of a wave per k-tile
  extern __shared__ __attribute__((aligned(1024))) unsigned char gsm[];
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
  const int wave = uniform_of(tid >> 6);
  const int tiles_n = (N + BT - 1) / BT, tiles_m = (M + BT - 1) / BT;
  int tm, tn;
  const int model = tile_of_block(tiles_m, tiles_n, models, tm, tn);
  if (model < 0) return;
  A = ahead(A, model * tw.a); W = ahead(W, model * tw.w); ep.out = ahead(ep.out, model * tw.out); ep.resid = ahead(ep.resid, model * tw.out); ep.bias = ahead(ep.bias, model * tw.bias);
  const int mb = tm * BT, nb = tn * BT;                        // of the block's tile
  const int m0 = SHARED ? mb + 64 * (wave >> 1) : mb, n0 = SHARED ? nb + 64 * (wave & 1) : nb;
  // lane L supplies row L / 8 of a transfer's eight rows, slot L % 8; rows past the matrix are its last row (not stored).  Byte offsets from the
  // tile's first row.  Shared tiles: wave w transfers rows 32 w .. 32 w + 31 of either operand.
  uint32_t off[LOADS];
#pragma unroll
  for (int g = 0; g < LOADS; ++g) {
    const int rl = (SHARED ? wave * 4 + (g & 3) : (g & 7)) * 8 + (lane >> 3), c = ((lane & 7) ^ ((rl >> 1) & 7)) * 16;
    off[g] = (uint32_t)(g < LOADS / 2 ? min(rl, M - 1 - mb) : min(rl, N - 1 - nb)) * (uint32_t)K * 4u + (uint32_t)c;
  }
  const int nk = K / kPlaneK, steps = SHARED ? nk : (wave < nk ? (nk - wave + 3) / 4 : 0);
  auto ktile = [&](int i) { const int j = i < steps ? i : steps - 1; return SHARED ? j : wave + 4 * j; };     // of step i
#if defined(__HIP_DEVICE_COMPILE__)
  const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(A + (size_t)mb * K), 0, 0xFFFFFFFFu, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsW = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(W + (size_t)nb * K), 0, 0xFFFFFFFFu, 0x00020000);
#endif
  const uint32_t own = SHARED ? 0u : (uint32_t)wave * 2 * STAGE;      // this wave's part of LDS
  // Transfer g of step i's k-tile into place pos, unconditionally, so that every step is the same: past the last step that one is read again into a
  // place nobody reads any more.
  auto transfer = [&](int i, int pos, int g) {
#if defined(__HIP_DEVICE_COMPILE__)
    const int rows8 = SHARED ? (g < 4 ? wave * 4 + g : 16 + wave * 4 + g - 4) : g;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(g < LOADS / 2 ? rsA : rsW, (__attribute__((address_space(3))) void*)(gsm + own + pos * STAGE + rows8 * 1024), 16, off[g], ktile(i) * (kPlaneK * 4), 0, 0);
#endif
  };
  f32x16 acc[2][2], low_[SHARED ? 1 : 2][2];
  f32x16 (&low)[2][2] = *reinterpret_cast<f32x16 (*)[2][2]>(SHARED ? &acc[0][0] : &low_[0][0]);
  auto clear = [&]() {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] = low[i][j][v] = 0.f;
  };
  clear();
  struct Frags { PlanesOf<3> f[4]; };                          // A's two, W's two
  struct Raw { f32x4v lo[4], hi[4]; };
  typedef __attribute__((address_space(3))) unsigned char lds_byte;
  typedef __attribute__((address_space(3))) const f32x4v lds_f32x4;
  const int swz = (l32 >> 1) & 7, rowA = SHARED ? 64 * (wave >> 1) : 0, rowW = BT + (SHARED ? 64 * (wave & 1) : 0);
  uint32_t ra[2][2];                                           // LDS addresses of a lane's two chunks of row l32, k-step ks
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
#pragma unroll
    for (int u = 0; u < 2; ++u) ra[ks][u] = (uint32_t)(uintptr_t)(lds_byte*)gsm + own + (uint32_t)l32 * 128 + (uint32_t)(((4 * ks + 2 * half + u) ^ swz) * 16);
  auto read = [&](int pos, int ks, int q, Raw& o) {
    const int f = q >> 1;
    const f32x4v v = *(lds_f32x4*)(uintptr_t)(ra[ks][q & 1] + (uint32_t)(pos * STAGE + ((f < 2 ? rowA : rowW) + 32 * (f & 1)) * 128));
    if (q & 1) o.hi[f] = v; else o.lo[f] = v;
  };
  auto mfma = [&](const Frags& o, int x, int y, int q, f32x16 (&to)[2][2]) {
    f32x16& t = to[q >> 1][q & 1];
    t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, o.f[q >> 1].p[x]), __builtin_bit_cast(bf16x8, o.f[2 + (q & 1)].p[y]), t, 0, 0, 0);
  };
  auto in_this_order = [&]() {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_sched_barrier(0);
#endif
  };
  // The products of one k-step, the cuts of the next (from place pos) and the transfers of step `fetch` (none if negative) into place `to`.  A read or
  // transfer holds the wave's issue up for 25 to 35 cycles, so none stands without a matrix instruction before it: two terms with a read behind each
  // instruction, then a fragment under each term, eleven vector instructions behind a matrix instruction, and the transfers.
  auto step = [&](const Frags& cur, int pos, int ks, Frags& next, int fetch, int to) {
    constexpr int X[6] = {2, 1, 0, 1, 0, 0}, Y[6] = {0, 1, 2, 0, 1, 0};        // the smallest first
    Raw r;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      read(pos, ks, q, r);
      in_this_order();
      mfma(cur, X[q >> 2], Y[q >> 2], q & 3, low);
      in_this_order();
    }
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      f32x16 (&sum)[2][2] = f == 3 ? acc : low;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        mfma(cur, X[2 + f], Y[2 + f], q, sum);
        if (fetch >= 0 && 4 * f + q < LOADS) transfer(fetch, to, 4 * f + q);
        const f32x4v& v = q < 2 ? r.lo[f] : r.hi[f];
        cut_pair_rounded(v[2 * (q & 1)], v[2 * (q & 1) + 1], q, next.f[f]);
        in_this_order();
      }
    }
  };
  if (steps > 0) {                                             // SHARED: the same for every wave of the block
    Frags f0, f1;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int g = 0; g < LOADS; ++g) transfer(i, i, g);
    wait_vmem_upto<LOADS>();
    if (SHARED) block_barrier();
    {
      Raw r;
#pragma unroll
      for (int q = 0; q < 8; ++q) read(0, 0, q, r);
#pragma unroll
      for (int f = 0; f < 4; ++f) {
        cut_pair_rounded(r.lo[f][0], r.lo[f][1], 0, f0.f[f]); cut_pair_rounded(r.lo[f][2], r.lo[f][3], 1, f0.f[f]);
        cut_pair_rounded(r.hi[f][0], r.hi[f][1], 2, f0.f[f]); cut_pair_rounded(r.hi[f][2], r.hi[f][3], 3, f0.f[f]);
      }
    }
    for (int i = 0; i < steps; ++i) {
      step(f0, i & 1, 1, f1, -1, 0);
      // this k-tile's values are in registers: its place may be overwritten once every wave that reads it is here, and the next one has
      // landed once every wave's share of it has
#if defined(__HIP_DEVICE_COMPILE__)
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#endif
      wait_vmem();
      if (SHARED) block_barrier();
      in_this_order();
      step(f1, (i + 1) & 1, 0, f0, i + 2, i & 1);              // behind the last step the cuts are of no use
    }
    wait_vmem();                                               // nothing on its way into LDS when it is used for the sums
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) if (!SHARED) acc[i][j] += low[i][j];
  }
  // a sum that is not finite: this wave's share of it again, by the fp32 instructions (planes.h)
  {
    float zero = 0.f;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) zero = __builtin_fmaf(acc[i][j][v], 0.f, zero);
    if (__ballot(!(zero == 0.f))) {
      clear();
      for (int i = 0; i < steps; ++i)
#pragma unroll 1
        for (int k = ktile(i) * kPlaneK; k < (ktile(i) + 1) * kPlaneK; k += 2) {
          float a[2], w[2];
#pragma unroll
          for (int f = 0; f < 2; ++f) { a[f] = A[(size_t)min(m0 + 32 * f + l32, M - 1) * K + k + half]; w[f] = W[(size_t)min(n0 + 32 * f + l32, N - 1) * K + k + half]; }
#pragma unroll
          for (int f = 0; f < 2; ++f)
#pragma unroll
            for (int g = 0; g < 2; ++g) acc[f][g] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[f], w[g], acc[f][g], 0, 0, 0);
        }
    }
  }
  // One fragment's rows 8 q + 4 half + v and column l32 from (m, n); the values a residual is added to are requested before anything is stored.
  auto store = [&](const float (&r)[16], int m, int n) {
    if (n >= N) return;
    const float b = ep.bias ? reinterpret_cast<const float*>(ep.bias)[n] : 0.f;
    float* o = reinterpret_cast<float*>(ep.out) + (size_t)m * N + n;
    const float* src = ep.resid + (size_t)m * N + n;
    const int rows = M - m;                                    // may be negative
    auto each = [&](auto f) {
#pragma unroll
      for (int v = 0; v < 16; ++v) { const int i = 8 * (v >> 2) + (v & 3); if (i < rows) f(v, o + (size_t)i * N); }
    };
    float old[16];
    switch (ep.mode) {                                         // uniform
      case EPI_GELU:  each([&](int v, float* p) { *p = gelu_f32(r[v] + b); }); break;
      case EPI_RELU:  each([&](int v, float* p) { *p = fmaxf(r[v] + b, 0.f); }); break;
      case EPI_RESID:
#pragma unroll
        for (int v = 0; v < 16; ++v) { const int i = 8 * (v >> 2) + (v & 3); old[v] = src[((ptrdiff_t)(i < rows ? i : rows - 1)) * N]; }
        arrived(old);
        each([&](int v, float* p) { *p = old[v] + (r[v] + b); });
        break;
      default:        each([&](int v, float* p) { *p = r[v] + b; }); break;
    }
  };
  if constexpr (SHARED) {
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      float r[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) r[v] = acc[f >> 1][f & 1][v];
      store(r, m0 + 32 * (f >> 1) + 4 * half, n0 + 32 * (f & 1) + l32);
    }
  } else {
    // the waves' sums in the order ((0 + 1) + (2 + 3)); wave w adds up and stores fragment w
    __syncthreads();
    f32x4v* parts = reinterpret_cast<f32x4v*>(gsm);            // [wave][fragment][4][lane]
#pragma unroll
    for (int f = 0; f < 4; ++f)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x16& a = acc[f >> 1][f & 1];
        parts[((wave * 4 + f) * 4 + q) * 64 + lane] = f32x4v{a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]};
      }
    __syncthreads();
    float r[16];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      f32x4v p[4];
#pragma unroll
      for (int w = 0; w < 4; ++w) p[w] = parts[((w * 4 + wave) * 4 + q) * 64 + lane];
      const f32x4v t = (p[0] + p[1]) + (p[2] + p[3]);
#pragma unroll
      for (int v = 0; v < 4; ++v) r[4 * q + v] = t[v];
    }
    store(r, m0 + 32 * (wave >> 1) + 4 * half, n0 + 32 * (wave & 1) + l32);
  }
}

template <bool SHARED>
static hipError_t launch_gemm_planes(const float* A, const float* W, int M, int N, int K, const GemmEpi& ep, const GemmTwin& gt, int models, hipStream_t s) {
  constexpr int BT = SHARED ? 128 : 64, lds = SHARED ? 2 * 2 * 128 * kPlaneK * 4 : 4 * 2 * 2 * 64 * kPlaneK * 4;
  static std::atomic<bool> attr_set{false};       // set twice by racing threads at worst: the call is idempotent
  auto kern = gemm_planes_kernel<SHARED>;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  const int64_t tiles = (int64_t)((M + BT - 1) / BT) * ((N + BT - 1) / BT) * models;
  hipLaunchKernelGGL(kern, dim3((unsigned)((tiles + 7) / 8 * 8)), dim3(256), lds, s, A, W, M, N, K, ep, gt, models);
  return hipGetLastError();
}

// bf16 path: MFMA 32x32x16.  Block tile BM x BN, BK = 64, WM x WN waves, each owning (BM / WM) x (BN / WN) of
// the output as FM x FN accumulator fragments of 32 x 32.  Operands go from global memory straight into LDS
// (no register staging).  Two main loops: the ping-pong pipeline (PP = 1, eight waves, large tiles) and a plain
// multi-stage loop with one barrier per k-tile (PP = 0, the 128 x 128 tile of small problems).
constexpr int GB_K = 64;

// erf-GELU, x Phi(x) = max(x, 0) - |x|/2 erfc(|x| / sqrt 2), with erfc(|x| / sqrt 2) = exp2(q(|x|)): q is a
// degree-6 fit of log2 erfc on [0, 6] (beyond 6 the term is below 1e-8 and |x| is clamped).  Absolute error of
// the result <= 1e-7 for all x, relative error <= 2e-5 for |x| < 3: far below the bf16 rounding of the result.
// One transcendental (v_exp_f32) and nine full-rate operations.
__device__ __forceinline__ float gelu_fast(float x) {
  const float a = fminf(fabsf(x), 6.0f);
  float q = 3.1244733690982684e-05f;
  q = __builtin_fmaf(q, a, -0.0007523701642639935f);
  q = __builtin_fmaf(q, a, 0.008023424074053764f);
  q = __builtin_fmaf(q, a, -0.05332072451710701f);
  q = __builtin_fmaf(q, a, -0.4588412642478943f);
  q = __builtin_fmaf(q, a, -1.1511778831481934f);
  q = __builtin_fmaf(q, a, 4.343822638475103e-06f);
  const float e = __builtin_amdgcn_exp2f(q);
  return __builtin_fmaf(-fabsf(0.5f * x), e, fmaxf(x, 0.f));
}

template <int MODE>
__device__ __forceinline__ void epilogue_bf16(void* out, size_t o, float v) {
  if (MODE == EPI_STORE) from_f32(v, reinterpret_cast<bf16_t*>(out)[o]);
  else if (MODE == EPI_GELU) from_f32(gelu_fast(v), reinterpret_cast<bf16_t*>(out)[o]);
  else if (MODE == EPI_RELU) from_f32(fmaxf(v, 0.f), reinterpret_cast<bf16_t*>(out)[o]);
  else if (MODE == EPI_RESID) reinterpret_cast<float*>(out)[o] += v;
  else reinterpret_cast<float*>(out)[o] = v;
}

// Tile (tm, tn) of the product.  FOLD: A's rows hold FOLD runs of K / FOLD terms and W's one, which every run is multiplied with.  Those are sums that
// stay fp32 throughout: they are taken in pieces of kPieceTiles k-tiles, so that the large sum rounds once a piece and not with every instruction
// (the adding up hides behind the other group's memory phase).
template <int BM, int BN, int WM, int WN, int BK, int STAGES, int MODE, int PP, int FOLD>
__device__ __forceinline__ void gemm_bf16_tile(const bf16_t* __restrict__ A, const bf16_t* __restrict__ W, int M, int N, int K, int lda, int ldw,
                                               void* out, const bf16_t* __restrict__ bias,      // resid may be out
                                               const int32_t* __restrict__ targets, float* __restrict__ tlogit, const float* resid, int tm, int tn) {
  constexpr int NW = WM * WN;
  constexpr int FM = BM / (32 * WM), FN = BN / (32 * WN);      // 32x32 fragments per wave
  constexpr int CPR = BK / 8;                                  // 16-byte chunks per LDS row
  constexpr int RPI = 64 / CPR;                                // rows one global_load_lds instruction fills (1 KiB)
  constexpr int RPB = 256 / (BK * 2);                          // rows per 256 B of LDS (one sweep over all banks)
  constexpr int GA = BM / RPI / NW, GW = BN / RPI / NW;        // instructions per wave per k-tile
  static_assert(PP != 0 || (GA >= 1 && GW >= 1 && (STAGES - 2) * (GA + GW) < 64), "tile / stage configuration");
  // LDS: STAGES slabs of [BM + BN][BK] bf16, rows unpadded; the 16-byte chunk c of row r sits in slot
  // c ^ ((r / RPB) % CPR), which makes the MFMA operand reads conflict-free.  The slabs are written by
  // global_load_lds (global memory -> LDS without passing registers): one instruction fills RPI rows, lane L
  // supplying row L / CPR, slot L % CPR, i.e. it fetches the global chunk (L % CPR) ^ swizzle(row).
  extern __shared__ __attribute__((aligned(1024))) unsigned char gsm[];
  bf16_t* As = reinterpret_cast<bf16_t*>(gsm);                 // [STAGES][BM][BK]
  bf16_t* Ws = As + STAGES * BM * BK;                          // [STAGES][BN][BK]
  const int tid = threadIdx.x, lane = tid & 63;
#if defined(__HIP_DEVICE_COMPILE__)
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: kept in a scalar register
#else
  const int wave = tid >> 6;
#endif
  const int wm = wave / WN, wn = wave % WN;
  constexpr int kPieceTiles = 2;
  constexpr bool PIECES = FOLD > 1;
  [[maybe_unused]] const int tiles_m = (M + BM - 1) / BM;
  const int m0 = tm * BM, n0 = tn * BN;
  f32x16 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  // Residual epilogue on the smaller tiles: this lane's part of the residual stream is requested now, ahead of
  // every operand transfer (loads complete in order, so the vmcnt counts of the main loop still only see the
  // transfers), and has long arrived when the epilogue adds to it; only the write-back remains exposed there.
  constexpr bool PRE_RES = MODE == EPI_RESID && FM * FN <= 4;
  const bool pre_res = PRE_RES && m0 + BM <= M && n0 + BN <= N;
  float res[PRE_RES ? FM * FN * 16 : 1];
  if (PRE_RES && pre_res) {
    const float* rp = resid + (size_t)(m0 + wm * (BM / WM) + 4 * (lane >> 5)) * N + n0 + wn * (BN / WN) + (lane & 31);
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) res[(i * FN + j) * 16 + v] = rp[(size_t)(i * 32 + 8 * (v >> 2) + (v & 3)) * N + j * 32];
  }
  f32x16 total[PIECES ? FM : 1][PIECES ? FN : 1];
  auto add_piece = [&](bool first) {
    if constexpr (PIECES) {
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v) { total[i][j][v] = first ? acc[i][j][v] : total[i][j][v] + acc[i][j][v]; acc[i][j][v] = 0.f; }
    }
  };
  add_piece(true);
  const int nk = K / BK, nkw = nk / FOLD;                       // k-tiles of A and of W
  auto w_ktile = [&](int kt) {
    if constexpr (FOLD == 1) return kt;
    else { const int r = kt < nkw ? kt : kt - nkw; return r < nkw ? r : r - nkw; }
  };
  static_assert(FOLD == 1 || FOLD == 3, "runs");
  // reader: lane (l32, half) reads row l32 of each fragment, logical chunk 2*ks + half
  const int l32 = lane & 31, half = lane >> 5, swz = (l32 / RPB) % CPR;
  int koff[BK / 16];
#pragma unroll
  for (int ks = 0; ks < BK / 16; ++ks) koff[ks] = ((2 * ks + half) ^ swz) << 3;
  if constexpr (PP != 0) {
    // Ping-pong pipeline.  Two groups of four waves (waves w and w + 4 share a SIMD) take turns: while one group
    // runs the MFMAs of half a k-tile (one wave per SIMD keeps the matrix pipe busy on its own: the products of
    // a half are independent), the other reads the operands of its next half from LDS and issues its share of
    // the global -> LDS transfers.  The groups run one phase apart (the second starts with an extra barrier,
    // the first ends with one) and every phase ends in a workgroup barrier, so a SIMD always holds one wave of
    // each kind and the transfers never wait behind a group that is issuing MFMAs.
    //
    // LDS is a ring of R units of 8 KiB: 64 rows of one operand over the BK = 64 columns of a k-tile (whole
    // 128-byte lines of the source).  One transfer
    // instruction per wave fills a unit (wave w supplies rows 8w .. 8w + 7).  K-tile kt owns the U = (BM + BN) / 64
    // units kt U .. kt U + U - 1 (A first), at ring positions taken modulo R.  Unit q may be overwritten by unit
    // q + R once k-tile q / U has been read by both groups, which is the case from the first memory phase of the
    // next k-tile on; so the two memory phases of k-tile kt issue the units R - U + kt U .. R + kt U - 1, i.e.
    // R - U units (one and a half k-tiles for 256 x 256 tiles) are in flight or landed ahead of the reader.
    // K-tile kt + 1 must have landed before the first group starts on it: the second group waits for its shares at
    // the end of its last memory phase of k-tile kt, the first at the end of its last MFMA phase, in both cases
    // with the R - 2U units of later k-tiles still in flight; the barrier that follows publishes them.
    static_assert(NW == 8 && BK == 64 && BM % 64 == 0 && BN % 64 == 0, "ping-pong configuration");
    constexpr int UA = BM / 64, U = (BM + BN) / 64, R = STAGES, Q0 = R - U;
    constexpr int UH0 = (U + 1) / 2;                             // units issued in the first memory phase of a k-tile
    static_assert(R >= 2 * U && R * 8192 <= 160 * 1024, "ring size");
    const int frow = wave * 8 + (lane >> 3);                     // row this lane supplies within a unit
    uint32_t uo[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool is_a = u < UA;
      const int rl = (is_a ? u : u - UA) * 64 + frow;
      int r = (is_a ? m0 : n0) + rl;
      const int lim = is_a ? M : N;
      r = r < lim ? r : lim - 1;
      uo[u] = ((uint32_t)r * (uint32_t)(is_a ? lda : ldw) + (((lane & 7) ^ ((frow >> 1) & 7)) << 3)) * 2;   // bytes
    }
#if defined(__HIP_DEVICE_COMPILE__)
    // buffer addressing: per-lane byte offset in a register, the k-tile's offset in a scalar, bounds-checked
    const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(A), 0, ((uint32_t)(M - 1) * (uint32_t)lda + (uint32_t)K) * 2u, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsW = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(W), 0, ((uint32_t)(N - 1) * (uint32_t)ldw + (uint32_t)(K / FOLD)) * 2u, 0x00020000);
#endif
    // Transfers are issued unconditionally, so that every wave's count of outstanding transfers is the same in
    // every k-tile: a unit past the last k-tile re-reads the last one into a ring slot nobody reads any more.
    auto issue_unit = [&](int u, int ktile, int pos) {           // u is a compile-time constant after unrolling
#if defined(__HIP_DEVICE_COMPILE__)
      const int kc = ktile < nk ? ktile : nk - 1;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(u < UA ? rsA : rsW, (__attribute__((address_space(3))) void*)(gsm + pos * 8192 + wave * 1024), 16, uo[u], (u < UA ? kc : w_ktile(kc)) * (BK * 2), 0, 0);
#endif
    };
    int wpos = 0;                                                // ring position of the next unit to issue
#pragma unroll
    for (int q = 0; q < Q0; ++q) {
      issue_unit(q % U, q / U, wpos);
      wpos = wpos + 1 == R ? 0 : wpos + 1;
    }
    wait_vmem_upto<Q0 - U>();
    block_barrier();
    int rbase = 0;                                               // ring position of unit 0 of k-tile kt
    const int rowA = wm * (BM / WM), rowW = wn * (BN / WN);      // this wave's first row of either operand
    const int grp = wave >> 2;
    if (grp) block_barrier();
    // LDS byte addresses of this lane's fragment reads in the coming memory phase.  They are worked out in the
    // MFMA phase before it, between the wave's own MFMAs: a vector instruction of the memory phase would queue
    // behind the other wave's MFMAs on the SIMD, so the memory phases hold LDS reads, transfers and scalar
    // bookkeeping only.
    typedef __attribute__((address_space(3))) unsigned char lds_byte;
    typedef __attribute__((address_space(3))) const bf16x8 lds_bf16x8;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_byte*)gsm;   // LDS address of the ring
    uint32_t lk[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) lk[ks] = lds0 + (uint32_t)(l32 * BK + koff[ks]) * 2u;
    uint32_t ra[2][FM], rb[2][FN];
    auto set_addrs = [&](int base, int h) {
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        int pos = base + (rowA + i * 32) / 64; pos = pos >= R ? pos - R : pos;
        const uint32_t sa = (uint32_t)(pos * 8192 + ((rowA + i * 32) % 64) * (BK * 2));
        ra[0][i] = sa + lk[2 * h]; ra[1][i] = sa + lk[2 * h + 1];
      }
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        int pos = base + UA + (rowW + j * 32) / 64; pos = pos >= R ? pos - R : pos;
        const uint32_t sb = (uint32_t)(pos * 8192 + ((rowW + j * 32) % 64) * (BK * 2));
        rb[0][j] = sb + lk[2 * h]; rb[1][j] = sb + lk[2 * h + 1];
      }
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {                           // keep the additions where they are written
#pragma unroll
        for (int i = 0; i < FM; ++i) asm volatile("" : "+v"(ra[ks][i]));
#pragma unroll
        for (int j = 0; j < FN; ++j) asm volatile("" : "+v"(rb[ks][j]));
      }
#endif
    };
    set_addrs(0, 0);
    for (int kt = 0; kt < nk; ++kt) {
      int rnext = rbase + U; rnext = rnext >= R ? rnext - R : rnext;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        bf16x8 a[2][FM], b[2][FN];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
          for (int i = 0; i < FM; ++i) a[ks][i] = *(lds_bf16x8*)(uintptr_t)ra[ks][i];
#pragma unroll
          for (int j = 0; j < FN; ++j) b[ks][j] = *(lds_bf16x8*)(uintptr_t)rb[ks][j];
        }
#pragma unroll
        for (int t = 0; t < (h == 0 ? UH0 : U - UH0); ++t) {
          const int qq = Q0 + (h == 0 ? 0 : UH0) + t;             // unit number relative to kt U
          issue_unit(qq % U, kt + qq / U, wpos);
          wpos = wpos + 1 == R ? 0 : wpos + 1;
        }
        if (h == 1 && grp) wait_vmem_upto<Q0 - U>();
#if defined(__HIP_DEVICE_COMPILE__)
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
#endif
        set_addrs(h == 0 ? rbase : rnext, h == 0 ? 1 : 0);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
          for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks][i], b[ks][j], acc[i][j], 0, 0, 0);
        if (h == 1 && PIECES && kt % kPieceTiles == kPieceTiles - 1) add_piece(false);
        if (h == 1 && !grp) wait_vmem_upto<Q0 - U>();
#if defined(__HIP_DEVICE_COMPILE__)
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
#endif
      }
      rbase = rnext;
    }
    if (!grp) block_barrier();
  } else {
  // loader: this lane's source offsets (elements) for the row groups its wave owns
  const int lrow = lane / CPR, lslot = lane % CPR;
  uint32_t ao[GA], wo[GW];
#pragma unroll
  for (int g = 0; g < GA; ++g) {
    const int rl = (wave * GA + g) * RPI + lrow;               // row within the tile
    int r = m0 + rl; r = r < M ? r : M - 1;
    ao[g] = (uint32_t)r * (uint32_t)lda + ((lslot ^ ((rl / RPB) % CPR)) << 3);
  }
#pragma unroll
  for (int g = 0; g < GW; ++g) {
    const int rl = (wave * GW + g) * RPI + lrow;
    int c = n0 + rl; c = c < N ? c : N - 1;
    wo[g] = (uint32_t)c * (uint32_t)ldw + ((lslot ^ ((rl / RPB) % CPR)) << 3);
  }
  auto issue = [&](int kt, int buf) {
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
    for (int g = 0; g < GA; ++g)
      __builtin_amdgcn_global_load_lds(A + ao[g] + kt * BK, As + (buf * BM + (wave * GA + g) * RPI) * BK, 16, 0, 0);
#pragma unroll
    for (int g = 0; g < GW; ++g)
      __builtin_amdgcn_global_load_lds(W + wo[g] + w_ktile(kt) * BK, Ws + (buf * BN + (wave * GW + g) * RPI) * BK, 16, 0, 0);
#endif
  };
  // prologue: STAGES - 1 k-tiles in flight
#pragma unroll
  for (int p = 0; p < STAGES - 1; ++p)
    if (p < nk) issue(p, p);
  int buf = 0;
  for (int kt = 0; kt < nk; ++kt) {
    // k-tile kt has landed once at most the STAGES - 2 younger tiles are still in flight
    if (kt + STAGES - 2 < nk) wait_vmem_upto<(STAGES - 2) * (GA + GW)>(); else wait_vmem_upto<0>();
    block_barrier();                                           // ... for every wave; and slab (kt - 1) % STAGES is free
    if (kt + STAGES - 1 < nk) issue(kt + STAGES - 1, buf == 0 ? STAGES - 1 : buf - 1);
    const bf16_t* as = As + (buf * BM + wm * (BM / WM) + l32) * BK;
    const bf16_t* ws = Ws + (buf * BN + wn * (BN / WN) + l32) * BK;
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) {
      bf16x8 a[FM], b[FN];
#pragma unroll
      for (int i = 0; i < FM; ++i) a[i] = *reinterpret_cast<const bf16x8*>(as + i * 32 * BK + koff[ks]);
#pragma unroll
      for (int j = 0; j < FN; ++j) b[j] = *reinterpret_cast<const bf16x8*>(ws + j * 32 * BK + koff[ks]);
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    if (PIECES && kt % kPieceTiles == kPieceTiles - 1) add_piece(false);
    buf = buf + 1 == STAGES ? 0 : buf + 1;
  }
  }
  if constexpr (PIECES) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) acc[i][j] += total[i][j];
    // a sum that is not finite: again by the fp32 instructions (planes.h; W's infinities meet the zeros in A's smaller planes), run by run the terms of A's number
    float zero = 0.f;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) zero = __builtin_fmaf(acc[i][j][v], 0.f, zero);
    if (__builtin_expect(__ballot(!(zero == 0.f)) != 0, 0)) {
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
#pragma unroll 1
      for (int k = half; k < nkw * BK; k += 2) {
        float a[FM], w[FN];
#pragma unroll
        for (int i = 0; i < FM; ++i) {
          const bf16_t* r = A + (size_t)min(m0 + wm * (BM / WM) + 32 * i + l32, M - 1) * lda + k;
          a[i] = 0.f;
#pragma unroll
          for (int f = 0; f < FOLD; ++f) a[i] += to_f32(r[f * nkw * BK]);
        }
#pragma unroll
        for (int j = 0; j < FN; ++j) w[j] = to_f32(W[(size_t)min(n0 + wn * (BN / WN) + 32 * j + l32, N - 1) * ldw + k]);
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], w[j], acc[i][j], 0, 0, 0);
      }
    }
  }
  if (MODE == EPI_CE) {
    // Cross-entropy partials instead of logits.  The product is taken transposed (rows = vocabulary entries,
    // columns = tokens), so a lane holds one token per fragment column and FM x 16 vocabulary rows of it in
    // registers: the maximum and the sum of exp(logit - max) over the wave's BM / WM vocabulary rows reduce
    // over registers plus one exchange with the partner lane (lane ^ 32).  Written to out as
    // float2 [tokens][tiles_m * WM]; the lane that meets the target row stores its logit.
    float2* part = reinterpret_cast<float2*>(out);
    const int pstride = tiles_m * WM, pcol = tm * WM + wm;
    const int rbase = m0 + wm * (BM / WM) + 4 * (lane >> 5);
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int token = n0 + wn * (BN / WN) + j * 32 + l32;
      const int tgt = token < N ? targets[token] : -1;
      float mx = -INFINITY;
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int r = rbase + i * 32 + 8 * (v >> 2) + (v & 3);
          if (r < M) { mx = fmaxf(mx, acc[i][j][v]); if (r == tgt) tlogit[token] = acc[i][j][v]; }
        }
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      const float msafe = mx == -INFINITY ? 0.f : mx;            // a strip entirely beyond the vocabulary contributes (-inf, 0)
      float sum = 0.f;
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int r = rbase + i * 32 + 8 * (v >> 2) + (v & 3);
          if (r < M) sum += __builtin_amdgcn_exp2f((acc[i][j][v] - msafe) * 1.44269504088896341f);
        }
      sum += __shfl_xor(sum, 32, 64);
      if (lane < 32 && token < N) part[(size_t)token * pstride + pcol] = make_float2(mx, sum);
    }
    return;
  }
  // epilogue: lane holds column l32, rows 8*(v/4) + 4*(lane/32) + v%4 of each 32x32 fragment
  float bv[FN];
#pragma unroll
  for (int j = 0; j < FN; ++j) {
    const int n = n0 + wn * (BN / WN) + j * 32 + l32;
    bv[j] = (bias && n < N) ? to_f32(bias[n]) : 0.f;
  }
  const int mbase = m0 + wm * (BM / WM) + 4 * (lane >> 5), nbase = n0 + wn * (BN / WN) + l32;
  if (PRE_RES && pre_res) {
    float* op = reinterpret_cast<float*>(out) + (size_t)mbase * N + nbase;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v)
          op[(size_t)(i * 32 + 8 * (v >> 2) + (v & 3)) * N + j * 32] = res[(i * FN + j) * 16 + v] + (acc[i][j][v] + bv[j]);
  } else if (MODE == EPI_RESID && m0 + BM <= M && n0 + BN <= N) {
    // larger tiles: the residual of the next fragment is requested before this one's sum is stored (one value after the other, each waiting for
    // the store before it: 2 x 4096 x 2048 x 2048 and x 8192 took 355 us on average, now 147)
    float* op = reinterpret_cast<float*>(out) + (size_t)mbase * N + nbase;
    const float* ip = resid + (size_t)mbase * N + nbase;
    float old[2][16];
    auto request = [&](int f) {
#pragma unroll
      for (int v = 0; v < 16; ++v) old[f & 1][v] = ip[(size_t)((f / FN) * 32 + 8 * (v >> 2) + (v & 3)) * N + (f % FN) * 32];
    };
    request(0);
#pragma unroll
    for (int f = 0; f < FM * FN; ++f) {
      if (f + 1 < FM * FN) request(f + 1);
#pragma unroll
      for (int v = 0; v < 16; ++v)
        op[(size_t)((f / FN) * 32 + 8 * (v >> 2) + (v & 3)) * N + (f % FN) * 32] = old[f & 1][v] + (acc[f / FN][f % FN][v] + bv[f % FN]);
    }
  } else if (m0 + BM <= M && n0 + BN <= N) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v)
          epilogue_bf16<MODE>(out, (size_t)(mbase + i * 32 + 8 * (v >> 2) + (v & 3)) * N + nbase + j * 32, acc[i][j][v] + bv[j]);
  } else {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const int n = nbase + j * 32;
        if (MODE == EPI_RESID) {                                   // all of the fragment's values, then its stores
          float* op = reinterpret_cast<float*>(out) + n;
          const float* ip = resid + n;
          float old[16];
#pragma unroll
          for (int v = 0; v < 16; ++v) { const int m = mbase + i * 32 + 8 * (v >> 2) + (v & 3); old[v] = ip[(size_t)(m < M ? m : M - 1) * N - (n < N ? 0 : n - (N - 1))]; }
          arrived(old);
#pragma unroll
          for (int v = 0; v < 16; ++v) { const int m = mbase + i * 32 + 8 * (v >> 2) + (v & 3); if (m < M && n < N) op[(size_t)m * N] = old[v] + (acc[i][j][v] + bv[j]); }
          continue;
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int m = mbase + i * 32 + 8 * (v >> 2) + (v & 3);
          if (m < M && n < N) epilogue_bf16<MODE>(out, (size_t)m * N + n, acc[i][j][v] + bv[j]);
        }
      }
  }
}

template <int BM, int BN, int WM, int WN, int BK, int STAGES, int MODE, int PP = 0>
__global__ void __launch_bounds__(64 * WM * WN) gemm_bf16_kernel(const bf16_t* __restrict__ A, const bf16_t* __restrict__ W, int M, int N, int K,
                                                                 void* out, const bf16_t* __restrict__ bias,
                                                                 const int32_t* __restrict__ targets, float* __restrict__ tlogit, GemmTwin tw, int models, const float* resid) {
  int tm, tn;
  const int model = tile_of_block((M + BM - 1) / BM, (N + BN - 1) / BN, models, tm, tn);
  if (model < 0) return;
  A = ahead(A, model * tw.a); W = ahead(W, model * tw.w); out = ahead(out, model * tw.out); bias = ahead(bias, model * tw.bias);
  if (MODE == EPI_CE) tlogit = ahead(tlogit, model * tw.tlogit);
  if (MODE == EPI_RESID) resid = ahead(resid, model * tw.out);
  gemm_bf16_tile<BM, BN, WM, WN, BK, STAGES, MODE, PP, 1>(A, W, M, N, K, K, K, out, bias, targets, tlogit, resid, tm, tn);
}

// Several products with fp32 results in one launch: the tiles of all of them, one after the other, dealt out as those of one product are.
// The four weight gradients of a block of 768 columns have 144, 144, 36 and 108 tiles of 128 x 128: one by one they left up to six sevenths of the
// chip idle (2048 tokens: 67 us in four launches, now 36, 0.8 PFLOP/s).
// FOLD = 3, a block of 1024 columns and 231 tokens: 32 us, 50 MB of results among them; product.hip's kernel, which cuts planes from fp32 operands as they lie, took
// 67 in four launches.  Off from fp64 by 0.7e-7 of the norm there (0.8e-7 in product.hip, which shares a sum among waves), 1.0e-7 at 2047 tokens (2.4e-7); with the sums in one
// piece 0.8e-7 and 2.7e-7, and 2 us less.
template <int BM, int BN, int WM, int WN, int BK, int STAGES, int PP, int FOLD>
__global__ void __launch_bounds__(64 * WM * WN) gemm_bf16_group_kernel(ProductGroup g) {
  auto tiles = [&](int j) { return ((g.job[j].M + BM - 1) / BM) * ((g.job[j].N + BN - 1) / BN); };
  int total = 0;
  for (int j = 0; j < g.count; ++j) total += tiles(j);
  int place = place_of_block(total), j = 0, tm, tn;
  if (place < 0) return;
  for (; place >= tiles(j); ++j) place -= tiles(j);
  const GroupedProduct p = g.job[j];
  tile_at(place, (p.M + BM - 1) / BM, (p.N + BN - 1) / BN, tm, tn);
  gemm_bf16_tile<BM, BN, WM, WN, BK, STAGES, EPI_F32, PP, FOLD>(reinterpret_cast<const bf16_t*>(p.A), reinterpret_cast<const bf16_t*>(p.W), p.M, p.N, p.K, p.lda, p.ldw, p.out, nullptr, nullptr, nullptr, nullptr, tm, tn);
}

template <int BM, int BN, int WM, int WN, int BK, int STAGES, int PP, int FOLD>
static hipError_t launch_group_t(const ProductGroup& g, int64_t tiles, hipStream_t s) {
  const size_t lds = PP ? (size_t)STAGES * 8192 : (size_t)STAGES * (BM + BN) * BK * sizeof(bf16_t);
  static std::atomic<bool> attr_set{false};   // set twice by racing threads at worst: the call is idempotent
  auto kern = gemm_bf16_group_kernel<BM, BN, WM, WN, BK, STAGES, PP, FOLD>;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)((tiles + 7) / 8 * 8)), dim3(64 * WM * WN), lds, s, g);
  return hipGetLastError();
}
template <int FOLD>
static hipError_t launch_group_f(const ProductGroup& g, hipStream_t s) {
  auto tiles = [&](int bm, int bn) {
    int64_t t = 0;
    for (int j = 0; j < g.count; ++j) t += (int64_t)((g.job[j].M + bm - 1) / bm) * ((g.job[j].N + bn - 1) / bn);
    return t;
  };
  const int64_t t256 = tiles(256, 256), t128 = tiles(128, 128);
  // The sizes at which one product takes these tiles (launch_gemm).  256 x 256 against 128 x 128 here: passes of four blocks of 2048 columns, 1024 tokens 2593 us against 2712, 4096
  // 6364 against 6887.  (Pieces of sums leave them no registers.)
  if constexpr (FOLD == 1) {
    if (t256 >= 512) return launch_group_t<256, 256, 2, 4, 64, 20, 1, FOLD>(g, t256, s);
  }
  if (t128 > 256) return launch_group_t<128, 128, 2, 4, 64, 8, 1, FOLD>(g, t128, s);
  if (t128 > 128) return launch_group_t<128, 128, 2, 4, 64, 20, 1, FOLD>(g, t128, s);
  return launch_group_t<64, 64, 2, 2, 64, 4, 0, FOLD>(g, tiles(64, 64), s);
}

template <int BM, int BN, int WM, int WN, int BK, int STAGES, int PP = 0>
hipError_t launch_gemm_bf16_t(const bf16_t* A, const bf16_t* W, const bf16_t* bias, void* out, int epi, int M, int N, int K, hipStream_t s, int models, const GemmTwin& tw,
                              const float* resid, const int32_t* targets = nullptr, float* tlogit = nullptr) {
  const size_t lds = PP ? (size_t)STAGES * 8192 : (size_t)STAGES * (BM + BN) * BK * sizeof(bf16_t);   // ping-pong: STAGES counts 8 KiB ring units
  const int grid = (((M + BM - 1) / BM) * ((N + BN - 1) / BN) * models + 7) / 8 * 8;
#define ZGR_GEMM_LAUNCH(MODE)                                                                                           \
  {                                                                                                                     \
    static std::atomic<bool> attr_set{false};   /* set twice by racing threads at worst: the call is idempotent */         \
    auto kern = gemm_bf16_kernel<BM, BN, WM, WN, BK, STAGES, MODE, PP>;                                                             \
    if (!attr_set) {                                                                                                    \
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); \
      if (e != hipSuccess) return e;                                                                                    \
      attr_set = true;                                                                                                  \
    }                                                                                                                   \
    hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * WM * WN), lds, s, A, W, M, N, K, out, bias, targets, tlogit, tw, models, resid); \
  }
  switch (epi) {
    case EPI_STORE: ZGR_GEMM_LAUNCH(EPI_STORE) break;
    case EPI_GELU:  ZGR_GEMM_LAUNCH(EPI_GELU) break;
    case EPI_RELU:  ZGR_GEMM_LAUNCH(EPI_RELU) break;
    case EPI_RESID: ZGR_GEMM_LAUNCH(EPI_RESID) break;
    case EPI_CE:    ZGR_GEMM_LAUNCH(EPI_CE) break;
    default:        ZGR_GEMM_LAUNCH(EPI_F32) break;
  }
#undef ZGR_GEMM_LAUNCH
  return hipGetLastError();
}

// The same product for few tiles: 32 x 32 of the result per block, one wave that reads and multiplies and two that only transfer (A's rows, W's rows), a ring
// of kFewRing k-tiles of 8 KB.  What counts there is the chain of one block: with 64 x 64 tiles every wave transfers, meets, reads eight operands
// of 33 cycles and then multiplies, some 700 cycles a k-tile on a quarter as many CUs; here the reading wave's eight reads run beside the other
// waves' transfers and over its own matrix instructions, and all of a short sum is on its way before the first wait.  The terms are taken in the same
// order, so the result is the same bit for bit.
// 231 x 1024 x 4096 20.9 us -> 10.8, 33 x 768 x 3072 15.3 -> 8.3, 256 x 1024 x 2048 11.8 -> 7.2; the loss of one 33-token prompt of a 125M-parameter model
// 691 us -> 545, a 24-block encoder's backward over 231 tokens 5.9 ms -> 5.6.  Up to 256 tiles, one block a CU: with 128 as the line 590 us and 5.94 ms, with
// 512 554 us.  The same form with 64 x 64 tiles and four readers gave these cases less than 1%.
constexpr int kFewRing = 16;
template <int MODE>
__global__ void __launch_bounds__(192) gemm_bf16_few_kernel(const bf16_t* __restrict__ A, const bf16_t* __restrict__ W, int M, int N, int K, void* out, const bf16_t* __restrict__ bias,      // resid may be out
                                                            GemmTwin tw, int models, const float* resid) {
  constexpr int SLAB = 64 * GB_K * 2;                          // bytes of a k-tile: 32 rows of A, 32 of W
  extern __shared__ __attribute__((aligned(1024))) unsigned char gsm[];
  const int lane = threadIdx.x & 63, wave = uniform_of(threadIdx.x >> 6), l32 = lane & 31, half = lane >> 5;
  int tm, tn;
  const int model = tile_of_block((M + 31) / 32, (N + 31) / 32, models, tm, tn);
  if (model < 0) return;
  A = ahead(A, model * tw.a); W = ahead(W, model * tw.w); out = ahead(out, model * tw.out); bias = ahead(bias, model * tw.bias);
  if (MODE == EPI_RESID) resid = ahead(resid, model * tw.out);
  const int m0 = tm * 32, n0 = tn * 32, nk = K / GB_K;
  if (wave != 0) {
    // transfers: rows of eight of one operand, the 16-byte chunk c of row r in slot c ^ ((r / 2) % 8); past the last k-tile that one is read again
    const bool is_a = wave == 1;
    uint32_t off[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int rl = 8 * g + (lane >> 3), row = is_a ? min(m0 + rl, M - 1) : min(n0 + rl, N - 1);
      off[g] = ((uint32_t)row * (uint32_t)K + (uint32_t)(((lane & 7) ^ ((rl >> 1) & 7)) << 3)) * 2u;
    }
#if defined(__HIP_DEVICE_COMPILE__)
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(is_a ? A : W), 0, (uint32_t)(is_a ? M : N) * (uint32_t)K * 2u, 0x00020000);
#endif
    [[maybe_unused]] const uint32_t base = is_a ? 0u : 32u * GB_K * 2u;   // (not used by the host's pass over this)
    auto issue = [&](int t, int pos) {
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)(gsm + pos * SLAB + base + g * 1024), 16, off[g], (t < nk ? t : nk - 1) * (GB_K * 2), 0, 0);
#endif
    };
    for (int t = 0; t < kFewRing; ++t) issue(t, t);
    wait_vmem_upto<(kFewRing - 1) * 4>();
    block_barrier();                                           // k-tile 0 is there
    int pos = 0;
    for (int kt = 0; kt + 1 < nk; ++kt) {
      wait_vmem_upto<(kFewRing - 2) * 4>();
      block_barrier();                                         // k-tile kt + 1 is there, and kt has been read: its place is free
      issue(kt + kFewRing, pos);
      pos = pos + 1 == kFewRing ? 0 : pos + 1;
    }
    wait_vmem();
    return;
  }
  typedef __attribute__((address_space(3))) unsigned char lds_byte;
  typedef __attribute__((address_space(3))) const bf16x8 lds_bf16x8;
  uint32_t ra[4];                                              // LDS addresses of this lane's reads of A in place 0; W's are 4 KB behind
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) ra[ks] = (uint32_t)(uintptr_t)(lds_byte*)gsm + (uint32_t)(l32 * GB_K * 2 + (((2 * ks + half) ^ ((l32 >> 1) & 7)) << 4));
  // what the epilogue needs is requested first
  const int n = n0 + l32, mb = m0 + 4 * half;
  const float bv = bias && n < N ? to_f32(bias[n]) : 0.f;
  float old[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) old[v] = MODE == EPI_RESID ? resid[(size_t)min(mb + 8 * (v >> 2) + (v & 3), M - 1) * N + min(n, N - 1)] : 0.f;
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  struct Frags { bf16x8 a[4], b[4]; };
  auto read = [&](int pos, Frags& f) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      f.a[ks] = *(lds_bf16x8*)(uintptr_t)(ra[ks] + (uint32_t)(pos * SLAB));
      f.b[ks] = *(lds_bf16x8*)(uintptr_t)(ra[ks] + (uint32_t)(pos * SLAB) + 32 * GB_K * 2);
    }
  };
  auto fixed = [&]() {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_sched_barrier(0);
#endif
  };
  auto multiply = [&](const Frags& f) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[ks], f.b[ks], acc, 0, 0, 0);
  };
  Frags f0, f1;
  int pos = 0;
  // k-tile kt is in `cur`; the next one is read while it is multiplied
  auto turn = [&](const Frags& cur, Frags& next) {
    pos = pos + 1 == kFewRing ? 0 : pos + 1;
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_s_waitcnt(0xC07F);                        // lgkmcnt(0): k-tile kt has been read
#endif
    fixed();
    block_barrier();
    read(pos, next);
    fixed();
    multiply(cur);
    fixed();
  };
  block_barrier();
  read(0, f0);
  int kt = 0;
  for (; kt + 2 < nk; kt += 2) { turn(f0, f1); turn(f1, f0); }
  if (kt + 1 < nk) { turn(f0, f1); multiply(f1); } else multiply(f0);
  if (MODE == EPI_RESID) arrived(old);
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int m = mb + 8 * (v >> 2) + (v & 3);
    if (m < M && n < N) {
      if (MODE == EPI_RESID) reinterpret_cast<float*>(out)[(size_t)m * N + n] = old[v] + (acc[v] + bv);
      else epilogue_bf16<MODE>(out, (size_t)m * N + n, acc[v] + bv);
    }
  }
}

static hipError_t launch_gemm_bf16_few(const bf16_t* A, const bf16_t* W, const bf16_t* bias, void* out, int epi, int M, int N, int K, hipStream_t s, int models, const GemmTwin& tw, const float* resid) {
  constexpr int lds = kFewRing * 64 * GB_K * 2;
  const int64_t tiles = (int64_t)((M + 31) / 32) * ((N + 31) / 32) * models;
  const dim3 grid((unsigned)((tiles + 7) / 8 * 8));
#define ZGR_FEW(MODE)                                                                                                                             \
  {                                                                                                                                               \
    static std::atomic<bool> attr_set{false};   /* set twice by racing threads at worst: the call is idempotent */                                \
    auto kern = gemm_bf16_few_kernel<MODE>;                                                                                                       \
    if (!attr_set) {                                                                                                                              \
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);                   \
      if (e != hipSuccess) return e;                                                                                                              \
      attr_set = true;                                                                                                                            \
    }                                                                                                                                             \
    hipLaunchKernelGGL(kern, grid, dim3(192), lds, s, A, W, M, N, K, out, bias, tw, models, resid);                                               \
  }
  switch (epi) {
    case EPI_STORE: ZGR_FEW(EPI_STORE) break;
    case EPI_GELU:  ZGR_FEW(EPI_GELU) break;
    case EPI_RELU:  ZGR_FEW(EPI_RELU) break;
    case EPI_RESID: ZGR_FEW(EPI_RESID) break;
    default:        ZGR_FEW(EPI_F32) break;
  }
#undef ZGR_FEW
  return hipGetLastError();
}

// ------------------------------------------------------------------ attention
// fp32 on the matrix cores (v_mfma_f32_32x32x2_f32), for fp32 storage and for the head sizes the bf16 kernel below does not take (heads
// of 8 in part only, see launch_attention_t).  One wave per 32 queries of a head, keys in blocks of 32: S^T = K Q^T, then O^T += V^T P^T, everything in registers.  A lane supplies
// half a row of K and of Q (the contraction index is split as d = half DH/2 + s), holds 16 keys of one query column of S^T, and its
// probabilities are the second product's operand as they are: instruction v sums over the keys 8 (v / 4) + 4 half + v % 4, in which order
// the rows of V are loaded.  Operands come straight from global memory: V while S^T is formed, the next block's K behind it.
// Bound by load latency on short sequences and by the fp32 matrix rate on long ones.  (One thread per query with its row in registers left
// 51 of 64 lanes idle at 77 tokens and walked the keys one by one: 75 us per layer for 60 heads of 64, now 11;
// 8 x 4 heads of 32 at 64 tokens: 34 us, now 6.)
template <typename T> struct alignas(sizeof(T) * 4) Quad { T e[4]; };
template <typename T, int N> __device__ __forceinline__ void load_row(const T* p, float (&f)[N]) {
#pragma unroll
  for (int i = 0; i < N; i += 4) {
    const Quad<T> q = *reinterpret_cast<const Quad<T>*>(p + i);
#pragma unroll
    for (int j = 0; j < 4; ++j) f[i + j] = to_f32(q.e[j]);
  }
}
template <typename T, int DH>
__global__ void __launch_bounds__(64, 2) attention_f32_kernel(const T* __restrict__ qkv, T* __restrict__ ctx, const int32_t* __restrict__ lengths,
                                                           int seq, int d, int n_head, int causal, int heads, int n_len) {
  constexpr int HK = DH / 2, F = DH > 32 ? DH / 32 : 1;
  const int lane = threadIdx.x, l32 = lane & 31, half = lane >> 5;
  // causal: the last query blocks have the most keys and are handed out first
  const int qblocks = (seq + 31) / 32, bh = (int)blockIdx.x % heads, qi0 = (int)blockIdx.x / heads;
  const int q0 = 32 * (causal ? qblocks - 1 - qi0 : qi0), qi = q0 + l32;
  const int h = bh % n_head, b = bh / n_head;
  const size_t ld = (size_t)3 * d;
  const T* base = qkv + (size_t)b * seq * ld + (size_t)h * DH;
  int kend = lengths ? lengths[b % n_len] : seq;                     // visible to every query; then the causal mask
  kend = kend < seq ? kend : seq;
  const int last = causal && q0 + 32 < kend ? q0 + 32 : kend;        // keys of this wave
  float q[HK], k[HK];
  load_row(base + (size_t)(qi < seq ? qi : seq - 1) * ld + half * HK, q);
  f32x16 o[F];
#pragma unroll
  for (int f = 0; f < F; ++f)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[f][v] = 0.f;
  float mx = -INFINITY, den = 0.f;
  const float scale_log2 = 1.44269504088896341f / sqrtf((float)DH);
  // a key past the end repeats the last one: its probability is zero
  auto k_row = [&](int k0) { const int key = k0 + l32; return base + (size_t)(key < last ? key : last - 1) * ld + d + half * HK; };
  if (last > 0) load_row(k_row(0), k);
  uint32_t wild = 0;                                                 // bit v F + f: vv[v][f] of the block on the diagonal is infinite or NaN
  for (int k0 = 0; k0 < last; k0 += 32) {
    float vv[16][F];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int key = k0 + 8 * (v >> 2) + 4 * half + (v & 3);
      const T* vr = base + (size_t)(key < last ? key : last - 1) * ld + 2 * d;
#pragma unroll
      for (int f = 0; f < F; ++f) vv[v][f] = DH >= 32 || l32 < DH ? to_f32(vr[32 * f + l32]) : 0.f;
    }
    f32x16 s;
#pragma unroll
    for (int v = 0; v < 16; ++v) s[v] = 0.f;
#pragma unroll
    for (int i = 0; i < HK; ++i) s = __builtin_amdgcn_mfma_f32_32x32x2f32(k[i], q[i], s, 0, 0, 0);
    if (k0 + 32 < last) load_row(k_row(k0 + 32), k);
    float mloc = -INFINITY;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int key = k0 + 8 * (v >> 2) + 4 * half + (v & 3);
      s[v] = key < last && (!causal || key <= qi) ? s[v] * scale_log2 : -INFINITY;
      mloc = fmaxf(mloc, s[v]);
    }
    mloc = fmaxf(mloc, __shfl_xor(mloc, 32, 64));
    const float mnew = fmaxf(mx, mloc), msafe = mnew == -INFINITY ? 0.f : mnew;
    const float corr = __builtin_amdgcn_exp2f(mx - msafe);           // mx = -inf -> 0
    float sum = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) { s[v] = __builtin_amdgcn_exp2f(s[v] - msafe); sum += s[v]; }
    den = den * corr + sum;
    mx = mnew;
    // The block on the diagonal (the wave's last) holds keys that some of its queries do not see.  Their probability is zero, but zero
    // times an infinite V would be NaN: such entries go into the product as zeros, and what the queries that do see the key get is made infinite after the loop.
    if (causal && k0 == q0) {
      float zero = 0.f;                                              // stays zero while every entry is finite
#pragma unroll
      for (int v = 0; v < 16; ++v)
#pragma unroll
        for (int f = 0; f < F; ++f) zero = __builtin_fmaf(vv[v][f], 0.f, zero);
      if (__ballot(!(zero == 0.f))) {
#pragma unroll
        for (int v = 0; v < 16; ++v)
#pragma unroll
          for (int f = 0; f < F; ++f) if (!__builtin_isfinite(vv[v][f])) { wild |= 1u << (v * F + f); vv[v][f] = 0.f; }
      }
    }
#pragma unroll
    for (int f = 0; f < F; ++f)
#pragma unroll
      for (int v = 0; v < 16; ++v) o[f][v] *= corr;
#pragma unroll
    for (int v = 0; v < 16; ++v)
#pragma unroll
      for (int f = 0; f < F; ++f) o[f] = __builtin_amdgcn_mfma_f32_32x32x2f32(vv[v][f], s[v], o[f], 0, 0, 0);
  }
  if (__ballot(wild != 0)) {                                         // 3e38 times 3e38 is infinite, and 0 times it is 0
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int key = q0 + 8 * (v >> 2) + 4 * half + (v & 3);
      const float sees = key < last && key <= qi ? 3e38f : 0.f;
#pragma unroll
      for (int f = 0; f < F; ++f) o[f] = __builtin_amdgcn_mfma_f32_32x32x2f32((wild >> (v * F + f)) & 1u ? 3e38f : 0.f, sees, o[f], 0, 0, 0);
    }
  }
  den += __shfl_xor(den, 32, 64);
  if (qi < seq) {
    const float inv = den > 0.f ? 1.0f / den : 0.f;
    T* orow = ctx + ((size_t)b * seq + qi) * d + (size_t)h * DH;
#pragma unroll
    for (int f = 0; f < F; ++f)
#pragma unroll
      for (int v4 = 0; v4 < 4; ++v4) {
        const int c = 32 * f + 8 * v4 + 4 * half;                    // lane holds four consecutive entries of its query's row
        Quad<T> r;
#pragma unroll
        for (int i = 0; i < 4; ++i) from_f32(o[f][4 * v4 + i] * inv, r.e[i]);
        if (c < DH) *reinterpret_cast<Quad<T>*>(orow + c) = r;
      }
  }
}

// The same attention key by key on the vector unit: one thread per query row, one block per (batch, head, 256-query chunk), keys and
// values through LDS in chunks of 32.  The forward half of the cloud's backward pass keeps it (keep_order below), and small heads where it is the faster one.
template <typename T, int DH>
__global__ void __launch_bounds__(256) attention_kernel(const T* __restrict__ qkv, T* __restrict__ ctx, const int32_t* __restrict__ lengths,
                                                        int seq, int d, int n_head, int causal, int n_len) {
  constexpr int KC = 32;
  __shared__ float Ks[KC][DH], Vs[KC][DH];
  const int chunks = (seq + 255) / 256;
  const int qc = blockIdx.x % chunks, h = (blockIdx.x / chunks) % n_head, b = blockIdx.x / (chunks * n_head);
  const int qi = qc * 256 + threadIdx.x;
  const bool active = qi < seq;
  const int len = lengths ? lengths[b % n_len] : seq;
  const size_t ld = (size_t)3 * d;
  const T* base = qkv + (size_t)b * seq * ld + (size_t)h * DH;
  float q[DH], acc[DH];
  const float scale = 1.0f / sqrtf((float)DH);
#pragma unroll
  for (int i = 0; i < DH; ++i) { q[i] = active ? to_f32(base[(size_t)qi * ld + i]) * scale : 0.f; acc[i] = 0.f; }
  float mx = -INFINITY, den = 0.f;
  int kend = len < seq ? len : seq;
  if (causal) { const int last = qc * 256 + 255; kend = kend < last + 1 ? kend : last + 1; }
  for (int k0 = 0; k0 < kend; k0 += KC) {
    __syncthreads();
    for (int i = threadIdx.x; i < KC * DH; i += 256) {
      const int r = i / DH, c = i - r * DH;
      const int kj = k0 + r;
      Ks[r][c] = kj < seq ? to_f32(base[(size_t)kj * ld + d + c]) : 0.f;
      Vs[r][c] = kj < seq ? to_f32(base[(size_t)kj * ld + 2 * d + c]) : 0.f;
    }
    __syncthreads();
    if (!active) continue;
    for (int r = 0; r < KC; ++r) {
      const int kj = k0 + r;
      if (kj >= kend || (causal && kj > qi)) break;
      float s = 0.f;
#pragma unroll
      for (int i = 0; i < DH; ++i) s = __builtin_fmaf(q[i], Ks[r][i], s);
      const float nm = fmaxf(mx, s);
      const float corr = __expf(mx - nm), p = __expf(s - nm);
      den = den * corr + p;
#pragma unroll
      for (int i = 0; i < DH; ++i) acc[i] = __builtin_fmaf(p, Vs[r][i], acc[i] * corr);
      mx = nm;
    }
  }
  if (active) {
    T* o = ctx + ((size_t)b * seq + qi) * d + (size_t)h * DH;
    const float inv = den > 0.f ? 1.0f / den : 0.f;
#pragma unroll
    for (int i = 0; i < DH; ++i) from_f32(acc[i] * inv, o[i]);
  }
}

// MFMA attention for bf16 storage and head size 64.  One block = 32 NW queries of one (batch, head), 32 per wave; the keys come in stages
// through two LDS buffers: the next stage's K and V rows are on their way to registers while this one's are multiplied, one barrier a stage.
// A wave walks the keys in blocks of 32, computing S^T = K Q^T and O^T += V^T P^T with v_mfma_f32_32x32x16_bf16.  In the S^T
// result a lane holds one query column and 16 keys in registers, so the softmax reductions run over
// registers plus one exchange with the partner lane (lane ^ 32); P goes straight from the accumulator
// registers into the B operand of the second product (the contraction order of that product is the
// accumulator's key order, which the V^T operand is read in as well).  V stays in rows: ds_read_b64_tr_b16 hands 16 lanes the columns of a
// 4 x 16 piece.  Bound by the vector unit (exponentials, masks) on long sequences, by the transfer of q, k, v on short ones.
// 128 heads at 2047 tokens 165 -> 119 us (512 keys staged at a time, V transposed by 2-byte stores, no load under the products), 96 heads at 513 tokens
// 20.5 -> 17.4, 512 heads at 256 tokens 20.7 -> 19.0, 384 at 128 tokens 10.6 -> 9.1; the results keep their bits.  Stages of 128 keys under eight
// waves: the two that are requested at the start hold a 256-token sequence (2048 heads of it 42.2 -> 37.4 us; a first form with stages of 64, one requested at
// a time and waited for in front of the products, 46.5).
constexpr int AT_LDK = 64 + 8;          // K row stride (bf16): 144 B
typedef short i16x4 __attribute__((ext_vector_type(4)));
// columns of a piece of 4 rows of 16 entries: lane i of 16 supplies where entries 4 (i % 4) .. + 4 of row i / 4 lie and receives entry i of each row
__device__ __forceinline__ uint2 lds_columns(const bf16_t* p) {
  return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)const_cast<bf16_t*>(p)));
}
// the larger of a lane's value and its partner's (lane ^ 32)
__device__ __forceinline__ float max_of_halves(float v) {
  const auto w = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(w[0]), __uint_as_float(w[1]));
}
// NW waves per block, 32 queries each: with NW = 8 one block covers 256 queries of a head, so K and V of a
// 256-token sequence are staged once per head instead of once per 128 queries.
template <int DH, int NW>
__global__ void __launch_bounds__(64 * NW, 4) attention_mfma_kernel(const bf16_t* __restrict__ qkv, bf16_t* __restrict__ ctx, const int32_t* __restrict__ lengths,
                                                                    int seq, int d, int n_head, int causal, int n_len) {
  static_assert(DH == 64, "head size 64");
  constexpr int QB = 32 * NW, NT = 64 * NW;                     // queries and threads per block
  constexpr int AT_KEYS = 16 * NW, PER = AT_KEYS * 8 / NT;      // keys of a stage, 16-byte pieces of its K (and V) per thread
  __shared__ __attribute__((aligned(16))) bf16_t Ks[2][AT_KEYS * AT_LDK];
  __shared__ __attribute__((aligned(16))) bf16_t Vs[2][AT_KEYS * DH];      // row r's halves are exchanged where r / 2 is odd: four rows of 16 entries then lie in 64 different banks
  const int qblocks = (seq + QB - 1) / QB;
  // Under the causal mask a query block's work grows with its position: the blocks are handed out longest first (all heads'
  // last query blocks, then the ones before, ...), so that the short ones fill the gaps at the end of the launch.
  const int heads = gridDim.x / qblocks;
  const int qb = (causal && qblocks > 1) ? qblocks - 1 - (int)blockIdx.x / heads : (int)blockIdx.x % qblocks;
  const int bh = (causal && qblocks > 1) ? (int)blockIdx.x % heads : (int)blockIdx.x / qblocks;
  const int h = bh % n_head, b = bh / n_head;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, half = lane >> 5;
  const int len = lengths ? min(lengths[b % n_len], seq) : seq;
  const size_t ld = (size_t)3 * d;
  const bf16_t* base = qkv + (size_t)b * seq * ld + (size_t)h * DH;
  // keys this block can need, rounded up to 32
  int kend = len;
  if (causal) kend = min(kend, qb * QB + QB);
  const int kblocks = (kend + 31) / 32;
  // this wave's queries: B operand of S^T = K Q^T, lane (query l32, k-group half) holds Q[q][16 s + 8 half .. +8]
  // Under the causal mask a wave's work grows with the position of its queries.  Waves w and w + 4 share a SIMD, so
  // with eight waves the upper four take their query groups in reverse order: every SIMD then holds the same total.
  const int qgroup = (NW == 8 && causal && wave >= 4) ? 11 - wave : wave;
  const int q0 = qb * QB + qgroup * 32;
  const int qi = q0 + l32;
  bf16x8 qf[DH / 16];
#pragma unroll
  for (int s4 = 0; s4 < DH / 16; ++s4) {
    qf[s4] = *reinterpret_cast<const bf16x8*>(base + (size_t)min(qi, seq - 1) * ld + s4 * 16 + half * 8);
  }
  f32x16 o[DH / 32];
#pragma unroll
  for (int f = 0; f < DH / 32; ++f)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[f][v] = 0.f;
  float mx = -INFINITY, lsum = 0.f;
  const float scale_log2 = 1.44269504088896341f / sqrtf((float)DH);
  int wave_kblocks = kblocks;
  if (causal) wave_kblocks = min(kblocks, (q0 + 31) / 32 + 1);
  if (q0 >= seq) wave_kblocks = 0;
  struct Pieces { planes_u32x4 k[PER], v[PER]; };
  auto request = [&](Pieces& t, int stage) {                            // without branches: the waits for these loads are then counted; beyond seq the last row again (masked)
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      const int i = tid + p * NT, key = min(stage * AT_KEYS + (i >> 3), seq - 1);
      const bf16_t* row = base + (size_t)key * ld + d + (i & 7) * 8;
      t.k[p] = *reinterpret_cast<const planes_u32x4*>(row);
      t.v[p] = *reinterpret_cast<const planes_u32x4*>(row + d);
    }
  };
  auto put = [&](const Pieces& t, int buf) {
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      const int i = tid + p * NT, r = i >> 3, c = (i & 7) * 8;
      *reinterpret_cast<planes_u32x4*>(Ks[buf] + r * AT_LDK + c) = t.k[p];
      *reinterpret_cast<planes_u32x4*>(Vs[buf] + r * DH + (c ^ ((r & 2) << 4))) = t.v[p];
    }
  };
  const int i16 = lane & 15, v_row = ((i16 >> 2) + 4 * half) * DH + (lane & 16) + 4 * (i16 & 3), v_swap = (i16 & 8) << 2;
  const int stages = max(1, (kblocks * 32 + AT_KEYS - 1) / AT_KEYS);    // the same for every wave of the block; one that no wave needs where no key is visible, so that no path leaves q's loads pending
  // The first two stages are requested together (the second may be past the last one: its rows are not used); from then on the one after next is
  // requested as soon as the one before it lies in LDS.
  Pieces next;
  {
    Pieces first;
    request(first, 0);
    request(next, 1);
    put(first, 0);
  }
  __syncthreads();
  for (int st = 0; st < stages; ++st) {
    const bf16_t* K = Ks[st & 1];
    const bf16_t* V = Vs[st & 1] + v_row;
    for (int kb = st * (AT_KEYS / 32); kb < min((st + 1) * (AT_KEYS / 32), wave_kblocks); ++kb) {
      const int kl = kb * 32 - st * AT_KEYS;                              // the block's first key within the stage
      f32x16 sacc;
#pragma unroll
      for (int v = 0; v < 16; ++v) sacc[v] = 0.f;
#pragma unroll
      for (int s4 = 0; s4 < DH / 16; ++s4) {
        const bf16x8 kf = *reinterpret_cast<const bf16x8*>(K + (kl + l32) * AT_LDK + s4 * 16 + half * 8);
        sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[s4], sacc, 0, 0, 0);
      }
      // lane: query qi, keys kb*32 + 8*(v/4) + 4*half + v%4; scores in log2 units
      float sv[16], mloc = -INFINITY;
      if (kb * 32 + 31 < len && (!causal || kb * 32 + 31 <= q0)) {      // every key of the block is visible to every query of the wave
#pragma unroll
        for (int v = 0; v < 16; ++v) { sv[v] = sacc[v] * scale_log2; mloc = fmaxf(mloc, sv[v]); }
      } else {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int key = kb * 32 + 8 * (v >> 2) + 4 * half + (v & 3);
          const bool ok = key < len && (!causal || key <= qi);
          sv[v] = ok ? sacc[v] * scale_log2 : -INFINITY;
          mloc = fmaxf(mloc, sv[v]);
        }
      }
      mloc = max_of_halves(mloc);
      const float mnew = fmaxf(mx, mloc);
      const float msafe = mnew == -INFINITY ? 0.f : mnew;
      // v_exp_f32 directly: the arguments are <= 0 (or -inf, which gives 0), so the library routine's range handling is not needed
      const float corr = __builtin_amdgcn_exp2f(mx - msafe);            // mx = -inf -> 0
      float psum = 0.f;
      union { uint32_t w[4]; bf16x8 v; } pk[2];                          // P^T operand: two probabilities per conversion
#pragma unroll
      for (int v = 0; v < 16; v += 2) {
        const float p0 = __builtin_amdgcn_exp2f(sv[v] - msafe), p1 = __builtin_amdgcn_exp2f(sv[v + 1] - msafe);
        psum += p0 + p1;
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        typedef float f32x2 __attribute__((ext_vector_type(2)));
        const f32x2 pp = {p0, p1};
        pk[v >> 3].w[(v & 7) >> 1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pp, bf16x2));
      }
      const bf16x8 pf[2] = {pk[0].v, pk[1].v};
      lsum = lsum * corr + psum;
      mx = mnew;
      if (__builtin_amdgcn_ballot_w64(corr != 1.0f) != 0) {              // nothing to rescale while no lane's maximum moved
#pragma unroll
        for (int f = 0; f < DH / 32; ++f)
#pragma unroll
          for (int v = 0; v < 16; ++v) o[f][v] *= corr;
      }
      // O^T += V^T P^T: A operand lane (dh row 32 f + l32, half) reads the keys in the accumulator's order
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
        for (int f = 0; f < DH / 32; ++f) {
          const bf16_t* vr = V + (kl + ks * 16) * DH + ((f * 32) ^ v_swap);
          const uint2 lo = lds_columns(vr), hi = lds_columns(vr + 8 * DH);
          uint4 t = make_uint4(lo.x, lo.y, hi.x, hi.y);
          o[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<bf16x8*>(&t), pf[ks], o[f], 0, 0, 0);
        }
      }
    }
    if (st + 1 == stages) break;
    put(next, (st + 1) & 1);                        // its readers of two stages ago are behind the last barrier
    request(next, st + 2);
    __syncthreads();
  }
  lsum += __shfl_xor(lsum, 32, 64);
  if (qi < seq) {
    const float inv = lsum > 0.f ? 1.0f / lsum : 0.f;
    bf16_t* orow = ctx + ((size_t)b * seq + qi) * d + (size_t)h * DH;
#pragma unroll
    for (int f = 0; f < DH / 32; ++f)
#pragma unroll
      for (int v4 = 0; v4 < 4; ++v4) {
        uint16_t pk[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) { bf16_t t; from_f32(o[f][v4 * 4 + i] * inv, t); pk[i] = t.bits; }
        *reinterpret_cast<uint2*>(orow + f * 32 + 8 * v4 + 4 * half) = *reinterpret_cast<uint2*>(pk);
      }
  }
}

// ------------------------------------------------------------------ losses
// Cross-entropy of one row of fp32 logits [n]: loss = logsumexp - logit[target]; target < 0: row skipped (loss 0).  A block holds
// THREADS MAXE entries in registers, so the row is read once (256 threads reading it twice: 135 us for 385 rows of 50272, now 26);
// entries beyond those are read again.
template <int THREADS, int MAXE>
__global__ void __launch_bounds__(THREADS) ce_rows_kernel(const float* __restrict__ logits, const int32_t* __restrict__ targets, float* __restrict__ row_loss, int n, int M, int64_t second) {
  constexpr int WAVES = THREADS / 64;
  __shared__ float red[WAVES];
  const int m = blockIdx.x, tid = threadIdx.x;
  int tgt = targets[m < M ? m : m - M];                              // two models: the same targets, row losses `second` floats further on
  row_loss += m < M ? m : m - M + second;
  if (tgt < 0) { if (tid == 0) *row_loss = 0.f; return; }          // uniform over the block
  tgt = tgt >= n ? n - 1 : tgt;
  const float* row = logits + (size_t)m * n;
  auto across = [&](float v, bool maximum) {                          // the block's waves, in order
    v = maximum ? wave_max(v) : wave_sum(v);
    __syncthreads();
    if ((tid & 63) == 0) red[tid >> 6] = v;
    __syncthreads();
    float r = red[0];
    for (int w = 1; w < WAVES; ++w) r = maximum ? fmaxf(r, red[w]) : r + red[w];
    return r;
  };
  float v[MAXE], mx = -INFINITY;
#pragma unroll
  for (int u = 0; u < MAXE; ++u) {
    const int i = tid + THREADS * u;
    v[u] = i < n ? row[i] : -INFINITY;
    mx = fmaxf(mx, v[u]);
  }
  for (int i = tid + THREADS * MAXE; i < n; i += THREADS) mx = fmaxf(mx, row[i]);
  mx = across(mx, true);
  float s = 0.f;
#pragma unroll
  for (int u = 0; u < MAXE; ++u) s += tid + THREADS * u < n ? expf(v[u] - mx) : 0.f;
  for (int i = tid + THREADS * MAXE; i < n; i += THREADS) s += expf(row[i] - mx);
  s = across(s, false);
  if (tid == 0) *row_loss = logf(s) + mx - row[tgt];
}

// Combines the cross-entropy partials of one row: loss = log(sum_i s_i exp(m_i - M)) + M - logit[target].
__global__ void __launch_bounds__(256) ce_combine_kernel(const float2* __restrict__ part, int n_part, const int32_t* __restrict__ targets,
                                                         const float* __restrict__ tlogit, float* __restrict__ row_loss, int M, int64_t second) {
  __shared__ float red[4];
  const int m = blockIdx.x;
  row_loss += m < M ? m : m - M + second;
  if (targets[m < M ? m : m - M] < 0) { if (threadIdx.x == 0) *row_loss = 0.f; return; }
  const float2* row = part + (size_t)m * n_part;
  float mx = -INFINITY;
  for (int i = threadIdx.x; i < n_part; i += 256) mx = fmaxf(mx, row[i].x);
  mx = block_max(mx, red);
  float s = 0.f;
  for (int i = threadIdx.x; i < n_part; i += 256) s += row[i].y * expf(row[i].x - mx);
  s = block_sum(s, red);
  if (threadIdx.x == 0) *row_loss = logf(s) + mx - tlogit[m];
}

// mean of n_rows losses (ignoring the skipped ones by dividing by `count`), accumulated in fp64; a block per model
__global__ void __launch_bounds__(256) mean_f64_kernel(const float* __restrict__ v, int n, double inv_count, double* __restrict__ out, int64_t second) {
  __shared__ double red[256];
  v += blockIdx.x * second;
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) s += (double)v[i];
  red[threadIdx.x] = s;
  __syncthreads();
  if (threadIdx.x >= 64) return;                                   // the first wave: the upper half onto the lower, again and again
  s = (red[threadIdx.x] + red[threadIdx.x + 128]) + (red[threadIdx.x + 64] + red[threadIdx.x + 192]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
  if (threadIdx.x == 0) out[blockIdx.x] = s * inv_count;
}

// classification head on token 0 of every sequence: logits[b][c] = h[b*seq] . Wc[c] + bc[c]
template <typename T>
__global__ void __launch_bounds__(64) cls_head_kernel(const T* __restrict__ h, const T* __restrict__ Wc, const T* __restrict__ bc, float* __restrict__ logits,
                                                      int seq, int d, int n_class, int batch, int64_t wb) {
  const int b = blockIdx.x / n_class, c = blockIdx.x % n_class;
  const T* x = h + (size_t)b * seq * d;
  const T* w = of_model(Wc, b >= batch, wb) + (size_t)c * d;
  float s = 0.f;
  for (int i = threadIdx.x; i < d; i += 64) s = __builtin_fmaf(to_f32(x[i]), to_f32(w[i]), s);
  s = wave_sum(s);
  if (threadIdx.x == 0) logits[b * n_class + c] = s + to_f32(of_model(bc, b >= batch, wb)[c]);
}

// least squares: row_loss[b] = sum_o (pred[b][o] - Y[b][o])^2 / 2
__global__ void __launch_bounds__(256) lsq_rows_kernel(const float* __restrict__ pred, const float* __restrict__ Y, float* __restrict__ row_loss, int n_out, int batch, int64_t second) {
  __shared__ float red[4];
  const int b = blockIdx.x, by = b < batch ? b : b - batch;
  float s = 0.f;
  for (int i = threadIdx.x; i < n_out; i += 256) { const float r = pred[(size_t)b * n_out + i] - Y[(size_t)by * n_out + i]; s = __builtin_fmaf(r, r, s); }
  s = block_sum(s, red);
  if (threadIdx.x == 0) row_loss[b < batch ? b : by + second] = 0.5f * s;
}

// The same rows and their mean in one launch, a block of sixteen waves per model, a wave per row at a time; each row summed in fp64 and rounded once.
template <int THREADS>
__global__ void __launch_bounds__(THREADS) lsq_loss_kernel(const float* __restrict__ pred, const float* __restrict__ Y, float* __restrict__ row_loss, int n_out, int batch, double inv_count,
                                                           double* __restrict__ out, int64_t second) {
  __shared__ double red[THREADS / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  pred += (size_t)blockIdx.x * batch * n_out;
  row_loss += blockIdx.x * second;
  double sum = 0.0;
  for (int b = wave; b < batch; b += THREADS / 64) {
    const float* p = pred + (size_t)b * n_out;
    const float* y = Y + (size_t)b * n_out;
    double s = 0.0;
#pragma unroll 4
    for (int i = lane; i < n_out; i += 64) { const float r = p[i] - y[i]; s = __builtin_fma((double)r, (double)r, s); }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    const float row = (float)(0.5 * s);
    if (lane == 0) row_loss[b] = row;
    sum += (double)row;
  }
  if (lane == 0) red[wave] = sum;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < THREADS / 64; ++w) sum += red[w];
    out[blockIdx.x] = sum * inv_count;
  }
}

}  // namespace

// ------------------------------------------------------------------ host launchers
hipError_t launch_embed(int dtype, const int32_t* tok, const void* E, const void* Pe, float* x, int M, int seq, int d, int vocab, int32_t* targets, hipStream_t s, Twin tw) {
  if (dtype == 0) hipLaunchKernelGGL(embed_kernel<float>, dim3(M * tw.models), dim3(256), 0, s, tok, (const float*)E, (const float*)Pe, x, M, seq, d, vocab, tw.w, targets);
  else            hipLaunchKernelGGL(embed_kernel<bf16_t>, dim3(M * tw.models), dim3(256), 0, s, tok, (const bf16_t*)E, (const bf16_t*)Pe, x, M, seq, d, vocab, tw.w, targets);
  return hipGetLastError();
}

hipError_t launch_layernorm(int dtype, const float* x, const void* g, const void* b, void* out, int M, int d, float eps, hipStream_t s, float* xout, Twin tw) {
  const int rows = M * tw.models;
  if (d % 4 == 0 && d <= 2048 && (((uintptr_t)g | (uintptr_t)b | (uintptr_t)out | (uintptr_t)xout | (uintptr_t)tw.w) & 15) == 0) {
    const dim3 grid((unsigned)((rows + 3) / 4));
    if (dtype == 0) hipLaunchKernelGGL(layernorm_wave_kernel<float>, grid, dim3(256), 0, s, x, (const float*)g, (const float*)b, (float*)out, rows, d, eps, xout, M, tw.w);
    else            hipLaunchKernelGGL(layernorm_wave_kernel<bf16_t>, grid, dim3(256), 0, s, x, (const bf16_t*)g, (const bf16_t*)b, (bf16_t*)out, rows, d, eps, xout, M, tw.w);
    return hipGetLastError();
  }
  if (d % 4 == 0 && d <= 8192 && (((uintptr_t)g | (uintptr_t)b | (uintptr_t)out | (uintptr_t)xout | (uintptr_t)tw.w) & 15) == 0) {
    if (dtype == 0) hipLaunchKernelGGL(layernorm_reg_kernel<float>, dim3(rows), dim3(256), 0, s, x, (const float*)g, (const float*)b, (float*)out, d, eps, xout, M, tw.w);
    else            hipLaunchKernelGGL(layernorm_reg_kernel<bf16_t>, dim3(rows), dim3(256), 0, s, x, (const bf16_t*)g, (const bf16_t*)b, (bf16_t*)out, d, eps, xout, M, tw.w);
    return hipGetLastError();
  }
  if (dtype == 0) hipLaunchKernelGGL(layernorm_kernel<float>, dim3(rows), dim3(256), 0, s, x, (const float*)g, (const float*)b, (float*)out, d, eps, xout, M, tw.w);
  else            hipLaunchKernelGGL(layernorm_kernel<bf16_t>, dim3(rows), dim3(256), 0, s, x, (const bf16_t*)g, (const bf16_t*)b, (bf16_t*)out, d, eps, xout, M, tw.w);
  return hipGetLastError();
}

// Whether an fp32 projection goes to product.hip, which splits its sums among waves and blocks, rather than to the 64 x 64 tiles through LDS.
// That pays where the tiles leave CUs idle and the sum is long enough to share out; times of a product against those of the tiles, with GELU:
//   up to 128 tiles      0.8 at K = 128, 0.4 - 0.7 at 1024; even at 64, 1.1 below
//   129 to 256 tiles     3.2 at K = 32 (4096 x 256: 25 us against 8), 1.2 at 192, 1.03 at 384, 0.85 - 0.99 at 512, 0.65 at 4096
//   257 to 319 tiles     1.1 - 1.2 at K = 768, 1.05 - 1.08 at 1024, 0.95 at 2048 (eight waves a tile, a few CUs with a second round of them)
//   320 to 511 tiles     2.7 at K = 32, 1.2 at 128, 1.00 - 1.06 at 512, 0.94 - 1.01 at 768, 0.91 - 0.97 at 1024
// From 512 on the tiles are the faster form (2048 x 2304 x 768, 1152 tiles: 81 us against 93).
static bool product_is_faster(int M, int N, int K) {
  const int64_t tiles = (((int64_t)M + 63) / 64) * (((int64_t)N + 63) / 64);
  if (tiles >= 512) return false;
  return K >= (tiles <= 128 ? 64 : tiles <= 256 ? 512 : tiles < 320 ? 2048 : 768);
}

// Which fp32 projections (K a multiple of 32) go to the bf16 instructions' planes, by one model's tiles of 128 x 128 and of 64 x 64; the kernels below
// are the faster ones elsewhere (us with GELU, then those of the planes):
//   shared:   2048 x 4096 (512 tiles) at K = 64 35 / 24, at 512 86 / 63; 2048 x 2048 (256) at 128 19.6 / 22.6, at 256 28.4 / 27.8, at 512 46 / 39;
//             2048 x 1024 (128) at 512 26 / 33; 385 x 50272 x 768 (1572) 335 / 252, 4096 x 2048 x 8192 980 / 743
//   private:  1024 x 1024 (256 tiles) at K = 128 10.1 / 9.8, at 512 17.1 / 14.2; 512 x 1024 (128) at 256 8.8 / 10.4, at 512 12.3 / 12.7; 1280 x 1280 (400) at 256
//             17.1 / 19.7, at 512 25.9 / 24.7; 2048 x 1024 (512) at 512 26.0 / 27.6, with the residual at 1024 48 / 33; 385 x 768 (84) at 768 15.8 / 12.4, at 3072
//             46 / 32; 231 x 1024 (64) at 1024 12.0 / 15.1
static bool planes_shared(int64_t t128, int K) { return t128 >= 512 || (t128 >= 256 && K >= 256); }
static bool planes_private(int64_t t64, int K) { return t64 >= 72 && K >= (t64 > 128 && t64 <= 256 ? 192 : 640); }

int fp32_projection_form(int M, int N, int K, bool whole_rows, bool keep_order) {
  const int64_t t128 = (int64_t)((M + 127) / 128) * ((N + 127) / 128), t64 = (int64_t)((M + 63) / 64) * ((N + 63) / 64);
  if (!whole_rows) return F32_VECTOR;
  if (!keep_order && K % kPlaneK == 0) {
    if (planes_shared(t128, K)) return F32_PLANES_128;
    if (planes_private(t64, K)) return F32_PLANES_64;
  }
  if (t128 >= 512) return F32_TILES_128;                 // enough 128 x 128 tiles for two blocks on every CU
  return !keep_order && product_is_faster(M, N, K) ? F32_PRODUCT : F32_TILES_64;
}

// 32 x 32 tiles that all get a CU of their own
static bool few_tiles(int M, int N, int models) { return (int64_t)((M + 31) / 32) * ((N + 31) / 32) * models <= 256; }

hipError_t launch_gemm(int dtype, const void* A, const void* W, const void* bias, void* out, int epi, int M, int N, int K, hipStream_t s, float* scratch, size_t scratch_floats, bool keep_order, Twin tw, bool shared_a, const float* resid) {
  const float* from = resid ? resid : (const float*)out;
  GemmEpi ep{epi, out, bias, from};
  if (resid && resid != out) keep_order = true;          // the kernels that split sums add to out itself
  const int es = dtype == 0 ? 4 : 2, n = tw.models;
  const GemmTwin gt{shared_a ? 0 : (int64_t)M * K * es, tw.w, (int64_t)M * N * (epi == EPI_RESID || epi == EPI_F32 ? 4 : es), tw.w, 0};
  if (dtype == 0) {
    const float* a = (const float*)A; const float* w = (const float*)W;
    const dim3 t64((N + 63) / 64, (M + 63) / 64, n), t128((N + 127) / 128, (M + 127) / 128, n);
    switch (fp32_projection_form(M, N, K, K % 4 == 0 && (((uintptr_t)A | (uintptr_t)W | (uintptr_t)tw.w) & 15) == 0, keep_order)) {     // one model's sizes
      case F32_PLANES_128: return launch_gemm_planes<true>(a, w, M, N, K, ep, gt, n, s);
      case F32_PLANES_64:  return launch_gemm_planes<false>(a, w, M, N, K, ep, gt, n, s);
      case F32_TILES_128:  hipLaunchKernelGGL((gemm_f32_mfma_kernel<2, 16>), t128, dim3(256), 0, s, a, w, M, N, K, ep, gt); break;
      case F32_TILES_64:   hipLaunchKernelGGL((gemm_f32_mfma_kernel<1, 16>), t64, dim3(256), 0, s, a, w, M, N, K, ep, gt); break;
      case F32_PRODUCT: {
        ProductArgs p;
        p.A = A; p.lda = K; p.B = W; p.b_k = true; p.ldb = K; p.C = (float*)out; p.ldc = N; p.M = M; p.N = N; p.K = K;
        p.epilogue = epi; p.bias = (const float*)bias; p.scratch = scratch; p.scratch_floats = scratch_floats;
        p.batches = p.models = n; p.a_outer = gt.a / 4; p.b_outer = p.bias_outer = tw.w / 4; p.c_outer = (int64_t)M * N;
        return launch_product(p, s);
      }
      default: hipLaunchKernelGGL(gemm_f32_kernel, t64, dim3(256), 0, s, a, w, M, N, K, ep, gt); break;
    }
  } else {
    if (K % GB_K != 0) return hipErrorInvalidValue;
    const bf16_t* a = (const bf16_t*)A; const bf16_t* w = (const bf16_t*)W; const bf16_t* b = (const bf16_t*)bias;
    // largest tile that still gives every CU a block.  The tiles of both models count where there are two: their number is what fills the chip, and all forms
    // take the terms of a sum in the same order.
    const long t256 = (long)((M + 255) / 256) * ((N + 255) / 256) * n, t128x256 = (long)((M + 127) / 128) * ((N + 255) / 256) * n;
    if ((size_t)M * K >= ((size_t)1 << 31) || (size_t)N * K >= ((size_t)1 << 31)) return hipErrorInvalidValue;   // 32-bit byte offsets
    // 256 x 256 tiles unless their count leaves the last round of 256 CUs less than ~85 % full and 256 x 192 tiles fill it better
    const long t192 = (long)((M + 255) / 256) * ((N + 191) / 192) * n;
    auto fill = [](long t) { const long rounds = (t + 255) / 256; return (double)t / (double)(rounds * 256); };
    if (t256 >= 256 && (fill(t256) >= 0.85 || fill(t192) <= fill(t256))) return launch_gemm_bf16_t<256, 256, 2, 4, 64, 20, 1>(a, w, b, out, epi, M, N, K, s, n, gt, from);
    if (t192 >= 256 && N % 192 == 0) return launch_gemm_bf16_t<256, 192, 4, 2, 64, 20, 1>(a, w, b, out, epi, M, N, K, s, n, gt, from);
    if (t256 >= 256) return launch_gemm_bf16_t<256, 256, 2, 4, 64, 20, 1>(a, w, b, out, epi, M, N, K, s, n, gt, from);
    if (t128x256 >= 200) return launch_gemm_bf16_t<128, 256, 2, 4, 64, 20, 1>(a, w, b, out, epi, M, N, K, s, n, gt, from);
    // small problems.  More 128 x 128 tiles than CUs: the ping-pong loop on a short ring (64 KB, two blocks per CU, one block's
    // epilogue under the other's loop).  Fewer than half the CUs would get such a tile: 64 x 64 tiles with the plain loop
    // (four times the blocks, two of them per CU; 64 x 128 tiles were a few per cent slower).
    // In between (about one tile per CU): the ping-pong loop on the full ring.
    const long t128 = (long)((M + 127) / 128) * ((N + 127) / 128) * n;
    if (t128 > 256) return launch_gemm_bf16_t<128, 128, 2, 4, 64, 8, 1>(a, w, b, out, epi, M, N, K, s, n, gt, from);
    if (few_tiles(M, N, n)) return launch_gemm_bf16_few(a, w, b, out, epi, M, N, K, s, n, gt, from);
    if (t128 <= 128) return launch_gemm_bf16_t<64, 64, 2, 2, 64, 4>(a, w, b, out, epi, M, N, K, s, n, gt, from);
    return launch_gemm_bf16_t<128, 128, 2, 4, 64, 20, 1>(a, w, b, out, epi, M, N, K, s, n, gt, from);
  }
  return hipGetLastError();
}

hipError_t launch_product_group(const ProductGroup& g, hipStream_t s) {
  if (g.count == 0) return hipSuccess;
  if (g.count < 0 || g.count > kGroupedProducts || (g.fold != 1 && g.fold != 3)) return hipErrorInvalidValue;
  for (int j = 0; j < g.count; ++j) {
    const GroupedProduct& p = g.job[j];
    if (p.M < 1 || p.N < 1 || p.K < 1 || p.K % (GB_K * g.fold) || p.lda < p.K || p.ldw < p.K / g.fold) return hipErrorInvalidValue;
    if ((size_t)p.M * p.lda >= ((size_t)1 << 31) || (size_t)p.N * p.ldw >= ((size_t)1 << 31)) return hipErrorInvalidValue;      // 32-bit byte offsets
  }
  return g.fold == 1 ? launch_group_f<1>(g, s) : launch_group_f<3>(g, s);
}

// Some 24 k-tiles a slice and up to two blocks a CU, where the undivided product would leave half of the CUs without a tile of 128 x 128 (and takes tiles of 64 x 64): the
// gradients of the inputs of FC1 and of Q, K, V at 2048 tokens and 768 columns (sums of 3072 and 2304) 21.5 us on average, in two slices 16.3, and of the head
// (50304) 290, in five 185; the LayerNorm rules behind them 9.8 us with one part, 11.7 with two on average.  Where the slices' tiles are still so few that the group takes
// 64 x 64: the heads' passes of 512 tokens, 768 columns and a vocabulary of 12000 304 -> 273 us, of 3000 219 -> 215.  Whole passes of 64 to 2048 columns and 64 to 8192 tokens were
// nowhere slower than undivided beyond their noise of 2 % (1536 columns, 256 tokens 1226 -> 1159).  Off from fp64: 2.3e-7 of the norm where undivided 3.4e-7 (2048 x 768, sum of
// 3072), 6.4e-7 where 14.4e-7 (50304).
int product_slices(int M, int N, int K, int most) {
  const int64_t t128 = (int64_t)((M + 127) / 128) * ((N + 127) / 128);
  if (t128 > 128 || few_tiles(M, N, 1)) return 1;
  return (int)std::max<int64_t>(1, std::min<int64_t>({512 / t128, (K / GB_K + 12) / 24, most, kGroupedProducts}));
}
hipError_t launch_product_slices(const void* A, const void* W, float* out, int M, int N, int K, int slices, hipStream_t s) {
  const int per = (K / GB_K + slices - 1) / slices * GB_K;
  ProductGroup g;
  if (slices < 1 || slices > kGroupedProducts || K % GB_K || (int64_t)per * (slices - 1) >= K) return hipErrorInvalidValue;
  for (int i = 0; i < slices; ++i)
    g.job[g.count++] = GroupedProduct{(const bf16_t*)A + (size_t)i * per, (const bf16_t*)W + (size_t)i * per, out + (size_t)i * M * N, M, N, std::min(per, K - i * per), K, K};
  return launch_product_group(g, s);
}

// Vocabulary projection fused with the row-wise cross-entropy (bf16 storage): logits are never stored.
// part: float2 scratch of ce_partials_per_row(N) entries per row; tlogit: float [M].
int ce_partials_per_row(int N) { return ((N + 255) / 256) * 2; }

hipError_t launch_gemm_ce_bf16(const void* A, const void* W, const int32_t* targets, void* part, float* tlogit, float* row_loss, int M, int N, int K, hipStream_t s, Twin tw) {
  if (K % GB_K != 0 || (size_t)M * K >= ((size_t)1 << 31) || (size_t)N * K >= ((size_t)1 << 31)) return hipErrorInvalidValue;
  // transposed product: the kernel's rows are the N vocabulary entries, its columns the M tokens.  The tile of 256 x 256 multiplies mostly
  // nothing for a short prompt: up to 128 tokens take tiles of 128 vocabulary entries x 64 tokens with one wave across the entries, so that
  // there is one partial per 128 entries as well (50272 x 768, with the layer's own projections: 33 tokens 138 -> 94 us, 128 tokens 135 -> 91;
  // 9000 x 2048: 102 -> 85).
  // (One tile of 128 x 128 for 65 to 128 tokens reads the weights once instead of twice and was slower than the
  // large tile on wide models: 50272 x 2048 247 us against 232, now 160.)
  const bf16_t* w = (const bf16_t*)W; const bf16_t* a = (const bf16_t*)A;
  hipError_t e;
  int n_part = ce_partials_per_row(N);
  // the kernel's first operand is the parameters here, its second the tokens
  auto twin = [&](int parts) { return GemmTwin{tw.w, (int64_t)M * K * 2, (int64_t)M * parts * (int64_t)sizeof(float2), 0, (int64_t)M * 4}; };
  if (M <= 128) {
    n_part = (N + 127) / 128;
    e = launch_gemm_bf16_t<128, 64, 1, 2, 64, 3>(w, a, nullptr, part, EPI_CE, N, M, K, s, tw.models, twin(n_part), nullptr, targets, tlogit);
  } else {
    e = launch_gemm_bf16_t<256, 256, 2, 4, 64, 20, 1>(w, a, nullptr, part, EPI_CE, N, M, K, s, tw.models, twin(n_part), nullptr, targets, tlogit);
  }
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(ce_combine_kernel, dim3(M * tw.models), dim3(256), 0, s, (const float2*)part, n_part, targets, tlogit, row_loss, M, tw.row_loss);
  return hipGetLastError();
}

template <typename T>
static hipError_t launch_attention_t(const T* qkv, T* ctx, const int32_t* lengths, int batch, int seq, int d, int n_head, int causal, hipStream_t s, bool keep_order, int models) {
  const int dh = d / n_head;
  const int heads = batch * models * n_head;
  // Heads of 8 leave the matrix instructions three quarters empty.  bf16: key by key is the faster form nearly everywhere (1 x 2048 tokens of
  // 32 heads, no causal mask: 174 us against 188, 4 x 2047: 180 against 334, 128 x 33: 21 against 28; only with few waves, 64 x 128, does it lose,
  // 65 against 57).  fp32: only on long sequences without a causal mask that fill the chip (3 x 2047: 175 against 181, 4 x 2047: 182 against
  // 237; 8 x 1024: 151 against 144, 2 x 2047: 178 against 168).
  const bool by_key = dh == 8 && (sizeof(T) == 2 || (!causal && seq > 1024 && (int64_t)batch * n_head * ((seq + 31) / 32) >= 6144));
  if (keep_order || by_key) {
    const dim3 grid((unsigned)heads * (unsigned)((seq + 255) / 256));
    switch (dh) {
      case 8:   hipLaunchKernelGGL((attention_kernel<T, 8>), grid, dim3(256), 0, s, qkv, ctx, lengths, seq, d, n_head, causal, batch); break;
      case 16:  hipLaunchKernelGGL((attention_kernel<T, 16>), grid, dim3(256), 0, s, qkv, ctx, lengths, seq, d, n_head, causal, batch); break;
      case 32:  hipLaunchKernelGGL((attention_kernel<T, 32>), grid, dim3(256), 0, s, qkv, ctx, lengths, seq, d, n_head, causal, batch); break;
      case 64:  hipLaunchKernelGGL((attention_kernel<T, 64>), grid, dim3(256), 0, s, qkv, ctx, lengths, seq, d, n_head, causal, batch); break;
      default:  return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  const dim3 grid((unsigned)heads * (unsigned)((seq + 31) / 32));
  switch (dh) {
    case 8:   if constexpr (sizeof(T) == 4) hipLaunchKernelGGL((attention_f32_kernel<T, 8>), grid, dim3(64), 0, s, qkv, ctx, lengths, seq, d, n_head, causal, heads, batch); break;
    case 16:  hipLaunchKernelGGL((attention_f32_kernel<T, 16>), grid, dim3(64), 0, s, qkv, ctx, lengths, seq, d, n_head, causal, heads, batch); break;
    case 32:  hipLaunchKernelGGL((attention_f32_kernel<T, 32>), grid, dim3(64), 0, s, qkv, ctx, lengths, seq, d, n_head, causal, heads, batch); break;
    case 64:  hipLaunchKernelGGL((attention_f32_kernel<T, 64>), grid, dim3(64), 0, s, qkv, ctx, lengths, seq, d, n_head, causal, heads, batch); break;
    default:  return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_attention(int dtype, const void* qkv, void* ctx, const int32_t* lengths, int batch, int seq, int d, int n_head, int causal, hipStream_t s, bool keep_order, int models) {
  if (dtype == 1 && d / n_head == 64 && d % 8 == 0) {
    if (seq > 128) {      // 256 queries per block: the keys of a head are staged once per 256 queries
      const int grid = batch * models * n_head * ((seq + 255) / 256);
      hipLaunchKernelGGL((attention_mfma_kernel<64, 8>), dim3(grid), dim3(512), 0, s, (const bf16_t*)qkv, (bf16_t*)ctx, lengths, seq, d, n_head, causal, batch);
    } else {
      const int grid = batch * models * n_head * ((seq + 127) / 128);
      hipLaunchKernelGGL((attention_mfma_kernel<64, 4>), dim3(grid), dim3(256), 0, s, (const bf16_t*)qkv, (bf16_t*)ctx, lengths, seq, d, n_head, causal, batch);
    }
    return hipGetLastError();
  }
  if (dtype == 0) return launch_attention_t<float>((const float*)qkv, (float*)ctx, lengths, batch, seq, d, n_head, causal, s, keep_order, models);
  return launch_attention_t<bf16_t>((const bf16_t*)qkv, (bf16_t*)ctx, lengths, batch, seq, d, n_head, causal, s, keep_order, models);
}

bool attention_head_dim_supported(int dh) { return dh == 8 || dh == 16 || dh == 32 || dh == 64; }

// The smallest block that holds the row: threads without an entry, and iterations without one, cost as much as those with (2048 rows of 33 / 4097 /
// 10000 / 20000, with the target and mean launches: 28 / 88 / 88 / 91 us when every row took 1024 threads of 4 or 50, now 20 / 28 / 37 / 58; 256
// threads reading the row twice: 20 / 31 / 48 / 76).
hipError_t launch_ce_rows(const float* logits, const int32_t* targets, float* row_loss, int M, int n, hipStream_t s, Twin tw) {
#define ZGR_CE_ROWS(THREADS, MAXE) hipLaunchKernelGGL((ce_rows_kernel<THREADS, MAXE>), dim3(M * tw.models), dim3(THREADS), 0, s, logits, targets, row_loss, n, M, tw.row_loss)
  if (n <= 1024)       ZGR_CE_ROWS(256, 4);
  else if (n <= 4096)  ZGR_CE_ROWS(256, 16);
  else if (n <= 8192)  ZGR_CE_ROWS(512, 16);
  else if (n <= 16384) ZGR_CE_ROWS(512, 32);
  else if (n <= 32768) ZGR_CE_ROWS(512, 64);
  else                 ZGR_CE_ROWS(1024, 50);
#undef ZGR_CE_ROWS
  return hipGetLastError();
}

hipError_t launch_mean_f64(const float* row_loss, int n, double inv_count, double* out, hipStream_t s, Twin tw) {
  hipLaunchKernelGGL(mean_f64_kernel, dim3(tw.models), dim3(256), 0, s, row_loss, n, inv_count, out, tw.row_loss);
  return hipGetLastError();
}

hipError_t launch_cls_head(int dtype, const void* h, const void* Wc, const void* bc, float* logits, int batch, int seq, int d, int n_class, hipStream_t s, Twin tw) {
  if (dtype == 0) hipLaunchKernelGGL(cls_head_kernel<float>, dim3(batch * tw.models * n_class), dim3(64), 0, s, (const float*)h, (const float*)Wc, (const float*)bc, logits, seq, d, n_class, batch, tw.w);
  else            hipLaunchKernelGGL(cls_head_kernel<bf16_t>, dim3(batch * tw.models * n_class), dim3(64), 0, s, (const bf16_t*)h, (const bf16_t*)Wc, (const bf16_t*)bc, logits, seq, d, n_class, batch, tw.w);
  return hipGetLastError();
}

// One block a model up to 16 entries a thread, or 64 a lane where there are fewer rows than waves (without the product in front: 1 x 4096 4.1 us against 5.9 in two launches,
// 16 x 1024 4.0 against 5.9, 64 x 256 4.3 against 5.9; 8 x 4096, 32 x 1024 and 64 x 512 6.5 against 5.9; 1 x 8192 6.2 either way, 1 x 16384 10.7 against 9.4).
bool lsq_in_one_block(int batch, int n_out) { return batch <= 64 && n_out <= 4096 && (int64_t)batch * n_out <= 16384; }
hipError_t launch_lsq_loss(const float* pred, const float* Y, float* row_loss, int batch, int n_out, double* out, hipStream_t s, Twin tw) {
  if (lsq_in_one_block(batch, n_out)) {
    hipLaunchKernelGGL(lsq_loss_kernel<1024>, dim3(tw.models), dim3(1024), 0, s, pred, Y, row_loss, n_out, batch, 1.0 / batch, out, tw.row_loss);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(lsq_rows_kernel, dim3(batch * tw.models), dim3(256), 0, s, pred, Y, row_loss, n_out, batch, tw.row_loss);
  return launch_mean_f64(row_loss, batch, 1.0 / batch, out, s, tw);
}

}  // namespace zgr
