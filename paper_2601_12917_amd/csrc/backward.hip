// Backward pass of the cloud block of Algorithm 1 (back-propagation on the public dataset with the current weights,
// whose gradients build the basis; Sec. 3.2, paragraph on guided perturbation sampling on the cloud): dL/dtheta of the loss of forward.hip, by the chain rule
// layer by layer, in fp32.  The forward pass that precedes it runs the client's kernels (fp32 products and attention in their undivided
// forms, forward.h) and keeps every layer's intermediate results; these kernels take them back in reverse order.
//
// This runs on the cloud once per stored gradient snapshot, not on the client's step.  The products run on the matrix cores (forward.hip
// for bf16 operands, product.hip for the others); LayerNorm and attention's softmax take a wave per row (LayerNorm rows of more than 2048
// entries a workgroup), cross-entropy a workgroup.  Deterministic: no atomics, every sum has a fixed order.
#include "backward.h"
#include "planes.h"
#include "wave.h"
#include "product.h"
#include <algorithm>

namespace zgr {

namespace {

struct bf16_t { uint16_t bits; };
__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(bf16_t x) { return __uint_as_float((uint32_t)x.bits << 16); }
__device__ __forceinline__ void from_f32(float x, float& o) { o = x; }
__device__ __forceinline__ void from_f32(float x, bf16_t& o) {
  const __bf16 h = static_cast<__bf16>(x);
  o.bits = __builtin_bit_cast(uint16_t, h);
}

// block of 256 threads
__device__ __forceinline__ float block_sum(float v, float* red) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return red[0] + red[1] + red[2] + red[3];
}

// ------------------------------------------------------------------ feed-forward activation: erf-GELU or ReLU
template <bool RELU> __device__ __forceinline__ float act_of(float x) { return RELU ? fmaxf(x, 0.f) : 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }
// du = df act'(u): GELU' = Phi(u) + u phi(u), ReLU' = [u > 0] (a zero slope gives zero whatever df holds)
template <bool RELU> __device__ __forceinline__ float act_rule(float x, float df) {
  if (RELU) return x > 0.f ? df : 0.f;
  const float cdf = 0.5f * (1.0f + erff(x * 0.70710678118654752f));
  const float pdf = 0.3989422804014327f * expf(-0.5f * x * x);
  return df * (cdf + x * pdf);
}

// ------------------------------------------------------------------ operands for the matrix-core products (bf16 models)
// The bf16 GEMM of the forward pass computes A W^T with both operands contiguous along the contraction.  A backward
// product contracts over another index, so its operands are first written out in bf16 with that index innermost.  One pass over
// in [rows, cols] (row stride ld_in) writes what is asked for:
//   cols_out[c][r] = in[r][c]  (row stride ld_cols, always),  rows_out[r][c] = in[r][c]  (ROWS, row stride ld_rows),
//   part[blockIdx.y][c] = the sum of the block's rows of column c in fp32  (SUMS, the bias gradient's first stage),
// with in = act'(u) in where ACT says so (1 GELU, 2 ReLU; u laid out as in).  What lies between the data and ld_cols or ld_rows (multiples of 64)
// is written as zeros: padding of the contraction.  64 x 64 tiles through LDS, tiles_per_block of them one below the other per
// block; loads and stores of 8 and 16 bytes.  Bound by memory: a gradient of 2048 x 3072 is read once and written twice in bf16,
// 50 MB in 14 us with the activation's slope, 6 us at 2048 x 768.  (A rounding pass, a transposing pass with 2-byte stores, an activation pass and a column sum took 50 us at 2048 x 3072.)
template <typename T> struct alignas(sizeof(T) * 4) Four { T e[4]; };
template <typename TIN, int ACT, bool ROWS, bool SUMS>
__global__ void __launch_bounds__(256) operand_kernel(const TIN* __restrict__ in, const float* __restrict__ u, int rows, int cols, int64_t ld_in, bf16_t* __restrict__ cols_out,
                                                      int64_t ld_cols, bf16_t* __restrict__ rows_out, int64_t ld_rows, float* __restrict__ part, int tiles_per_block) {
  __shared__ float tile[64][65];
  const int tid = threadIdx.x, c4 = (tid & 15) * 4, rq = tid >> 4, c0 = blockIdx.x * 64;
  float sum[4] = {0.f, 0.f, 0.f, 0.f};
  for (int t = 0; t < tiles_per_block; ++t) {
    const int r0 = ((int)blockIdx.y * tiles_per_block + t) * 64;
    if (r0 >= rows && r0 >= ld_cols) break;
    __syncthreads();                                       // the previous tile has been read
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = r0 + rq + 16 * i, c = c0 + c4;
      float f[4] = {0.f, 0.f, 0.f, 0.f};
      if (r < rows) {
        const int64_t o = (int64_t)r * ld_in + c;
        if (c + 4 <= cols) {
          const Four<TIN> v = *reinterpret_cast<const Four<TIN>*>(in + o);
#pragma unroll
          for (int q = 0; q < 4; ++q) f[q] = to_f32(v.e[q]);
          if (ACT) {
            const Four<float> x = *reinterpret_cast<const Four<float>*>(u + o);
#pragma unroll
            for (int q = 0; q < 4; ++q) f[q] = act_rule<ACT == 2>(x.e[q], f[q]);
          }
        } else {
          for (int q = 0; q < 4; ++q) if (c + q < cols) f[q] = ACT ? act_rule<ACT == 2>(u[o + q], to_f32(in[o + q])) : to_f32(in[o + q]);
        }
        if (ROWS && c < ld_rows) {
          Four<bf16_t> h;
#pragma unroll
          for (int q = 0; q < 4; ++q) from_f32(f[q], h.e[q]);
          *reinterpret_cast<Four<bf16_t>*>(rows_out + (int64_t)r * ld_rows + c) = h;
        }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) { if (SUMS) sum[q] += f[q]; tile[rq + 16 * i][c4 + q] = f[q]; }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int c = (tid >> 3) + 32 * i, r = (tid & 7) * 8;
      if (c0 + c < cols && r0 + r < ld_cols) {
        struct alignas(16) Eight { bf16_t e[8]; } h;
#pragma unroll
        for (int q = 0; q < 8; ++q) from_f32(tile[r + q][c], h.e[q]);
        *reinterpret_cast<Eight*>(cols_out + (int64_t)(c0 + c) * ld_cols + r0 + r) = h;
      }
    }
  }
  if (SUMS) {                                              // sixteen row groups, added in their order
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) tile[rq][c4 + q] = sum[q];
    __syncthreads();
    if (tid < 64 && c0 + tid < cols) {
      float v = 0.f;
      for (int g = 0; g < 16; ++g) v += tile[g][tid];
      part[(size_t)blockIdx.y * cols + c0 + tid] = v;
    }
  }
}

// The operand of a weight's gradient from fp32 dy [rows, cols] (cols a multiple of 64) with any number of rows: its planes (planes.h, with a bf16 factor) as three runs of
// ld terms a row, ld = rows rounded up to a multiple of 64, zeros past the rows: cols_out[c][run ld + r], the smallest plane first.  dy <- act'(u) dy where ACT
// says so, and part[blockIdx.y][c] as above.  An infinite entry is its first plane and nothing else (Inf - Inf would make a NaN of it).
// The blocks behind those (blockIdx.x >= cols / 64) write the product's other operand, x [rows, x_cols] transposed.
// 231 tokens, 4096 columns: 8 us with the activation's slope, which a launch of its own took 5 for (x on its own: 6).
__device__ __forceinline__ void transpose_tile(const uint16_t* in, int rows, int cols, int r0, int c0, uint16_t* out, int64_t ld, uint16_t (*tile)[72]);
template <int ACT>
__global__ void __launch_bounds__(256) gradient_planes_kernel(float* __restrict__ dy, const float* __restrict__ u, int rows, int cols, bf16_t* __restrict__ cols_out, int64_t ld, float* __restrict__ part,
                                                              int tiles_per_block, const bf16_t* __restrict__ x, int x_cols, bf16_t* __restrict__ x_out) {
  __shared__ __attribute__((aligned(16))) float tile[64][65];
  const int tid = threadIdx.x, c4 = (tid & 15) * 4, rq = tid >> 4, c0 = blockIdx.x * 64;
  if ((int)blockIdx.x >= cols >> 6) {
    uint16_t (*half)[72] = reinterpret_cast<uint16_t(*)[72]>(tile);
    const int x0 = ((int)blockIdx.x - (cols >> 6)) * 64;
    for (int t = 0; t < tiles_per_block; ++t) {
      const int r0 = ((int)blockIdx.y * tiles_per_block + t) * 64;
      if (r0 >= ld) break;
      transpose_tile(reinterpret_cast<const uint16_t*>(x), rows, x_cols, r0, x0, reinterpret_cast<uint16_t*>(x_out), ld, half);
    }
    return;
  }
  double sum[4] = {0., 0., 0., 0.};
  for (int t = 0; t < tiles_per_block; ++t) {
    const int r0 = ((int)blockIdx.y * tiles_per_block + t) * 64;
    if (r0 >= ld) break;
    __syncthreads();                                       // the previous tile has been read
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = r0 + rq + 16 * i;
      Four<float> f{};
      if (r < rows) {
        const int64_t o = (int64_t)r * cols + c0 + c4;
        f = *reinterpret_cast<const Four<float>*>(dy + o);
        if (ACT) {
          const Four<float> x = *reinterpret_cast<const Four<float>*>(u + o);
#pragma unroll
          for (int q = 0; q < 4; ++q) f.e[q] = act_rule<ACT == 2>(x.e[q], f.e[q]);
          *reinterpret_cast<Four<float>*>(dy + o) = f;
        }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) { sum[q] += f.e[q]; tile[rq + 16 * i][c4 + q] = f.e[q]; }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int c = (tid >> 3) + 32 * i, r = (tid & 7) * 8;
      planes_u32x4 h[3];
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const float x0 = tile[r + 2 * w][c], x1 = tile[r + 2 * w + 1][c];
        const uint32_t u0 = __float_as_uint(x0), u1 = __float_as_uint(x1);
        PlanesOf<3> o;
        cut_rest(__builtin_fabsf(x0) == INFINITY ? 0.f : x0 - high_float(u0), __builtin_fabsf(x1) == INFINITY ? 0.f : x1 - high_float(u1), 0, o);
        h[2][w] = high_halves(u1, u0); h[1][w] = o.p[1][0]; h[0][w] = o.p[2][0];
      }
#pragma unroll
      for (int x = 0; x < 3; ++x) *reinterpret_cast<planes_u32x4*>(cols_out + (int64_t)(c0 + c) * 3 * ld + x * ld + r0 + r) = h[x];
    }
  }
  __syncthreads();                                         // sixteen row groups, added in their order
  double* all = reinterpret_cast<double*>(tile);
#pragma unroll
  for (int q = 0; q < 4; ++q) all[rq * 64 + c4 + q] = sum[q];
  __syncthreads();
  if (tid < 64) {
    double v = 0.;
    for (int g = 0; g < 16; ++g) v += all[g * 64 + tid];
    part[(size_t)blockIdx.y * cols + c0 + tid] = (float)v;
  }
}

// out[c][r] = in[r][c] for the 64 x 64 entries from (r0, c0) on, zeros past the rows; a block of 256 threads, 16-byte loads and stores.
__device__ __forceinline__ void transpose_tile(const uint16_t* in, int rows, int cols, int r0, int c0, uint16_t* out, int64_t ld, uint16_t (*tile)[72]) {
  const int tid = threadIdx.x, q = (tid & 7) * 8, row = tid >> 3;
  __syncthreads();                                         // the previous tile has been read
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int r = row + 32 * i;
    const planes_u32x4 v = *reinterpret_cast<const planes_u32x4*>(in + (int64_t)min(r0 + r, rows - 1) * cols + c0 + q);
    *reinterpret_cast<planes_u32x4*>(&tile[r][q]) = r0 + r < rows ? v : planes_u32x4{0, 0, 0, 0};
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int c = row + 32 * i;
    struct alignas(16) Eight { uint16_t e[8]; } h;
#pragma unroll
    for (int k = 0; k < 8; ++k) h.e[k] = tile[q + k][c];
    *reinterpret_cast<Eight*>(out + (int64_t)(c0 + c) * ld + r0 + q) = h;
  }
}

// The transposed operands of a whole block's products in one launch (whole 64 x 64 tiles): the weights and kept
// activations of a 125M model's block are 72 MB in and out, 8 launches of 6.3 us one by one.
__global__ void __launch_bounds__(256) transposes_kernel(TransposeJobs jobs) {
  __shared__ __attribute__((aligned(16))) uint16_t tile[64][72];
  int b = blockIdx.x, j = 0;
  for (; j + 1 < jobs.count; ++j) {
    const int n = (jobs.job[j].rows >> 6) * (jobs.job[j].cols >> 6);
    if (b < n) break;
    b -= n;
  }
  const TransposeJob job = jobs.job[j];
  const int ct = job.cols >> 6, r = b / ct;
  transpose_tile(reinterpret_cast<const uint16_t*>(job.in), job.rows, job.cols, r * 64, (b - r * ct) * 64, reinterpret_cast<uint16_t*>(job.out), job.rows, tile);
}

// Sums over rows run in two stages with a fixed shape, so that the order of the additions never depends on scheduling: up to kColParts
// chunks of rows are summed side by side, then the chunk sums are added in their order:
// blockIdx.y = job: out[c] = sum over p of part[p stride + c], c < n.  32 columns per block, eight threads to a column: each adds an
// eighth of the parts in order, then the eighths are added in order.
constexpr int kColParts = 64;
__global__ void __launch_bounds__(256) colsum_final_kernel(SumJobs jobs) {
  __shared__ double sums[8][32];
  const SumJob j = jobs.job[blockIdx.y];
  const int c = blockIdx.x * 32 + (threadIdx.x & 31), q = threadIdx.x >> 5, per = (j.parts + 7) / 8;
  if ((int)blockIdx.x * 32 >= j.n) return;                 // the whole block
  double s = 0.;                                           // as free as fp32 here
  if (c < j.n) {
    const int end = j.parts < (q + 1) * per ? j.parts : (q + 1) * per;
#pragma unroll 8
    for (int p = q * per; p < end; ++p) s += j.part[p * j.stride + c];
  }
  sums[q][threadIdx.x & 31] = s;
  __syncthreads();
  if (q == 0 && c < j.n) {
    for (int i = 1; i < 8; ++i) s += sums[i][threadIdx.x];
    j.out[c] = (float)s;
  }
}

__global__ void __launch_bounds__(256) fill_kernel(float* __restrict__ p, int64_t n, float v) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) p[i] = v;
}

// ------------------------------------------------------------------ softmax cross-entropy
// One row of logits per block: row_loss = logsumexp - logit[target] (0 where target < 0; a target past the end counts as the last entry) and
// d = (softmax - onehot(target)) inv_count, zeros for a row without a target in [0, n).  d goes in place (fp32), or in bf16 to
// d16 [rows, ld16] with zeros between n and ld16.  1024 threads hold 1024 MAXE entries in registers, so the row is read once and its exponentials
// are taken once; entries beyond those are read again.  (Separate kernels for the loss and the gradient read the row five
// times: 690 us for 2048 rows of 50272, now 176.)
template <int MAXE, bool TO16>
__global__ void __launch_bounds__(1024) ce_backward_kernel(float* __restrict__ logits, const int32_t* __restrict__ targets, int n, float inv_count, float* __restrict__ row_loss,
                                                           bf16_t* __restrict__ d16, int64_t ld16) {
  __shared__ float red[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  float* row = logits + (size_t)blockIdx.x * n;
  bf16_t* out16 = TO16 ? d16 + (size_t)blockIdx.x * ld16 : nullptr;
  const int tgt = targets[blockIdx.x];
  const bool has = tgt >= 0 && tgt < n;                    // uniform over the block
  auto put = [&](int i, float d) { if (TO16) from_f32(d, out16[i]); else row[i] = d; };
  auto across = [&](float v, bool maximum) {               // the block's 16 waves, in order
    v = maximum ? wave_max(v) : wave_sum(v);
    __syncthreads();
    if (lane == 0) red[wave] = v;
    __syncthreads();
    float r = red[0];
    for (int w = 1; w < 16; ++w) r = maximum ? fmaxf(r, red[w]) : r + red[w];
    return r;
  };
  if (TO16) for (int i = n + tid; i < ld16; i += 1024) from_f32(0.f, out16[i]);
  if (tgt < 0) {
    for (int i = tid; i < n; i += 1024) put(i, 0.f);
    if (tid == 0) row_loss[blockIdx.x] = 0.f;
    return;
  }
  const float at_target = row[has ? tgt : n - 1];          // read before anything is written
  float v[MAXE], mx = -INFINITY;
#pragma unroll
  for (int u = 0; u < MAXE; ++u) {
    const int i = tid + 1024 * u;
    v[u] = i < n ? row[i] : -INFINITY;
    mx = fmaxf(mx, v[u]);
  }
  for (int i = tid + 1024 * MAXE; i < n; i += 1024) mx = fmaxf(mx, row[i]);
  mx = across(mx, true);
  float s = 0.f;
#pragma unroll
  for (int u = 0; u < MAXE; ++u) { v[u] = tid + 1024 * u < n ? expf(v[u] - mx) : 0.f; s += v[u]; }
  for (int i = tid + 1024 * MAXE; i < n; i += 1024) s += expf(row[i] - mx);
  s = across(s, false);
  if (tid == 0) row_loss[blockIdx.x] = logf(s) + mx - at_target;
  const float inv = 1.0f / s;
#pragma unroll
  for (int u = 0; u < MAXE; ++u) {
    const int i = tid + 1024 * u;
    if (i < n) put(i, has ? (v[u] * inv - (i == tgt ? 1.0f : 0.f)) * inv_count : 0.f);
  }
  for (int i = tid + 1024 * MAXE; i < n; i += 1024) put(i, has ? (expf(row[i] - mx) * inv - (i == tgt ? 1.0f : 0.f)) * inv_count : 0.f);
}

// ------------------------------------------------------------------ LayerNorm
// y = xhat g + b, xhat = (x - mu) rstd.  Per row: dx = rstd (dy g - mean(dy g) - xhat mean(dy g xhat)), written as
// dx_out = (add ? add : 0) + dx (dx_out may be add or dy itself: every sum over the row is taken before the row is
// written, and an element is written by the thread that read it).
template <typename T>
__global__ void __launch_bounds__(256) ln_backward_kernel(const float* __restrict__ x, const T* __restrict__ g, const float* dy,
                                                          const float* add, float* dx_out, int d, float eps) {   // add or dy may be dx_out
  __shared__ float red[4];
  const size_t o = (size_t)blockIdx.x * d;
  const float* row = x + o;
  const float* drow = dy + o;
  float s = 0.f;
  for (int i = threadIdx.x; i < d; i += 256) s += row[i];
  const float mu = block_sum(s, red) / d;
  float v = 0.f;
  for (int i = threadIdx.x; i < d; i += 256) { const float t = row[i] - mu; v += t * t; }
  const float rstd = 1.0f / sqrtf(block_sum(v, red) / d + eps);
  float s1 = 0.f, s2 = 0.f;
  for (int i = threadIdx.x; i < d; i += 256) {
    const float dg = drow[i] * to_f32(g[i]);
    s1 += dg;
    s2 += dg * ((row[i] - mu) * rstd);
  }
  s1 = block_sum(s1, red) / d;
  s2 = block_sum(s2, red) / d;
  for (int i = threadIdx.x; i < d; i += 256) {
    const float xhat = (row[i] - mu) * rstd;
    const float r = rstd * (drow[i] * to_f32(g[i]) - s1 - xhat * s2);
    dx_out[o + i] = (add ? add[o + i] : 0.f) + r;
  }
}

// The same rule and the parameter gradients in one pass over x and dy, for d % 4 == 0 and d <= 256 MAXV: a wave takes rows in turn, the
// row in registers (one read of x and dy, no barrier), and keeps its rows' share of dg[c] = sum_m dy[m][c] xhat[m][c] and
// db[c] = sum_m dy[m][c] in registers too.  part[b][0 | 1][c]: the block's sums, its four waves added in order.  Bound by launch and
// load latency at a few thousand rows: with a kernel each for the row statistics, the partial sums and the two final sums the rule
// took five launches and three reads (27 us per LayerNorm of 2048 x 768, now 13).
// dy comes as dy_parts parts, dy_stride floats apart, which are added in their order: those of a product whose sums are split over blocks, whose adding up was a launch
// of 4.4 us (four parts of 231 x 1024 7.9 us here, one 7.7; loaded one after the other 11).
template <typename T, int MAXV, bool PARTS>
__global__ void __launch_bounds__(256) ln_backward_wave_kernel(const float* __restrict__ x, const T* __restrict__ g, const float* dy, int dy_parts, int64_t dy_stride, const float* add, float* dx_out,
                                                               float* __restrict__ part, int M, int d, float eps) {            // add or dy may be dx_out
  __shared__ __attribute__((aligned(16))) float red[4][256 * MAXV];
  struct alignas(sizeof(T) * 4) V4 { T e[4]; };
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nv = d >> 2;
  float4 gain[MAXV], sg[MAXV], sb[MAXV];
#pragma unroll
  for (int j = 0; j < MAXV; ++j) {
    const int i = lane + 64 * j;
    sg[j] = sb[j] = gain[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (i < nv) { const V4 t = *reinterpret_cast<const V4*>(g + 4 * i); gain[j] = make_float4(to_f32(t.e[0]), to_f32(t.e[1]), to_f32(t.e[2]), to_f32(t.e[3])); }
  }
  for (int row = blockIdx.x * 4 + wave; row < M; row += gridDim.x * 4) {
    const float4* xr = reinterpret_cast<const float4*>(x + (size_t)row * d);
    const float4* dr = reinterpret_cast<const float4*>(dy + (size_t)row * d);
    float4 v[MAXV], w[MAXV];
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < MAXV; ++j) {
      const int i = lane + 64 * j;
      v[j] = w[j] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (i < nv) { v[j] = xr[i]; w[j] = dr[i]; }
    }
    constexpr int AHEAD = MAXV > 4 ? 1 : 3;                  // parts under way at a time (past the last one the first is read and left)
    for (int p = 1; PARTS && p < dy_parts; p += AHEAD) {
      float4 t[AHEAD][MAXV];
#pragma unroll
      for (int u = 0; u < AHEAD; ++u)
#pragma unroll
        for (int j = 0; j < MAXV; ++j) t[u][j] = reinterpret_cast<const float4*>(dy + (size_t)row * d + (p + u < dy_parts ? p + u : 0) * dy_stride)[min(lane + 64 * j, nv - 1)];
#pragma unroll
      for (int u = 0; u < AHEAD; ++u)
        if (p + u < dy_parts)
#pragma unroll
          for (int j = 0; j < MAXV; ++j)
            if (lane + 64 * j < nv) { w[j].x += t[u][j].x; w[j].y += t[u][j].y; w[j].z += t[u][j].z; w[j].w += t[u][j].w; }
    }
#pragma unroll
    for (int j = 0; j < MAXV; ++j) s += (v[j].x + v[j].y) + (v[j].z + v[j].w);
    const float mu = wave_sum(s) / d;
    float q = 0.f;
#pragma unroll
    for (int j = 0; j < MAXV; ++j)
      if (lane + 64 * j < nv) {
        v[j].x -= mu; v[j].y -= mu; v[j].z -= mu; v[j].w -= mu;
        q += (v[j].x * v[j].x + v[j].y * v[j].y) + (v[j].z * v[j].z + v[j].w * v[j].w);
      }
    const float rstd = 1.0f / sqrtf(wave_sum(q) / d + eps);
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int j = 0; j < MAXV; ++j) {
      v[j].x *= rstd; v[j].y *= rstd; v[j].z *= rstd; v[j].w *= rstd;                  // xhat; zeros past the row's end
      sg[j].x += w[j].x * v[j].x; sg[j].y += w[j].y * v[j].y; sg[j].z += w[j].z * v[j].z; sg[j].w += w[j].w * v[j].w;
      sb[j].x += w[j].x; sb[j].y += w[j].y; sb[j].z += w[j].z; sb[j].w += w[j].w;
      w[j].x *= gain[j].x; w[j].y *= gain[j].y; w[j].z *= gain[j].z; w[j].w *= gain[j].w;
      s1 += (w[j].x + w[j].y) + (w[j].z + w[j].w);
      s2 += (w[j].x * v[j].x + w[j].y * v[j].y) + (w[j].z * v[j].z + w[j].w * v[j].w);
    }
    s1 = wave_sum(s1) / d;
    s2 = wave_sum(s2) / d;
    const float4* ar = add ? reinterpret_cast<const float4*>(add + (size_t)row * d) : nullptr;
    float4* out = reinterpret_cast<float4*>(dx_out + (size_t)row * d);
#pragma unroll
    for (int j = 0; j < MAXV; ++j) {
      const int i = lane + 64 * j;
      if (i < nv) {
        float4 r = make_float4(rstd * (w[j].x - s1 - v[j].x * s2), rstd * (w[j].y - s1 - v[j].y * s2), rstd * (w[j].z - s1 - v[j].z * s2), rstd * (w[j].w - s1 - v[j].w * s2));
        if (ar) { const float4 t = ar[i]; r.x += t.x; r.y += t.y; r.z += t.z; r.w += t.w; }
        out[i] = r;
      }
    }
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    __syncthreads();
#pragma unroll
    for (int j = 0; j < MAXV; ++j) *reinterpret_cast<float4*>(&red[wave][4 * (lane + 64 * j)]) = h ? sb[j] : sg[j];
    __syncthreads();
    for (int c = threadIdx.x; c < d; c += 256) part[((size_t)blockIdx.x * 2 + h) * d + c] = (red[0][c] + red[1][c]) + (red[2][c] + red[3][c]);
  }
}

// (mu, rstd) of every row, for the parameter gradients
__global__ void __launch_bounds__(256) ln_stats_kernel(const float* __restrict__ x, float* __restrict__ stats, int d, float eps) {
  __shared__ float red[4];
  const float* row = x + (size_t)blockIdx.x * d;
  float s = 0.f;
  for (int i = threadIdx.x; i < d; i += 256) s += row[i];
  const float mu = block_sum(s, red) / d;
  float v = 0.f;
  for (int i = threadIdx.x; i < d; i += 256) { const float t = row[i] - mu; v += t * t; }
  const float rstd = 1.0f / sqrtf(block_sum(v, red) / d + eps);
  if (threadIdx.x == 0) { stats[2 * blockIdx.x] = mu; stats[2 * blockIdx.x + 1] = rstd; }
}

// dg[c] = sum_m dy[m][c] xhat[m][c], db[c] = sum_m dy[m][c]: chunk sums as above (part: [kColParts][2][d]), then
// colsum_final_kernel on each half
__global__ void __launch_bounds__(256) ln_param_grad_partial_kernel(const float* __restrict__ x, const float* __restrict__ dy, const float* __restrict__ stats,
                                                                    int M, int d, float* __restrict__ part) {
  __shared__ float pg[4][64], pb[4][64];
  const int c = blockIdx.x * 64 + (threadIdx.x & 63), grp = threadIdx.x >> 6;
  const int chunk = (M + kColParts - 1) / kColParts;
  const int m_begin = blockIdx.y * chunk, m_end = min(M, m_begin + chunk);
  float sg = 0.f, sb = 0.f;
  if (c < d)
    for (int m = m_begin + grp; m < m_end; m += 4) {
      const float dyv = dy[(size_t)m * d + c];
      sg += dyv * ((x[(size_t)m * d + c] - stats[2 * m]) * stats[2 * m + 1]);
      sb += dyv;
    }
  pg[grp][threadIdx.x & 63] = sg; pb[grp][threadIdx.x & 63] = sb;
  __syncthreads();
  if (grp == 0 && c < d) {
    part[(size_t)2 * blockIdx.y * d + c] = (pg[0][threadIdx.x] + pg[1][threadIdx.x]) + (pg[2][threadIdx.x] + pg[3][threadIdx.x]);
    part[(size_t)(2 * blockIdx.y + 1) * d + c] = (pb[0][threadIdx.x] + pb[1][threadIdx.x]) + (pb[2][threadIdx.x] + pb[3][threadIdx.x]);
  }
}

// Four entries per thread (n4 of them), the last n % 4 by the first threads of the grid.
template <typename T, bool RELU>
__global__ void __launch_bounds__(256) act_forward_kernel(const float* __restrict__ u, T* __restrict__ f, int64_t n) {
  struct alignas(sizeof(T) * 4) V4 { T e[4]; };
  const int64_t first = (int64_t)blockIdx.x * 256 + threadIdx.x, n4 = n >> 2;
  for (int64_t i = first; i < n4; i += (int64_t)gridDim.x * 256) {
    const float4 x = reinterpret_cast<const float4*>(u)[i];
    V4 r;
    from_f32(act_of<RELU>(x.x), r.e[0]); from_f32(act_of<RELU>(x.y), r.e[1]); from_f32(act_of<RELU>(x.z), r.e[2]); from_f32(act_of<RELU>(x.w), r.e[3]);
    reinterpret_cast<V4*>(f)[i] = r;
  }
  if (first < (n & 3)) from_f32(act_of<RELU>(u[4 * n4 + first]), f[4 * n4 + first]);
}
// df <- df act'(u)
template <bool RELU>
__global__ void __launch_bounds__(256) act_backward_kernel(const float* __restrict__ u, float* __restrict__ df, int64_t n) {
  const int64_t first = (int64_t)blockIdx.x * 256 + threadIdx.x, n4 = n >> 2;
  for (int64_t i = first; i < n4; i += (int64_t)gridDim.x * 256) {
    const float4 x = reinterpret_cast<const float4*>(u)[i];
    float4 r = reinterpret_cast<float4*>(df)[i];
    r = make_float4(act_rule<RELU>(x.x, r.x), act_rule<RELU>(x.y, r.y), act_rule<RELU>(x.z, r.z), act_rule<RELU>(x.w, r.w));
    reinterpret_cast<float4*>(df)[i] = r;
  }
  if (first < (n & 3)) df[4 * n4 + first] = act_rule<RELU>(u[4 * n4 + first], df[4 * n4 + first]);
}

__global__ void __launch_bounds__(256) add_kernel(float* __restrict__ dst, const float* __restrict__ src, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) dst[i] += src[i];
}

// ------------------------------------------------------------------ attention
// qkv [B T, 3 d]: query, key, value of head h at columns h dh, d + h dh, 2 d + h dh.  Key j takes part in query i's
// softmax when j < length (the sequence's length, or T) and, under the causal mask, j <= i.
// Five batched products per head and one row-wise rule between them:
//   S = Q K^T / sqrt dh and dP = dctx V^T             (into the P and dS buffers)
//   p = softmax(S) over the visible keys, ds = p (dP - p . dP), zeros at masked keys        (attn_backward_rows_kernel, in place)
//   dQ = dS K / sqrt dh,   dK = dS^T Q / sqrt dh,   dV = P^T dctx
// One wave per row (b, h, i) of the two [T, T] buffers, four rows per block; a lane holds up to MAXJ of the row's entries (T <= 64 MAXJ),
// so the three reductions stay inside the wave.  (One block of 256 threads per row: 40 us for 24576 rows of 128, most of the
// threads without an entry and six barriers per row.)
template <int MAXJ>
__global__ void __launch_bounds__(256) attn_backward_rows_kernel(const int32_t* __restrict__ lengths, int64_t rows, int seq, int n_head, int causal,
                                                                 float* __restrict__ P, float* __restrict__ dS) {
  const int lane = threadIdx.x & 63;
  const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= rows) return;                                             // whole waves leave: no barrier below
  const int i = (int)(r % seq), b = (int)(r / ((int64_t)seq * n_head));
  int kend = lengths ? lengths[b] : seq;
  kend = kend < seq ? kend : seq;
  if (causal) kend = kend < i + 1 ? kend : i + 1;
  float* prow = P + (size_t)r * seq;
  float* srow = dS + (size_t)r * seq;
  float sc[MAXJ], dp[MAXJ];
  float mx = -INFINITY;
#pragma unroll
  for (int u = 0; u < MAXJ; ++u) {
    const int j = lane + 64 * u;
    sc[u] = -INFINITY; dp[u] = 0.f;
    if (j < kend) { sc[u] = prow[j]; dp[u] = srow[j]; mx = fmaxf(mx, sc[u]); }
  }
  mx = wave_max(mx);
  float den = 0.f;
#pragma unroll
  for (int u = 0; u < MAXJ; ++u) { sc[u] = (lane + 64 * u < kend) ? expf(sc[u] - mx) : 0.f; den += sc[u]; }
  den = wave_sum(den);
  const float inv = den > 0.f ? 1.0f / den : 0.f;
  float dot = 0.f;
#pragma unroll
  for (int u = 0; u < MAXJ; ++u) { sc[u] *= inv; dot += sc[u] * dp[u]; }
  dot = wave_sum(dot);
#pragma unroll
  for (int u = 0; u < MAXJ; ++u) {
    const int j = lane + 64 * u;
    if (j < seq) { prow[j] = sc[u]; srow[j] = sc[u] * (dp[u] - dot); }
  }
}

// The same rule for heads of 16, 32 and 64 without the [T, T] buffers, where there are enough rows (bw_attention_buffers), in two kernels of one wave per 32 rows.  The first has 32 queries in its lanes and
// walks the keys in blocks of 32 twice: S^T = K Q^T and dP^T = V dctx^T give the maximum, the sum of exponentials and p . dP of each query (stats), then
// again dS and with it dQ^T += K^T dS^T.  The second has 32 keys in its lanes and walks the queries that see them: S, dP, P and dS from the stats,
// dK^T += Q^T dS, dV^T += dctx^T P.  A lane holds 16 rows of one column of these 32 x 32 pieces, which are the next product's operand as they
// are: its terms are taken in the order 8 (v / 4) + 4 half + v % 4, in which the other operand's rows are loaded.  Probabilities and dS stay in fp32: bf16
// models take the products with dS and dctx on the bf16 instruction in three planes (planes.h), those of two fp32 operands are fp32 instructions.
// Bound by load latency on short sequences, by the vector unit (exponentials, planes) on long ones.  Five batched products and the row rule with their
// [T, T] buffers took 67 us for 192 heads of 64 at 128 tokens and 46 for 48 at 77.
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
constexpr float kLog2e = 1.44269504088896341f;

// A lane's part of the 32 rows of an operand contracted over the head: row l32 (lane % 32).  fp32: entries half DH / 2 .. of it; bf16: eight
// entries from 16 s + 8 half on for every instruction s.
template <typename T, int DH> struct HeadRow;
template <int DH> struct HeadRow<float, DH> {
  float v[DH / 2];
  __device__ __forceinline__ void load(const float* row, int half) {
#pragma unroll
    for (int i = 0; i < DH / 2; i += 4) {
      const float4 t = *reinterpret_cast<const float4*>(row + half * (DH / 2) + i);
      v[i] = t.x; v[i + 1] = t.y; v[i + 2] = t.z; v[i + 3] = t.w;
    }
  }
};
template <int DH> struct HeadRow<bf16_t, DH> {
  bf16x8 v[DH / 16];
  __device__ __forceinline__ void load(const bf16_t* row, int half) {
#pragma unroll
    for (int s = 0; s < DH / 16; ++s) v[s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(row + 16 * s + 8 * half));
  }
};
// The fp32 rows that meet rows of storage type T: as they are, or cut into planes (ready()) once they have arrived.
template <typename T, int DH> struct GradRow : HeadRow<float, DH> { __device__ __forceinline__ void ready() {} };
template <int DH> struct GradRow<bf16_t, DH> {
  float4 raw[DH / 16][2];
  PlanesOf<3> v[DH / 16];
  __device__ __forceinline__ void load(const float* row, int half) {
#pragma unroll
    for (int s = 0; s < DH / 16; ++s)
#pragma unroll
      for (int q = 0; q < 2; ++q) raw[s][q] = *reinterpret_cast<const float4*>(row + 16 * s + 8 * half + 4 * q);
  }
  __device__ __forceinline__ void ready() {
#pragma unroll
    for (int s = 0; s < DH / 16; ++s)
#pragma unroll
      for (int q = 0; q < 2; ++q) { cut_pair(raw[s][q].x, raw[s][q].y, 2 * q, v[s]); cut_pair(raw[s][q].z, raw[s][q].w, 2 * q + 1, v[s]); }
  }
};
__device__ __forceinline__ f32x16 zeros16() {
  f32x16 z;
#pragma unroll
  for (int v = 0; v < 16; ++v) z[v] = 0.f;
  return z;
}
template <int DH> __device__ __forceinline__ f32x16 rows_product(const HeadRow<float, DH>& a, const HeadRow<float, DH>& b) {
  f32x16 s = zeros16();
#pragma unroll
  for (int i = 0; i < DH / 2; ++i) s = __builtin_amdgcn_mfma_f32_32x32x2f32(a.v[i], b.v[i], s, 0, 0, 0);
  return s;
}
template <int DH> __device__ __forceinline__ f32x16 rows_product(const HeadRow<bf16_t, DH>& a, const HeadRow<bf16_t, DH>& b) {
  f32x16 s = zeros16();
#pragma unroll
  for (int i = 0; i < DH / 16; ++i) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.v[i], b.v[i], s, 0, 0, 0);
  return s;
}
template <int DH> __device__ __forceinline__ f32x16 rows_product(const HeadRow<bf16_t, DH>& a, const GradRow<bf16_t, DH>& b) {
  f32x16 s = zeros16();
#pragma unroll
  for (int x = 2; x >= 0; --x)
#pragma unroll
    for (int i = 0; i < DH / 16; ++i) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.v[i], __builtin_bit_cast(bf16x8, b.v[i].p[x]), s, 0, 0, 0);
  return s;
}
template <int DH> __device__ __forceinline__ f32x16 rows_product(const GradRow<bf16_t, DH>& a, const HeadRow<bf16_t, DH>& b) {
  f32x16 s = zeros16();
#pragma unroll
  for (int x = 2; x >= 0; --x)
#pragma unroll
    for (int i = 0; i < DH / 16; ++i) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a.v[i].p[x]), b.v[i], s, 0, 0, 0);
  return s;
}
// Entry 32 f + l32 of the 16 rows that meet a lane's 16 values: rows(v) is where row 8 (v / 4) + 4 half + v % 4 of the operand starts.  Requested ahead
// of what they are multiplied with.
template <typename T, int DH> struct Columns {
  static constexpr int F = DH > 32 ? DH / 32 : 1;
  T c[16][F];
  template <typename R> __device__ __forceinline__ void load(R rows, int l32) {
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const T* r = rows(v);
#pragma unroll
      for (int f = 0; f < F; ++f) { c[v][f] = T{}; if (DH >= 32 || l32 < DH) c[v][f] = r[32 * f + l32]; }
    }
  }
};
// o[f][t][column] += sum over v of c[v][f] (of lane t) x[v].  fp32 sums the 32 rows by themselves first: a long sequence's sum then rounds at its full size once a
// block, not 16 times (gradients of an fp32 model on 1100 tokens 1.96e-6 off fp64, now 1.93e-6, the key bias's 1.8e-8 off zero, now 0.7e-8, at no cost).  bf16 models'
// gradients are 9e-3 off fp64 either way, and lose 1 to 3 % of time to it.
template <int DH> __device__ __forceinline__ void add_columns(f32x16* o, const Columns<float, DH>& a, const f32x16& x) {
  constexpr int F = Columns<float, DH>::F;
  f32x16 sum[F];
#pragma unroll
  for (int f = 0; f < F; ++f) sum[f] = zeros16();
#pragma unroll
  for (int v = 0; v < 16; ++v)
#pragma unroll
    for (int f = 0; f < F; ++f) sum[f] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.c[v][f], x[v], sum[f], 0, 0, 0);
#pragma unroll
  for (int f = 0; f < F; ++f) o[f] += sum[f];
}
template <int DH> __device__ __forceinline__ void add_columns(f32x16* o, const Columns<bf16_t, DH>& a, const f32x16& x) {
  constexpr int F = Columns<bf16_t, DH>::F;
  PlanesOf<3> p[2];
#pragma unroll
  for (int v = 0; v < 16; v += 2) cut_pair(x[v], x[v + 1], (v & 7) >> 1, p[v >> 3]);
#pragma unroll
  for (int st = 0; st < 2; ++st)
#pragma unroll
    for (int f = 0; f < F; ++f) {
      planes_u32x4 w;
#pragma unroll
      for (int i = 0; i < 4; ++i) w[i] = (uint32_t)a.c[8 * st + 2 * i][f].bits | ((uint32_t)a.c[8 * st + 2 * i + 1][f].bits << 16);
#pragma unroll
      for (int y = 2; y >= 0; --y) o[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, p[st].p[y]), o[f], 0, 0, 0);
    }
}
// the rows of a transposed result: lane (l32, half) holds four consecutive entries of row l32 at a time
template <int DH> __device__ __forceinline__ void store_head_row(float* row, const f32x16* o, int half, float scale) {
  constexpr int F = DH > 32 ? DH / 32 : 1;
#pragma unroll
  for (int f = 0; f < F; ++f)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int t = 32 * f + 8 * q + 4 * half;
      if (t < DH) *reinterpret_cast<float4*>(row + t) = make_float4(o[f][4 * q] * scale, o[f][4 * q + 1] * scale, o[f][4 * q + 2] * scale, o[f][4 * q + 3] * scale);
    }
}

// exp(scale s) over 2 to the maximum.  Both kernels take it this way: a query's dS then sum to zero but for rounding (rounded apart in one of them, the key bias's
// gradient, which is nothing but that, was twice as far from zero).
__device__ __forceinline__ float softmax_term(float s, float scale_log2, float max_log2) { return __builtin_amdgcn_exp2f(__builtin_fmaf(s, scale_log2, -max_log2)); }

// stats: [3][heads][T rounded up to 32], the maximum of the scaled scores in log2 units, 1 / (sum of exponentials) and p . dP.  The last query blocks come first:
// under the causal mask they have the most keys.  The next block's rows are requested before this one's are used.
template <typename T, int DH>
__global__ void __launch_bounds__(64, 1) attn_backward_q_kernel(const T* __restrict__ qkv, const float* __restrict__ dctx, const int32_t* __restrict__ lengths, int seq, int d, int n_head, int causal,
                                                                int heads, float* __restrict__ stats, float* __restrict__ dqkv) {
  constexpr int F = DH > 32 ? DH / 32 : 1;
  const int lane = threadIdx.x, l32 = lane & 31, half = lane >> 5;
  const int blocks = (seq + 31) / 32, bh = (int)blockIdx.x % heads, q0 = 32 * (blocks - 1 - (int)blockIdx.x / heads), qi = q0 + l32, qr = qi < seq ? qi : seq - 1;
  const int h = bh % n_head, b = bh / n_head;
  const int64_t ld = (int64_t)3 * d;
  const T* base = qkv + (int64_t)b * seq * ld + (int64_t)h * DH;
  const float scale = 1.0f / sqrtf((float)DH), scale_log2 = kLog2e * scale;
  int kend = lengths ? lengths[b] : seq;
  kend = kend < seq ? kend : seq;
  const int last = causal && q0 + 32 < kend ? q0 + 32 : kend;        // keys of this wave
  HeadRow<T, DH> q, k, vv;
  GradRow<T, DH> g;
  q.load(base + qr * ld, half);
  g.load(dctx + ((int64_t)b * seq + qr) * d + (int64_t)h * DH, half);
  auto sees = [&](int key) { return key < last && (!causal || key <= qi); };
  auto key_of = [&](int k0, int v) { return k0 + 8 * (v >> 2) + 4 * half + (v & 3); };
  auto request = [&](int k0) {                                       // a key past the end repeats the last one
    const T* row = base + (int64_t)(k0 + l32 < last ? k0 + l32 : last - 1) * ld + d;
    k.load(row, half);
    vv.load(row + d, half);
  };
  f32x16 s, dp;
  auto scores = [&](int k0, int next) {                              // -inf where the query doesn't see the key, and dP
    s = rows_product(k, q);
    dp = rows_product(vv, g);
    request(next);
#pragma unroll
    for (int v = 0; v < 16; ++v) s[v] = sees(key_of(k0, v)) ? s[v] : -INFINITY;
  };
  float mx = -INFINITY, den = 0.f, dot = 0.f;
  if (last > 0) request(0);
  g.ready();
  for (int k0 = 0; k0 < last; k0 += 32) {
    scores(k0, k0 + 32 < last ? k0 + 32 : 0);                        // behind the last block, the first one for the second walk
    float m = s[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) m = fmaxf(m, s[v]);
    m = fmaxf(mx, fmaxf(m, __shfl_xor(m, 32, 64)) * scale_log2);
    const float safe = m == -INFINITY ? 0.f : m, corr = __builtin_amdgcn_exp2f(mx - safe);
    float pd[4] = {0.f, 0.f, 0.f, 0.f}, pt[4] = {0.f, 0.f, 0.f, 0.f};      // the block's share apart: a long sequence's chain rounds once a block, not once a key
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const float p = softmax_term(s[v], scale_log2, safe);
      pd[v & 3] += p;
      pt[v & 3] += sees(key_of(k0, v)) ? p * dp[v] : 0.f;
    }
    den = __builtin_fmaf(den, corr, (pd[0] + pd[1]) + (pd[2] + pd[3]));
    dot = __builtin_fmaf(dot, corr, (pt[0] + pt[1]) + (pt[2] + pt[3]));
    mx = m;
  }
  den += __shfl_xor(den, 32, 64);
  dot += __shfl_xor(dot, 32, 64);
  const float inv = den > 0.f ? 1.0f / den : 0.f, safe = mx == -INFINITY ? 0.f : mx;
  dot *= inv;
  if (qi < seq && half == 0) {
    const int64_t i = (int64_t)bh * (32 * blocks) + qi, n = (int64_t)heads * (32 * blocks);
    stats[i] = safe; stats[n + i] = inv; stats[2 * n + i] = dot;
  }
  f32x16 o[F];
#pragma unroll
  for (int f = 0; f < F; ++f) o[f] = zeros16();
  for (int k0 = 0; k0 < last; k0 += 32) {
    Columns<T, DH> kc;
    kc.load([&](int v) { const int key = key_of(k0, v); return base + (int64_t)(key < last ? key : last - 1) * ld + d; }, l32);
    scores(k0, k0 + 32 < last ? k0 + 32 : k0);
#pragma unroll
    for (int v = 0; v < 16; ++v) s[v] = sees(key_of(k0, v)) ? softmax_term(s[v], scale_log2, safe) * inv * (dp[v] - dot) : 0.f;
    add_columns<DH>(o, kc, s);
  }
  if (qi < seq) store_head_row<DH>(dqkv + ((int64_t)b * seq + qi) * ld + (int64_t)h * DH, o, half, scale);
}

template <typename T, int DH>
__global__ void __launch_bounds__(64, 1) attn_backward_kv_kernel(const T* __restrict__ qkv, const float* __restrict__ dctx, const int32_t* __restrict__ lengths, int seq, int d, int n_head, int causal,
                                                                 int heads, const float* __restrict__ stats, float* __restrict__ dqkv) {
  constexpr int F = DH > 32 ? DH / 32 : 1;
  const int lane = threadIdx.x, l32 = lane & 31, half = lane >> 5;
  const int blocks = (seq + 31) / 32, bh = (int)blockIdx.x % heads, k0 = 32 * ((int)blockIdx.x / heads), kj = k0 + l32, kr = kj < seq ? kj : seq - 1;
  const int h = bh % n_head, b = bh / n_head;
  const int64_t ld = (int64_t)3 * d;
  const T* base = qkv + (int64_t)b * seq * ld + (int64_t)h * DH;
  const float* dbase = dctx + (int64_t)b * seq * d + (int64_t)h * DH;
  const float scale = 1.0f / sqrtf((float)DH), scale_log2 = kLog2e * scale;
  const float* mx = stats + (int64_t)bh * (32 * blocks);
  const float* inv = mx + (int64_t)heads * (32 * blocks);
  const float* dot = inv + (int64_t)heads * (32 * blocks);
  int kend = lengths ? lengths[b] : seq;
  kend = kend < seq ? kend : seq;
  HeadRow<T, DH> k, vv, q;
  GradRow<T, DH> g;
  auto request = [&](int q0) {
    const int qr = q0 + l32 < seq ? q0 + l32 : seq - 1;
    q.load(base + qr * ld, half);
    g.load(dbase + (int64_t)qr * d, half);
  };
  const int first = k0 >= kend ? seq : (causal ? k0 : 0);            // no query sees keys past the end
  if (first < seq) request(first);
  k.load(base + kr * ld + d, half);
  vv.load(base + kr * ld + 2 * d, half);
  f32x16 dk[F], dv[F];
#pragma unroll
  for (int f = 0; f < F; ++f) dk[f] = dv[f] = zeros16();
  for (int q0 = first; q0 < seq; q0 += 32) {
    auto query = [&](int v) { const int i = q0 + 8 * (v >> 2) + 4 * half + (v & 3); return i < seq ? i : seq - 1; };      // one past the end repeats the last: its P and dS are zero
    Columns<float, DH> dc;
    Columns<T, DH> qc;
    float4 stat[3][4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = q0 + 8 * u + 4 * half;
      stat[0][u] = *reinterpret_cast<const float4*>(mx + i); stat[1][u] = *reinterpret_cast<const float4*>(inv + i); stat[2][u] = *reinterpret_cast<const float4*>(dot + i);
    }
    dc.load([&](int v) { return dbase + (int64_t)query(v) * d; }, l32);
    qc.load([&](int v) { return base + (int64_t)query(v) * ld; }, l32);
    g.ready();
    f32x16 p = rows_product(q, k), ds = rows_product(g, vv);
    request(q0 + 32 < seq ? q0 + 32 : q0);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int i = q0 + 8 * (v >> 2) + 4 * half + (v & 3);
      const bool seen = i < seq && kj < kend && (!causal || kj <= i);
      const float m = reinterpret_cast<const float*>(&stat[0][v >> 2])[v & 3], w = reinterpret_cast<const float*>(&stat[1][v >> 2])[v & 3], t = reinterpret_cast<const float*>(&stat[2][v >> 2])[v & 3];
      const float e = seen ? softmax_term(p[v], scale_log2, m) * w : 0.f;
      p[v] = e;
      ds[v] = seen ? e * (ds[v] - t) : 0.f;
    }
    add_columns<DH>(dv, dc, p);
    add_columns<DH>(dk, qc, ds);
  }
  if (kj < seq) {
    float* row = dqkv + ((int64_t)b * seq + kj) * ld + (int64_t)h * DH;
    store_head_row<DH>(row + d, dk, half, scale);
    store_head_row<DH>(row + 2 * d, dv, half, 1.0f);
  }
}

// ------------------------------------------------------------------ embeddings
// x0[m] = E[tok[m]] + Pe[m mod seq].  dE accumulates (the tied head has written it), dPe is overwritten; the rows that share a token or a
// position are added in the order of the rows, so the result is reproducible.
// Block m < M: if m is the first row with its token, adds every row with that token to the token's row of dE, in order (the tokens are
// listed 1024 at a time, then their rows requested sixteen at a time; a thread holds two columns).  Block M + p: row p of dPe.
// What bounds it is the most frequent token's chain, a ninth of the rows of a Zipf text: 2048 tokens of 768 columns 35 us, 84 with the rows
// requested eight at a time out of the 64 matches of one wave.
// (One thread per column walking all the rows took 0.8 ms for 2048 rows of 768: three workgroups and a chain of 2048 additions to memory.)
constexpr int kEmbedCols = 2, kEmbedAhead = 16;
__global__ void __launch_bounds__(256) embed_backward_kernel(const int32_t* __restrict__ tok, const float* __restrict__ dx, int M, int seq, int d, int vocab,
                                                             float* __restrict__ dE, float* __restrict__ dPe) {
  __shared__ int list[1024], counts[16];
  const int tid = threadIdx.x, c0 = blockIdx.y * 256 * kEmbedCols + tid;
  auto token = [&](int m) { const int t = tok[m]; return t < 0 ? 0 : (t >= vocab ? vocab - 1 : t); };
  float acc[kEmbedCols];
  float* row;
  if ((int)blockIdx.x >= M) {
    const int p = (int)blockIdx.x - M;
    row = dPe + (size_t)p * d;
#pragma unroll
    for (int u = 0; u < kEmbedCols; ++u) acc[u] = 0.f;
    if (p < seq)
#pragma unroll 8
      for (int m = p; m < M; m += seq)
#pragma unroll
        for (int u = 0; u < kEmbedCols; ++u) if (c0 + 256 * u < d) acc[u] += dx[(size_t)m * d + c0 + 256 * u];
  } else {
    const int m = blockIdx.x, t = token(m);
    for (int b = 0; b < m; b += 1024) {
      bool seen = false;
#pragma unroll
      for (int u = 0; u < 4; ++u) { const int q = b + 256 * u + tid; seen |= q < m && token(q) == t; }
      if (__syncthreads_or(seen)) return;                            // the whole block leaves
    }
    row = dE + (size_t)t * d;
#pragma unroll
    for (int u = 0; u < kEmbedCols; ++u) acc[u] = c0 + 256 * u < d ? row[c0 + 256 * u] : 0.f;
    for (int b = m; b < M; b += 1024) {
      unsigned long long mine[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) { const int q = b + 256 * u + tid; mine[u] = __ballot(q < M && token(q) == t); }
      __syncthreads();                                               // the previous list has been read
      if ((tid & 63) == 0)
#pragma unroll
        for (int u = 0; u < 4; ++u) counts[4 * u + (tid >> 6)] = __popcll(mine[u]);
      __syncthreads();
      int total = 0;
#pragma unroll
      for (int w = 0; w < 16; ++w) {                                 // rows in their order: 256 u + 64 wave + lane
        if ((w & 3) == tid >> 6) {
          const unsigned long long own = mine[w >> 2], bit = 1ull << (tid & 63);
          if (own & bit) list[total + __popcll(own & (bit - 1))] = b + 256 * (w >> 2) + tid;
        }
        total += counts[w];
      }
      __syncthreads();
      for (int i = 0; i < total; i += kEmbedAhead) {                 // requested before the first is added: each would cost a memory latency otherwise
        float v[kEmbedAhead][kEmbedCols];
#pragma unroll
        for (int q = 0; q < kEmbedAhead; ++q) {
          const float* src = dx + (size_t)list[i + q < total ? i + q : i] * d;
#pragma unroll
          for (int u = 0; u < kEmbedCols; ++u) v[q][u] = c0 + 256 * u < d ? src[c0 + 256 * u] : 0.f;
        }
#pragma unroll
        for (int q = 0; q < kEmbedAhead; ++q)
#pragma unroll
          for (int u = 0; u < kEmbedCols; ++u) acc[u] = i + q < total ? acc[u] + v[q][u] : acc[u];
      }
    }
  }
#pragma unroll
  for (int u = 0; u < kEmbedCols; ++u) if (c0 + 256 * u < d) row[c0 + 256 * u] = acc[u];
}

}  // namespace

static unsigned grid_1d(int64_t n) { const int64_t b = (n + 255) / 256; return (unsigned)(b < 1 ? 1 : (b > 4096 ? 4096 : b)); }

hipError_t SumQueue::flush() {
  if (count_ == 0) return hipSuccess;
  hipLaunchKernelGGL(colsum_final_kernel, dim3((unsigned)((widest_ + 31) / 32), (unsigned)count_), dim3(256), 0, s_, jobs_);
  used_ = 0; count_ = 0; widest_ = 0;
  return hipGetLastError();
}
hipError_t SumQueue::take(size_t floats, int n_jobs, float** part) {
  const size_t room = (floats + 63) / 64 * 64;
  if (floats > floats_) return hipErrorInvalidValue;
  if (count_ + n_jobs > kSumJobs || used_ + floats > floats_) {
    const hipError_t e = flush();
    if (e != hipSuccess) return e;
  }
  *part = arena_ + used_;
  used_ += room;
  return hipSuccess;
}

hipError_t launch_bw_transpose_bf16(const void* in, int rows, int cols, int64_t ld_in, void* out, int64_t ld_out, hipStream_t s) {
  if (rows < 1 || cols < 1) return hipSuccess;
  const dim3 grid((unsigned)((cols + 63) / 64), (unsigned)((ld_out + 63) / 64));
  hipLaunchKernelGGL((operand_kernel<bf16_t, 0, false, false>), grid, dim3(256), 0, s, reinterpret_cast<const bf16_t*>(in), nullptr, rows, cols, ld_in, reinterpret_cast<bf16_t*>(out), ld_out,
                     nullptr, (int64_t)0, nullptr, 1);
  return hipGetLastError();
}

hipError_t launch_bw_transposes_bf16(const TransposeJobs& jobs, hipStream_t s) {
  int64_t blocks = 0;
  if (jobs.count < 0 || jobs.count > kTransposeJobs) return hipErrorInvalidValue;
  for (int i = 0; i < jobs.count; ++i) {
    const TransposeJob& j = jobs.job[i];
    if (j.rows < 64 || j.cols < 64 || j.rows % 64 || j.cols % 64 || (((uintptr_t)j.in | (uintptr_t)j.out) & 15)) return hipErrorInvalidValue;
    blocks += (int64_t)(j.rows / 64) * (j.cols / 64);
  }
  if (blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(transposes_kernel, dim3((unsigned)blocks), dim3(256), 0, s, jobs);
  return hipGetLastError();
}

hipError_t launch_bw_gradient_operands(const float* dy, const float* u, int relu, int M, int N, void* cols_out, void* rows_out, float* const* dbias, int n_bias, SumQueue& sums, hipStream_t s) {
  if (M < 1 || N < 1 || M % 64 || N % 64 || n_bias < 1 || n_bias > 3 || N % n_bias) return hipErrorInvalidValue;
  const int tiles = M / 64, per = (tiles + kColParts - 1) / kColParts, parts = (tiles + per - 1) / per;
  const dim3 grid((unsigned)(N / 64), (unsigned)parts);
  float* part = nullptr;
  const hipError_t e = sums.take((size_t)parts * N, n_bias, &part);
  if (e != hipSuccess) return e;
#define ZGR_OPERANDS(ACT)                                                                                                                                          \
  hipLaunchKernelGGL((operand_kernel<float, ACT, true, true>), grid, dim3(256), 0, s, dy, u, M, N, (int64_t)N, reinterpret_cast<bf16_t*>(cols_out), (int64_t)M,    \
                     reinterpret_cast<bf16_t*>(rows_out), (int64_t)N, part, per)
  if (!u) ZGR_OPERANDS(0); else if (relu) ZGR_OPERANDS(2); else ZGR_OPERANDS(1);
#undef ZGR_OPERANDS
  const int n = N / n_bias;
  for (int i = 0; i < n_bias; ++i) sums.add(SumJob{part + (size_t)i * n, dbias[i], (int64_t)N, parts, n});
  return hipGetLastError();
}

hipError_t launch_bw_gradient_planes(float* dy, const float* u, int relu, int M, int N, void* cols_out, const void* x, int x_cols, void* x_out, float* const* dbias, int n_bias, SumQueue& sums,
                                     hipStream_t s) {
  if (M < 1 || N < 64 || N % 64 || x_cols < 64 || x_cols % 64 || n_bias < 1 || n_bias > 3 || N % n_bias) return hipErrorInvalidValue;
  const int tiles = (M + 63) / 64, per = (tiles + kColParts - 1) / kColParts, parts = (tiles + per - 1) / per;
  const dim3 grid((unsigned)(N / 64 + x_cols / 64), (unsigned)parts);
  float* part = nullptr;
  const hipError_t e = sums.take((size_t)parts * N, n_bias, &part);
  if (e != hipSuccess) return e;
  auto kern = !u ? gradient_planes_kernel<0> : relu ? gradient_planes_kernel<2> : gradient_planes_kernel<1>;
  hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, dy, u, M, N, reinterpret_cast<bf16_t*>(cols_out), (int64_t)tiles * 64, part, per, reinterpret_cast<const bf16_t*>(x), x_cols,
                     reinterpret_cast<bf16_t*>(x_out));
  const int n = N / n_bias;
  for (int i = 0; i < n_bias; ++i) sums.add(SumJob{part + (size_t)i * n, dbias[i], (int64_t)N, parts, n});
  return hipGetLastError();
}

constexpr int kLnBlocks = 256;       // blocks of the LayerNorm rule, each with a partial sum of both parameter gradients
size_t bw_scratch_floats(int d, int n_widest) {
  const size_t ln = (size_t)2 * kLnBlocks * (size_t)d, sums = (size_t)2 * kColParts * (size_t)n_widest;
  return ln > sums ? ln : sums;
}

hipError_t launch_bw_fill(float* p, int64_t n, float v, hipStream_t s) {
  if (n < 1) return hipSuccess;
  hipLaunchKernelGGL(fill_kernel, dim3(grid_1d(n)), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

hipError_t launch_bw_cross_entropy(float* logits, const int32_t* targets, int rows, int n, float inv_count, float* row_loss, void* d16, int64_t ld16, hipStream_t s) {
#define ZGR_CE(MAXE, TO16) hipLaunchKernelGGL((ce_backward_kernel<MAXE, TO16>), dim3((unsigned)rows), dim3(1024), 0, s, logits, targets, n, inv_count, row_loss, reinterpret_cast<bf16_t*>(d16), ld16)
  if (n <= 8 * 1024) { if (d16) ZGR_CE(8, true); else ZGR_CE(8, false); }
  else               { if (d16) ZGR_CE(50, true); else ZGR_CE(50, false); }
#undef ZGR_CE
  return hipGetLastError();
}

static bool ln_wave_form(int d) { return d % 4 == 0 && d <= 2048; }
static int ln_blocks(int M) { return M < 4 * kLnBlocks ? (M + 3) / 4 : kLnBlocks; }
size_t bw_layernorm_floats(int M, int d) { return ((size_t)2 * (ln_wave_form(d) ? ln_blocks(M) : kColParts) * d + 63) / 64 * 64; }
size_t bw_bias_floats(int M, int n) { const size_t tiles = (size_t)(M + 63) / 64; return std::min(tiles, (size_t)kColParts) * n + 4 * 64; }

bool bw_layernorm_adds_parts(int d) { return ln_wave_form(d); }
hipError_t launch_bw_layernorm(int dtype, const float* x, const void* g, const float* dy, const float* add, float* dx_out, float* stats, float* dg, float* db,
                               SumQueue& sums, int M, int d, float eps, hipStream_t s, int dy_parts) {
  float* part = nullptr;
  if (dy_parts < 1 || (dy_parts > 1 && !ln_wave_form(d))) return hipErrorInvalidValue;
  const int64_t dy_stride = (int64_t)M * d;
  auto queue = [&](int parts) { sums.add(SumJob{part, dg, (int64_t)2 * d, parts, d}); sums.add(SumJob{part + d, db, (int64_t)2 * d, parts, d}); };
  if (ln_wave_form(d)) {
    const int blocks = ln_blocks(M);
    const dim3 grid((unsigned)blocks);
    const hipError_t e = sums.take((size_t)2 * blocks * d, 2, &part);
    if (e != hipSuccess) return e;
#define ZGR_LN_BACKWARD(T, MAXV) hipLaunchKernelGGL((dy_parts > 1 ? ln_backward_wave_kernel<T, MAXV, true> : ln_backward_wave_kernel<T, MAXV, false>), grid, dim3(256), 0, s, x, reinterpret_cast<const T*>(g), dy, dy_parts, dy_stride, add, dx_out, part, M, d, eps)
    if (dtype == 1) { if (d <= 512) ZGR_LN_BACKWARD(bf16_t, 2); else if (d <= 1024) ZGR_LN_BACKWARD(bf16_t, 4); else ZGR_LN_BACKWARD(bf16_t, 8); }
    else            { if (d <= 512) ZGR_LN_BACKWARD(float, 2); else if (d <= 1024) ZGR_LN_BACKWARD(float, 4); else ZGR_LN_BACKWARD(float, 8); }
#undef ZGR_LN_BACKWARD
    queue(blocks);
    return hipGetLastError();
  }
  // the parameter gradients read dy: they go first, so that dx_out may overwrite it
  hipError_t e = sums.take((size_t)2 * kColParts * d, 2, &part);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(ln_stats_kernel, dim3((unsigned)M), dim3(256), 0, s, x, stats, d, eps);
  hipLaunchKernelGGL(ln_param_grad_partial_kernel, dim3((unsigned)((d + 63) / 64), kColParts), dim3(256), 0, s, x, dy, stats, M, d, part);
  queue(kColParts);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (dtype == 1) hipLaunchKernelGGL(ln_backward_kernel<bf16_t>, dim3((unsigned)M), dim3(256), 0, s, x, reinterpret_cast<const bf16_t*>(g), dy, add, dx_out, d, eps);
  else            hipLaunchKernelGGL(ln_backward_kernel<float>, dim3((unsigned)M), dim3(256), 0, s, x, reinterpret_cast<const float*>(g), dy, add, dx_out, d, eps);
  return hipGetLastError();
}

hipError_t launch_bw_act_forward(int dtype, int relu, const float* u, void* f, int64_t n, hipStream_t s) {
  const dim3 grid(grid_1d(n));
  if (dtype == 1) {
    if (relu) hipLaunchKernelGGL((act_forward_kernel<bf16_t, true>), grid, dim3(256), 0, s, u, reinterpret_cast<bf16_t*>(f), n);
    else      hipLaunchKernelGGL((act_forward_kernel<bf16_t, false>), grid, dim3(256), 0, s, u, reinterpret_cast<bf16_t*>(f), n);
  } else {
    if (relu) hipLaunchKernelGGL((act_forward_kernel<float, true>), grid, dim3(256), 0, s, u, reinterpret_cast<float*>(f), n);
    else      hipLaunchKernelGGL((act_forward_kernel<float, false>), grid, dim3(256), 0, s, u, reinterpret_cast<float*>(f), n);
  }
  return hipGetLastError();
}

hipError_t launch_bw_act(int relu, const float* u, float* df, int64_t n, hipStream_t s) {
  if (relu) hipLaunchKernelGGL(act_backward_kernel<true>, dim3(grid_1d(n)), dim3(256), 0, s, u, df, n);
  else      hipLaunchKernelGGL(act_backward_kernel<false>, dim3(grid_1d(n)), dim3(256), 0, s, u, df, n);
  return hipGetLastError();
}

hipError_t launch_bw_add(float* dst, const float* src, int64_t n, hipStream_t s) {
  if (n < 1) return hipSuccess;
  hipLaunchKernelGGL(add_kernel, dim3(grid_1d(n)), dim3(256), 0, s, dst, src, n);
  return hipGetLastError();
}

// The kernels without the [T, T] buffers have a wave per 32 rows, which walks the whole sequence: with few of them most of the chip stands by. Longer than `after`
// tokens and up to `waves` of them the five products with the buffers are the faster form.  Time with the buffers / without, of the whole pass of a 2-block model:
//   fp32 64   4 heads at 64 tokens 0.98, 128 0.94, 512 0.84, 2048 0.80 (256 waves); 24 at 1024 (768) 0.95; 32 at 1024 (1024) 0.99; 24 at 2048 (1536) 1.06, without the causal mask 0.90;
//             32 at 2048 (2048) 1.15 and 0.96; 96 at 1024 (3072) 1.18 and 1.00
//   fp32 32   4 at 128 1.00, 256 0.94, 2048 0.83; 32 at 512 (512) 0.94; 48 at 512 (768) 0.98; 24 at 1024 (768) 1.05         fp32 16   4 at 192 0.99, 256 0.95, 2048 0.82; 32 at 512 0.95; 48 at 512 1.00
//   bf16 64   16 at 128 1.07, 192 1.01, 256 0.97, 4 at 2048 0.67; 32 at 512 0.96; 48 at 384 (576) 1.04; 12 at 2048 (768) 1.15
//   bf16 32   4 at 256 1.00, 16 at 300 1.02, 4 at 384 0.97, 2048 0.89; 32 at 512 1.00; 24 at 1024 1.07                                            bf16 16   4 at 256 0.99, 16 at 300 1.04, 4 at 384 0.93, 512 0.91, 2048 0.83; 32 at 512 0.97; 48 at 512 1.03
static bool bw_attention_has_kernels(int d, int n_head) { const int dh = d / n_head; return (dh == 16 || dh == 32 || dh == 64) && d % 8 == 0; }
struct FewWaves { int after, waves; };
static FewWaves bw_attention_few_waves(int dtype, int dh, int seq, int causal) {
  if (dtype == 0 && dh == 64) return {64, causal || seq <= 256 ? 1024 : 2048};
  if (dtype == 0) return {dh == 32 ? 128 : 192, 512};
  return {dh == 64 ? 192 : 320, 512};
}
static bool bw_attention_buffers(int dtype, int d, int n_head, int batch, int seq, int causal) {
  if (!bw_attention_has_kernels(d, n_head)) return true;
  const FewWaves f = bw_attention_few_waves(dtype, d / n_head, seq, causal);
  return seq > f.after && (int64_t)batch * n_head * ((seq + 31) / 32) <= f.waves;
}
static size_t bw_attention_pair(int heads, int seq) { return ((size_t)heads * seq * seq + 63) / 64 * 64; }
size_t bw_attention_scratch(int dtype, int d, int n_head, int batch, int seq, int causal) {
  const size_t heads = (size_t)batch * n_head, stats = 3 * heads * (((size_t)seq + 31) / 32 * 32);
  if (!bw_attention_has_kernels(d, n_head)) return 2 * bw_attention_pair((int)heads, seq);
  // the largest that a smaller batch or a shorter sequence may ask for, so that room for the largest is room for all: up to `waves` blocks of 32 rows have buffers
  const FewWaves f = bw_attention_few_waves(dtype, d / n_head, seq, causal);
  const size_t rows = std::min(heads * (size_t)seq, (size_t)f.waves * 32);
  return std::max(stats, seq > f.after ? 2 * (rows * (size_t)seq + 64) : (size_t)0);
}

hipError_t launch_bw_attention(int dtype, const void* qkv, const float* dctx, const int32_t* lengths, int batch, int seq, int d, int n_head, int causal,
                               float* scratch, float* dqkv, hipStream_t s) {
  if (batch < 1 || seq < 1 || n_head < 1 || seq > kBackwardMaxSeq || d % n_head != 0) return hipErrorInvalidValue;
  const int dh = d / n_head, heads = batch * n_head;
  if (!bw_attention_buffers(dtype, d, n_head, batch, seq, causal)) {
    const dim3 grid((unsigned)heads * (unsigned)((seq + 31) / 32));
#define ZGR_ATTENTION(T, DH)                                                                                                                                              \
    {                                                                                                                                                                     \
      hipLaunchKernelGGL((attn_backward_q_kernel<T, DH>), grid, dim3(64), 0, s, reinterpret_cast<const T*>(qkv), dctx, lengths, seq, d, n_head, causal, heads, scratch, dqkv);  \
      hipLaunchKernelGGL((attn_backward_kv_kernel<T, DH>), grid, dim3(64), 0, s, reinterpret_cast<const T*>(qkv), dctx, lengths, seq, d, n_head, causal, heads, scratch, dqkv); \
      return hipGetLastError();                                                                                                                                           \
    }
    switch (dh | (dtype == 1 ? 256 : 0)) {
      case 16: ZGR_ATTENTION(float, 16)
      case 32: ZGR_ATTENTION(float, 32)
      case 64: ZGR_ATTENTION(float, 64)
      case 256 | 16: ZGR_ATTENTION(bf16_t, 16)
      case 256 | 32: ZGR_ATTENTION(bf16_t, 32)
      default: ZGR_ATTENTION(bf16_t, 64)
    }
#undef ZGR_ATTENTION
  }
  float* P = scratch;
  float* dS = P + bw_attention_pair(heads, seq);
  // head z = (b, h): the [T, T] buffers are consecutive in z; q, k, v of the head are the columns h dh, d + h dh, 2 d + h dh of
  // the [T, 3 d] rows of sequence b, dctx its columns h dh of [T, d] rows
  const int64_t tt = (int64_t)seq * seq, ld = (int64_t)3 * d;
  const float scale = 1.0f / sqrtf((float)dh);
  const int64_t sq_outer = (int64_t)seq * ld, dc_outer = (int64_t)seq * d, p_outer = n_head * tt;
  const size_t es = dtype == 1 ? 2 : 4;
  const char* q0 = reinterpret_cast<const char*>(qkv);
  const char* k0 = q0 + es * d;
  const char* v0 = k0 + es * d;
  ProductArgs p;
  p.batches = heads; p.zdiv = n_head;
  auto product = [&](const void* A, int a_dtype, bool a_k, int64_t lda, int64_t a_outer, int64_t a_inner, const void* B, int b_dtype, bool b_k, int64_t ldb, int64_t b_outer, int64_t b_inner,
                     float* C, int64_t ldc, int64_t c_outer, int64_t c_inner, int N, int K, float alpha) {
    p.A = A; p.a_dtype = a_dtype; p.a_k = a_k; p.lda = lda; p.a_outer = a_outer; p.a_inner = a_inner;
    p.B = B; p.b_dtype = b_dtype; p.b_k = b_k; p.ldb = ldb; p.b_outer = b_outer; p.b_inner = b_inner;
    p.C = C; p.ldc = ldc; p.c_outer = c_outer; p.c_inner = c_inner;
    p.M = seq; p.N = N; p.K = K; p.alpha = alpha;
    return launch_product(p, s);
  };
  hipError_t e;
  // S [i][j] = sum_t q[i][t] k[j][t] / sqrt dh,  dP [i][j] = sum_t dctx[i][t] v[j][t]
  if ((e = product(q0, dtype, true, ld, sq_outer, dh, k0, dtype, true, ld, sq_outer, dh, P, seq, p_outer, tt, seq, dh, scale)) != hipSuccess) return e;
  if ((e = product(dctx, 0, true, d, dc_outer, dh, v0, dtype, true, ld, sq_outer, dh, dS, seq, p_outer, tt, seq, dh, 1.0f)) != hipSuccess) return e;
  const int64_t rows = (int64_t)heads * seq;
  const dim3 row_grid((unsigned)((rows + 3) / 4));
  if (seq <= 128)      hipLaunchKernelGGL(attn_backward_rows_kernel<2>, row_grid, dim3(256), 0, s, lengths, rows, seq, n_head, causal, P, dS);
  else if (seq <= 512) hipLaunchKernelGGL(attn_backward_rows_kernel<8>, row_grid, dim3(256), 0, s, lengths, rows, seq, n_head, causal, P, dS);
  else                 hipLaunchKernelGGL(attn_backward_rows_kernel<kBackwardMaxSeq / 64>, row_grid, dim3(256), 0, s, lengths, rows, seq, n_head, causal, P, dS);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // dQ [i][t] = sum_j dS[i][j] k[j][t] / sqrt dh,  dK [j][t] = sum_i dS[i][j] q[i][t] / sqrt dh,  dV [j][t] = sum_i P[i][j] dctx[i][t]
  if ((e = product(dS, 0, true, seq, p_outer, tt, k0, dtype, false, ld, sq_outer, dh, dqkv, ld, sq_outer, dh, dh, seq, scale)) != hipSuccess) return e;
  if ((e = product(dS, 0, false, seq, p_outer, tt, q0, dtype, false, ld, sq_outer, dh, dqkv + d, ld, sq_outer, dh, dh, seq, scale)) != hipSuccess) return e;
  return product(P, 0, false, seq, p_outer, tt, dctx, 0, false, d, dc_outer, dh, dqkv + 2 * d, ld, sq_outer, dh, dh, seq, 1.0f);
}

hipError_t launch_bw_embedding(const int32_t* tok, const float* dx, int M, int seq, int d, int vocab, float* dE, float* dPe, int max_pos, hipStream_t s) {
  hipLaunchKernelGGL(embed_backward_kernel, dim3((unsigned)(M + max_pos), (unsigned)((d + 256 * kEmbedCols - 1) / (256 * kEmbedCols))), dim3(256), 0, s, tok, dx, M, seq, d, vocab, dE, dPe);
  return hipGetLastError();
}

}  // namespace zgr
