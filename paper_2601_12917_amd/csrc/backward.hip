// Backward pass of the cloud block of Algorithm 1 (back-propagation on the public dataset with the current weights,
// whose gradients build the basis; Sec. 3.2, paragraph on guided perturbation sampling on the cloud): dL/dtheta of the loss of forward.hip, by the chain rule
// layer by layer, in fp32.  The forward pass that precedes it runs the client's own kernels and keeps every layer's
// intermediate results; these kernels take them back in reverse order.
//
// This runs on the cloud once per stored gradient snapshot, not on the client's step.  The products run on the matrix cores (forward.hip
// for bf16 operands, product.hip for the others); the row-wise rules take one workgroup per row.  Deterministic: no atomics, every
// sum has a fixed order.
#include "backward.h"
#include "product.h"

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

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
// block of 256 threads
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

// ------------------------------------------------------------------ operands for the matrix-core products (bf16 models)
// The bf16 GEMM of the forward pass computes A W^T with both operands contiguous along the contraction.  A backward
// product contracts over another index, so its operands are first written out in bf16 with that index innermost:
//   out[c][r] = in[r][c]   (transpose, 64 x 64 tiles through LDS)      or      out[r][c] = in[r][c]   (rounding only)
// Elements [rows, ld_out) of every output row (transpose) and [cols, ld_out) (rounding) are written as zeros: padding of the
// contraction up to the multiple of 64 the GEMM asks for.
template <typename TIN>
__global__ void __launch_bounds__(256) transpose_bf16_kernel(const TIN* __restrict__ in, int rows, int cols, int64_t ld_in, bf16_t* __restrict__ out, int64_t ld_out) {
  __shared__ float tile[64][65];
  const int r0 = blockIdx.y * 64, c0 = blockIdx.x * 64;
  for (int i = threadIdx.x; i < 64 * 64; i += 256) {
    const int r = i >> 6, c = i & 63;
    tile[r][c] = (r0 + r < rows && c0 + c < cols) ? to_f32(in[(int64_t)(r0 + r) * ld_in + c0 + c]) : 0.f;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < 64 * 64; i += 256) {
    const int c = i >> 6, r = i & 63;
    if (r0 + r < ld_out && c0 + c < cols) from_f32(tile[r][c], out[(int64_t)(c0 + c) * ld_out + r0 + r]);      // tile holds zeros past `rows`
  }
}
__global__ void __launch_bounds__(256) round_bf16_kernel(const float* __restrict__ in, int rows, int cols, int64_t ld_in, bf16_t* __restrict__ out, int64_t ld_out) {
  const int64_t n = (int64_t)rows * ld_out;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const int64_t r = i / ld_out, c = i % ld_out;
    from_f32(c < cols ? in[r * ld_in + c] : 0.f, out[i]);
  }
}

// out[n] = sum_m Y[m ld + n]  (bias gradients), in two stages with a fixed shape so that the order of the additions
// never depends on scheduling: kColParts row chunks are summed side by side (64 columns per block, 4 row groups),
// then the chunk sums are added in chunk order.
constexpr int kColParts = 64;
__global__ void __launch_bounds__(256) colsum_partial_kernel(const float* __restrict__ Y, int M, int N, int64_t ld, float* __restrict__ part) {
  __shared__ float acc[4][64];
  const int c = blockIdx.x * 64 + (threadIdx.x & 63), g = threadIdx.x >> 6;
  const int chunk = (M + kColParts - 1) / kColParts;
  const int m_begin = blockIdx.y * chunk, m_end = min(M, m_begin + chunk);
  float s = 0.f;
  if (c < N)
    for (int m = m_begin + g; m < m_end; m += 4) s += Y[(int64_t)m * ld + c];
  acc[g][threadIdx.x & 63] = s;
  __syncthreads();
  if (g == 0 && c < N) part[(size_t)blockIdx.y * N + c] = (acc[0][threadIdx.x] + acc[1][threadIdx.x]) + (acc[2][threadIdx.x] + acc[3][threadIdx.x]);
}
__global__ void __launch_bounds__(256) colsum_final_kernel(const float* __restrict__ part, int N, float* __restrict__ out) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= N) return;
  float s = 0.f;
  for (int p = 0; p < kColParts; ++p) s += part[(size_t)p * N + c];
  out[c] = s;
}

__global__ void __launch_bounds__(256) fill_kernel(float* __restrict__ p, int64_t n, float v) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) p[i] = v;
}

// ------------------------------------------------------------------ softmax cross-entropy
// In place on a row of logits: d = (softmax - onehot(target)) * inv_count, or zeros for a row without a target.
__global__ void __launch_bounds__(256) ce_backward_kernel(float* __restrict__ logits, const int32_t* __restrict__ targets, int n, float inv_count) {
  __shared__ float red[4];
  float* row = logits + (size_t)blockIdx.x * n;
  const int tgt = targets[blockIdx.x];
  if (tgt < 0 || tgt >= n) {                        // uniform over the block
    for (int i = threadIdx.x; i < n; i += 256) row[i] = 0.f;
    return;
  }
  float mx = -INFINITY;
  for (int i = threadIdx.x; i < n; i += 256) mx = fmaxf(mx, row[i]);
  mx = block_max(mx, red);
  float s = 0.f;
  for (int i = threadIdx.x; i < n; i += 256) s += expf(row[i] - mx);
  s = block_sum(s, red);
  const float inv = 1.0f / s;
  for (int i = threadIdx.x; i < n; i += 256) row[i] = (expf(row[i] - mx) * inv - (i == tgt ? 1.0f : 0.f)) * inv_count;
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

// dg[c] = sum_m dy[m][c] xhat[m][c], db[c] = sum_m dy[m][c]: chunk sums as above (part: [2][kColParts][d]), then
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
    part[(size_t)blockIdx.y * d + c] = (pg[0][threadIdx.x] + pg[1][threadIdx.x]) + (pg[2][threadIdx.x] + pg[3][threadIdx.x]);
    part[(size_t)(kColParts + blockIdx.y) * d + c] = (pb[0][threadIdx.x] + pb[1][threadIdx.x]) + (pb[2][threadIdx.x] + pb[3][threadIdx.x]);
  }
}

// ------------------------------------------------------------------ feed-forward activation: erf-GELU or ReLU
template <typename T, bool RELU>
__global__ void __launch_bounds__(256) act_forward_kernel(const float* __restrict__ u, T* __restrict__ f, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const float x = u[i];
    from_f32(RELU ? fmaxf(x, 0.f) : 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)), f[i]);
  }
}
// du = df * act'(u), in place on df: GELU' = Phi(u) + u phi(u), ReLU' = [u > 0]
template <bool RELU>
__global__ void __launch_bounds__(256) act_backward_kernel(const float* __restrict__ u, float* __restrict__ df, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const float x = u[i];
    if (RELU) { if (!(x > 0.f)) df[i] = 0.f; continue; }
    const float cdf = 0.5f * (1.0f + erff(x * 0.70710678118654752f));
    const float pdf = 0.3989422804014327f * expf(-0.5f * x * x);
    df[i] *= cdf + x * pdf;
  }
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
// One block per row (b, h, i) of the two [T, T] buffers; a thread holds up to MAXJ of the row's entries (T <= 256 MAXJ).
__global__ void __launch_bounds__(256) attn_backward_rows_kernel(const int32_t* __restrict__ lengths, int seq, int n_head, int causal,
                                                                 float* __restrict__ P, float* __restrict__ dS) {
  __shared__ float red[4];
  const int i = blockIdx.x % seq, b = blockIdx.x / (seq * n_head);
  int kend = lengths ? lengths[b] : seq;
  kend = kend < seq ? kend : seq;
  if (causal) kend = kend < i + 1 ? kend : i + 1;
  float* prow = P + (size_t)blockIdx.x * seq;
  float* srow = dS + (size_t)blockIdx.x * seq;
  constexpr int MAXJ = kBackwardMaxSeq / 256;
  float sc[MAXJ], dp[MAXJ];
  float mx = -INFINITY;
#pragma unroll
  for (int u = 0; u < MAXJ; ++u) {
    const int j = threadIdx.x + 256 * u;
    sc[u] = -INFINITY; dp[u] = 0.f;
    if (j < kend) { sc[u] = prow[j]; dp[u] = srow[j]; mx = fmaxf(mx, sc[u]); }
  }
  mx = block_max(mx, red);
  float den = 0.f;
#pragma unroll
  for (int u = 0; u < MAXJ; ++u) { sc[u] = (threadIdx.x + 256 * u < kend) ? expf(sc[u] - mx) : 0.f; den += sc[u]; }
  den = block_sum(den, red);
  const float inv = den > 0.f ? 1.0f / den : 0.f;
  float dot = 0.f;
#pragma unroll
  for (int u = 0; u < MAXJ; ++u) { sc[u] *= inv; dot += sc[u] * dp[u]; }
  dot = block_sum(dot, red);
#pragma unroll
  for (int u = 0; u < MAXJ; ++u) {
    const int j = threadIdx.x + 256 * u;
    if (j < seq) { prow[j] = sc[u]; srow[j] = sc[u] * (dp[u] - dot); }
  }
}

// ------------------------------------------------------------------ embeddings
// x0[m] = E[tok[m]] + Pe[m mod seq]: one thread per column walks the rows in order (tokens repeat, so the adds into
// one row of dE must be ordered to be reproducible); dE accumulates (the tied head has written it), dPe is overwritten.
__global__ void __launch_bounds__(256) embed_backward_kernel(const int32_t* __restrict__ tok, const float* __restrict__ dx, int M, int seq, int d, int vocab,
                                                             float* __restrict__ dE, float* __restrict__ dPe, int max_pos) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= d) return;
  for (int p = 0; p < max_pos; ++p) dPe[(size_t)p * d + c] = 0.f;
  for (int m = 0; m < M; ++m) {
    int t = tok[m];
    t = t < 0 ? 0 : (t >= vocab ? vocab - 1 : t);
    const float g = dx[(size_t)m * d + c];
    dE[(size_t)t * d + c] += g;
    dPe[(size_t)(m % seq) * d + c] += g;
  }
}

}  // namespace

static unsigned grid_1d(int64_t n) { const int64_t b = (n + 255) / 256; return (unsigned)(b < 1 ? 1 : (b > 4096 ? 4096 : b)); }

hipError_t launch_bw_transpose_bf16(int in_dtype, const void* in, int rows, int cols, int64_t ld_in, void* out, int64_t ld_out, hipStream_t s) {
  if (rows < 1 || cols < 1) return hipSuccess;
  const dim3 grid((unsigned)((cols + 63) / 64), (unsigned)((ld_out + 63) / 64));
  if (in_dtype == 1) hipLaunchKernelGGL(transpose_bf16_kernel<bf16_t>, grid, dim3(256), 0, s, reinterpret_cast<const bf16_t*>(in), rows, cols, ld_in, reinterpret_cast<bf16_t*>(out), ld_out);
  else               hipLaunchKernelGGL(transpose_bf16_kernel<float>, grid, dim3(256), 0, s, reinterpret_cast<const float*>(in), rows, cols, ld_in, reinterpret_cast<bf16_t*>(out), ld_out);
  return hipGetLastError();
}

hipError_t launch_bw_round_bf16(const float* in, int rows, int cols, int64_t ld_in, void* out, int64_t ld_out, hipStream_t s) {
  if (rows < 1 || cols < 1) return hipSuccess;
  hipLaunchKernelGGL(round_bf16_kernel, dim3(grid_1d((int64_t)rows * ld_out)), dim3(256), 0, s, in, rows, cols, ld_in, reinterpret_cast<bf16_t*>(out), ld_out);
  return hipGetLastError();
}

size_t bw_colsum_scratch_floats(int n_max) { return (size_t)2 * kColParts * (size_t)n_max; }

hipError_t launch_bw_colsum(const float* Y, int M, int N, int64_t ld, float* out, float* part, hipStream_t s) {
  hipLaunchKernelGGL(colsum_partial_kernel, dim3((unsigned)((N + 63) / 64), kColParts), dim3(256), 0, s, Y, M, N, ld, part);
  hipLaunchKernelGGL(colsum_final_kernel, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, s, part, N, out);
  return hipGetLastError();
}

hipError_t launch_bw_fill(float* p, int64_t n, float v, hipStream_t s) {
  if (n < 1) return hipSuccess;
  hipLaunchKernelGGL(fill_kernel, dim3(grid_1d(n)), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

hipError_t launch_bw_cross_entropy(float* logits, const int32_t* targets, int rows, int n, float inv_count, hipStream_t s) {
  hipLaunchKernelGGL(ce_backward_kernel, dim3((unsigned)rows), dim3(256), 0, s, logits, targets, n, inv_count);
  return hipGetLastError();
}

hipError_t launch_bw_layernorm(int dtype, const float* x, const void* g, const float* dy, const float* add, float* dx_out, float* stats, float* dg, float* db,
                               float* part, int M, int d, float eps, hipStream_t s) {
  // the parameter gradients read dy: they go first, so that dx_out may overwrite it
  hipLaunchKernelGGL(ln_stats_kernel, dim3((unsigned)M), dim3(256), 0, s, x, stats, d, eps);
  hipLaunchKernelGGL(ln_param_grad_partial_kernel, dim3((unsigned)((d + 63) / 64), kColParts), dim3(256), 0, s, x, dy, stats, M, d, part);
  hipLaunchKernelGGL(colsum_final_kernel, dim3((unsigned)((d + 255) / 256)), dim3(256), 0, s, part, d, dg);
  hipLaunchKernelGGL(colsum_final_kernel, dim3((unsigned)((d + 255) / 256)), dim3(256), 0, s, part + (size_t)kColParts * d, d, db);
  hipError_t e = hipGetLastError();
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

hipError_t launch_bw_attention(int dtype, const void* qkv, const float* dctx, const int32_t* lengths, int batch, int seq, int d, int n_head, int causal,
                               float* P, float* dS, float* dqkv, hipStream_t s) {
  if (batch < 1 || seq < 1 || n_head < 1 || seq > kBackwardMaxSeq || d % n_head != 0) return hipErrorInvalidValue;
  const int dh = d / n_head, heads = batch * n_head;
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
  hipLaunchKernelGGL(attn_backward_rows_kernel, dim3((unsigned)heads * seq), dim3(256), 0, s, lengths, seq, n_head, causal, P, dS);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // dQ [i][t] = sum_j dS[i][j] k[j][t] / sqrt dh,  dK [j][t] = sum_i dS[i][j] q[i][t] / sqrt dh,  dV [j][t] = sum_i P[i][j] dctx[i][t]
  if ((e = product(dS, 0, true, seq, p_outer, tt, k0, dtype, false, ld, sq_outer, dh, dqkv, ld, sq_outer, dh, dh, seq, scale)) != hipSuccess) return e;
  if ((e = product(dS, 0, false, seq, p_outer, tt, q0, dtype, false, ld, sq_outer, dh, dqkv + d, ld, sq_outer, dh, dh, seq, scale)) != hipSuccess) return e;
  return product(P, 0, false, seq, p_outer, tt, dctx, 0, false, d, dc_outer, dh, dqkv + 2 * d, ld, sq_outer, dh, dh, seq, 1.0f);
}

hipError_t launch_bw_embedding(const int32_t* tok, const float* dx, int M, int seq, int d, int vocab, float* dE, float* dPe, int max_pos, hipStream_t s) {
  hipLaunchKernelGGL(embed_backward_kernel, dim3((unsigned)((d + 255) / 256)), dim3(256), 0, s, tok, dx, M, seq, d, vocab, dE, dPe, max_pos);
  return hipGetLastError();
}

}  // namespace zgr
