// Cloud block of Algorithm 1 (the gradients collected on the cloud build the basis; Sec. 3.2, paragraph on guided
// perturbation sampling on the cloud): the orthonormal basis U [rows, k] of one weight matrix from its stored gradient snapshots G_1 .. G_s
// (each [rows, cols] fp32, row-major), and the gradient of the least-squares model.
//
// U spans the k-dimensional subspace of R^rows that captures the most of the snapshots (the k leading left singular
// vectors of [G_1 | ... | G_s]).  It is reached by block subspace iteration on the operator C = sum_t G_t G_t^T,
// which is never formed:
//     Y = sum_t G_t Omega              (Omega [cols, k]: the caller's seeded Gaussian start)
//     Q = orth(Y)
//     n_iter times:  T_t = G_t^T Q,  Y = sum_t G_t T_t,  Q = orth(Y)
// Each sweep reads every snapshot twice and is a pair of tall-skinny products (HBM-bound: 2 rows cols 4 bytes per
// snapshot and sweep); orth is Gram-Schmidt in matrix form (Cholesky-QR) in fp64, taken twice.  The subspace converges like (sigma_{k+1} / sigma_k)^(2 n):
// the caller picks n_iter for the gap it expects.  This runs every gamma rounds on the cloud, not on the client's
// step: it is written to be correct and bandwidth-shaped, not tuned.
#include "internal.h"

namespace zgr {

namespace {

constexpr int kTile = 64;      // columns (or rows) of G a block owns
constexpr int kChunk = 32;     // the other dimension, staged per step

// T[c][j] (+)= sum_r G[r][c] Q[r][j],  c < cols, j < n: G [rows, cols] (row stride ldg), Q [rows, n] (row stride ldq).
// Block = 64 columns c x 64 columns j (blockIdx.y tiles j); thread (c = tid % 64, jg = tid / 64) holds 16 values of j.
// blockIdx.z = part of the sum: rows [z row_part, (z + 1) row_part) go to T + z t_part (partial sums that sum_parts_kernel adds in order).
__global__ void __launch_bounds__(256) gt_q_kernel(const float* __restrict__ G, int64_t rows, int64_t cols, int64_t ldg, const float* __restrict__ Q, int n, int64_t ldq,
                                                   float* __restrict__ T, int64_t ldt, float scale, int accumulate, int64_t row_part, int64_t t_part) {
  __shared__ float Gs[kChunk][kTile + 1], Qs[kChunk][kTile + 1];
  const int tid = threadIdx.x, cl = tid & 63, jg = tid >> 6;
  const int64_t c0 = (int64_t)blockIdx.x * kTile;
  const int j0 = blockIdx.y * kTile;
  const int64_t r_begin = (int64_t)blockIdx.z * row_part;
  rows = rows < r_begin + row_part ? rows : r_begin + row_part;
  T += (int64_t)blockIdx.z * t_part;
  float acc[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;
  for (int64_t r0 = r_begin; r0 < rows; r0 += kChunk) {
    __syncthreads();
    for (int i = tid; i < kChunk * kTile; i += 256) {
      const int rr = i >> 6, cc = i & 63;
      const int64_t r = r0 + rr;
      Gs[rr][cc] = (r < rows && c0 + cc < cols) ? G[r * ldg + c0 + cc] : 0.f;
      Qs[rr][cc] = (r < rows && j0 + cc < n) ? Q[r * ldq + j0 + cc] : 0.f;
    }
    __syncthreads();
#pragma unroll 4
    for (int rr = 0; rr < kChunk; ++rr) {
      const float g = Gs[rr][cl];
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[i] = __builtin_fmaf(g, Qs[rr][jg * 16 + i], acc[i]);
    }
  }
  if (c0 + cl < cols)
    for (int i = 0; i < 16; ++i) {
      const int j = j0 + jg * 16 + i;
      if (j < n) { float* t = T + (c0 + cl) * ldt + j; *t = (accumulate ? *t : 0.f) + scale * acc[i]; }
    }
}

// Y[r][j] (+)= sum_c G[r][c] T[c][j],  r < rows, j < k <= 64.  Block = 64 rows; thread (r = tid % 64, jg = tid / 64).
// blockIdx.y = part of the sum: columns [y col_part, (y + 1) col_part) go to Y + y y_part.
__global__ void __launch_bounds__(256) g_t_kernel(const float* __restrict__ G, int64_t rows, int64_t cols, const float* __restrict__ T, int k,
                                                  float* __restrict__ Y, int accumulate, int64_t col_part, int64_t y_part) {
  __shared__ float Gs[kTile][kChunk + 1], Ts[kChunk][kTile + 1];
  const int tid = threadIdx.x, rl = tid & 63, jg = tid >> 6;
  const int64_t r0 = (int64_t)blockIdx.x * kTile;
  const int64_t c_begin = (int64_t)blockIdx.y * col_part;
  const int64_t c_end = cols < c_begin + col_part ? cols : c_begin + col_part;
  Y += (int64_t)blockIdx.y * y_part;
  float acc[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;
  for (int64_t c0 = c_begin; c0 < c_end; c0 += kChunk) {
    __syncthreads();
    for (int i = tid; i < kTile * kChunk; i += 256) {
      const int rr = i >> 5, cc = i & 31;                 // consecutive threads read consecutive columns of G
      Gs[rr][cc] = (r0 + rr < rows && c0 + cc < c_end) ? G[(r0 + rr) * cols + c0 + cc] : 0.f;
    }
    for (int i = tid; i < kChunk * kTile; i += 256) {
      const int cc = i >> 6, jj = i & 63;
      Ts[cc][jj] = (c0 + cc < c_end && jj < k) ? T[(c0 + cc) * k + jj] : 0.f;
    }
    __syncthreads();
#pragma unroll 4
    for (int cc = 0; cc < kChunk; ++cc) {
      const float g = Gs[rl][cc];
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[i] = __builtin_fmaf(g, Ts[cc][jg * 16 + i], acc[i]);
    }
  }
  if (r0 + rl < rows)
    for (int i = 0; i < 16; ++i) {
      const int j = jg * 16 + i;
      if (j < k) { float* y = Y + (r0 + rl) * k + j; *y = (accumulate ? *y : 0.f) + acc[i]; }
    }
}

// In-place orthonormalisation of the k columns of Y [rows, k] (row stride k), in the order of the columns: Gram-Schmidt in its
// matrix form, Cholesky-QR, taken twice.  One round is
//     W = Y^T Y        (fp64 sums, one partial W per block of rows: gram_kernel)
//     W = L L^T        (fp64, one workgroup, which first adds the partial W in their order: cholesky_kernel)
//     Y <- Y L^-T      (fp64 forward substitution, one row per thread: substitute_kernel)
// Column j becomes y_j minus its projection on the earlier columns, divided by the norm that is left.  The second round takes
// out what the first left of the earlier columns (at most cond(Y)^2 2^-53, 1e-4 at the dependence threshold), so the result is
// orthonormal to the rounding of its fp32 entries.  A column that the earlier ones already span (norm below 1e-6 of what it
// started with) is stored as zeros and counted in *dependent.
// The column-by-column form needs 3 k dependent sweeps over the rows, which one workgroup has to make: 33 ms for
// 8192 x 64, waiting for the L2 in every sweep.  This form reads the block three times per round, spread over all the rows'
// blocks, and what is serial (k pivots) stays inside one workgroup's LDS.
constexpr int kGramRows = 64;        // rows staged at a time
constexpr int kGramMaxParts = 64;    // partial W at most: the workgroup that factorises adds them all
constexpr int kGramLd = kMaxK + 1;

// part[p][i k + j] = sum over the rows of part p of Y[r][i] Y[r][j], for every i >= j (16 x 16 tiles on and below the diagonal).
// Thread (tx, ty) holds element (16 a + ty, 16 b + tx) of each tile (a, b).  NT = ceil(k / 16) tiles.
template <int NT>
__global__ void __launch_bounds__(256) gram_kernel(const float* __restrict__ Y, int64_t rows, int k, int64_t rows_per_part, double* __restrict__ part) {
  __shared__ float Ys[kGramRows][NT * 16 + 1];
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  const int64_t r_begin = (int64_t)blockIdx.x * rows_per_part;
  const int64_t r_end = rows < r_begin + rows_per_part ? rows : r_begin + rows_per_part;
  double acc[NT][NT];
#pragma unroll
  for (int a = 0; a < NT; ++a)
#pragma unroll
    for (int b = 0; b <= a; ++b) acc[a][b] = 0.0;
  for (int64_t r0 = r_begin; r0 < r_end; r0 += kGramRows) {
    __syncthreads();
    for (int i = tid; i < kGramRows * NT * 16; i += 256) {
      const int rr = i / (NT * 16), c = i % (NT * 16);
      Ys[rr][c] = (r0 + rr < r_end && c < k) ? Y[(r0 + rr) * k + c] : 0.f;
    }
    __syncthreads();
#pragma unroll 2
    for (int rr = 0; rr < kGramRows; ++rr) {
      double yi[NT], yj[NT];
#pragma unroll
      for (int a = 0; a < NT; ++a) { yi[a] = (double)Ys[rr][16 * a + ty]; yj[a] = (double)Ys[rr][16 * a + tx]; }
#pragma unroll
      for (int a = 0; a < NT; ++a)
#pragma unroll
        for (int b = 0; b <= a; ++b) acc[a][b] = __builtin_fma(yi[a], yj[b], acc[a][b]);
    }
  }
  double* out = part + (int64_t)blockIdx.x * k * k;
#pragma unroll
  for (int a = 0; a < NT; ++a)
#pragma unroll
    for (int b = 0; b <= a; ++b) {
      const int i = 16 * a + ty, j = 16 * b + tx;
      if (i < k && j <= i) out[i * k + j] = acc[a][b];
    }
}

// Adds the partial W and factorises it in LDS, one pivot per barrier.  fac [k][k]: below the diagonal L, on it 1 / L_jj
// (0 for a dependent column, whose row and column of L are zero as well).
__global__ void __launch_bounds__(256) cholesky_kernel(const double* __restrict__ part, int n_parts, int k, double* __restrict__ fac, int* __restrict__ dependent) {
  __shared__ double W[kMaxK][kGramLd];
  __shared__ double inv[kMaxK], norm0[kMaxK];
  const int tid = threadIdx.x;
  const int n = k * k;
  for (int e = tid; e < n; e += 256) {
    const int i = e / k, j = e % k;
    if (j > i) continue;
    double v = 0.0;
#pragma unroll 8
    for (int p = 0; p < n_parts; ++p) v += part[(int64_t)p * n + e];
    W[i][j] = v;
    if (i == j) norm0[j] = v;                      // the column's size before anything is taken out
  }
  int n_dep = 0;
  const int tx = tid & 15, ty = tid >> 4;
  for (int j = 0; j < k; ++j) {
    __syncthreads();                               // W is final up to column j
    const double pivot = W[j][j];
    const bool dep = !(pivot > 1e-12 * norm0[j]) || !(pivot > 0.0);
    n_dep += dep;
    const double ip = dep ? 0.0 : 1.0 / pivot;
    if (tid == 0) inv[j] = dep ? 0.0 : 1.0 / sqrt(pivot);
    for (int i = j + 1 + ty; i < k; i += 16) {
      const double f = W[i][j] * ip;
      for (int c = j + 1 + tx; c <= i; c += 16) W[i][c] -= f * W[c][j];
    }
  }
  __syncthreads();
  for (int e = tid; e < n; e += 256) {
    const int i = e / k, j = e % k;
    fac[e] = j < i ? W[i][j] * inv[j] : (j == i ? inv[i] : 0.0);
  }
  if (tid == 0) *dependent = n_dep;
}

// Row y of Y becomes q with q_j = (y_j - sum_{i<j} L_ji q_i) / L_jj.  One wave per block, 64 rows, one row per lane in registers;
// rows come and go through LDS so that global accesses are contiguous.
template <int NT>
__global__ void __launch_bounds__(64) substitute_kernel(float* __restrict__ Y, int64_t rows, int k, const double* __restrict__ fac) {
  constexpr int KP = NT * 16;
  __shared__ double F[KP][KP];
  __shared__ float Ys[64][KP + 1];
  const int lane = threadIdx.x;
  const int64_t r0 = (int64_t)blockIdx.x * 64;
  const int n_rows = (int)(rows - r0 < 64 ? rows - r0 : 64);
  for (int i = lane; i < KP * KP; i += 64) { const int a = i / KP, b = i % KP; F[a][b] = (a < k && b < k) ? fac[a * k + b] : 0.0; }
  for (int i = lane; i < n_rows * k; i += 64) Ys[i / k][i % k] = Y[r0 * k + i];
  __syncthreads();
  double q[KP];
#pragma unroll
  for (int j = 0; j < KP; ++j) {
    double v = j < k ? (double)Ys[lane][j] : 0.0;
#pragma unroll
    for (int i = 0; i < j; ++i) v = __builtin_fma(-F[j][i], q[i], v);
    q[j] = v * F[j][j];
    if (j < k) Ys[lane][j] = (float)q[j];
  }
  __syncthreads();
  for (int i = lane; i < n_rows * k; i += 64) Y[r0 * k + i] = Ys[i / k][i % k];
}

// out[i] = (accumulate ? out[i] : 0) + scale (part[0][i] + part[1][i] + ...): the parts of a split sum, added in their order
__global__ void __launch_bounds__(256) sum_parts_kernel(const float* __restrict__ part, int n_parts, int64_t stride, int64_t n, float* __restrict__ out, float scale, int accumulate) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    float v = 0.f;
    for (int z = 0; z < n_parts; ++z) v += part[(int64_t)z * stride + i];
    out[i] = (accumulate ? out[i] : 0.f) + scale * v;
  }
}

__global__ void __launch_bounds__(256) copy_basis_kernel(const float* __restrict__ Q, int64_t rows, int k, float* __restrict__ U, int ldu) {
  const int64_t n = rows * k;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) U[(i / k) * ldu + (i % k)] = Q[i];
}

// R[b][o] -= Y[b][o]  (R holds the predictions on entry)
__global__ void __launch_bounds__(256) residual_kernel(float* __restrict__ R, const float* __restrict__ Y, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) R[i] -= Y[i];
}

}  // namespace

// How many parts to split a sum over `span` terms into, so that `blocks` blocks become about one per CU-slot: at most kCloudMaxParts,
// each part a whole number of staged chunks.
static int cloud_sum_parts(int64_t blocks, int64_t span) {
  int64_t z = blocks > 0 ? 512 / blocks : 1;
  const int64_t chunks = (span + kChunk - 1) / kChunk;
  if (z > chunks) z = chunks;
  if (z > kCloudMaxParts) z = kCloudMaxParts;
  return z < 1 ? 1 : (int)z;
}

static hipError_t launch_sum_parts(const float* part, int n_parts, int64_t stride, int64_t n, float* out, float scale, int accumulate, hipStream_t s) {
  hipLaunchKernelGGL(sum_parts_kernel, dim3((unsigned)(n / 256 + 1 < 1024 ? n / 256 + 1 : 1024)), dim3(256), 0, s, part, n_parts, stride, n, out, scale, accumulate);
  return hipGetLastError();
}

// part: scratch of kCloudMaxParts * cols * n floats (ldt == n), or NULL for a single pass over all the rows
hipError_t launch_cloud_gt_q(const float* G, int64_t rows, int64_t cols, int64_t ldg, const float* Q, int n, int64_t ldq, float* T, int64_t ldt, float scale,
                             int accumulate, hipStream_t s, float* part) {
  const unsigned gx = (unsigned)((cols + kTile - 1) / kTile), gy = (unsigned)((n + kTile - 1) / kTile);
  const int z = (part && ldt == n) ? cloud_sum_parts((int64_t)gx * gy, rows) : 1;
  if (z <= 1) {
    hipLaunchKernelGGL(gt_q_kernel, dim3(gx, gy), dim3(256), 0, s, G, rows, cols, ldg, Q, n, ldq, T, ldt, scale, accumulate, rows, (int64_t)0);
    return hipGetLastError();
  }
  const int64_t chunks = (rows + kChunk - 1) / kChunk, row_part = (chunks + z - 1) / z * kChunk, stride = cols * (int64_t)n;
  hipLaunchKernelGGL(gt_q_kernel, dim3(gx, gy, (unsigned)z), dim3(256), 0, s, G, rows, cols, ldg, Q, n, ldq, part, (int64_t)n, 1.0f, 0, row_part, stride);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_sum_parts(part, z, stride, stride, T, scale, accumulate, s);
}

// part: scratch of kCloudMaxParts * rows * k floats, or NULL for a single pass over all the columns
hipError_t launch_cloud_g_t(const float* G, int64_t rows, int64_t cols, const float* T, int k, float* Y, int accumulate, hipStream_t s, float* part) {
  const unsigned gx = (unsigned)((rows + kTile - 1) / kTile);
  const int z = part ? cloud_sum_parts(gx, cols) : 1;
  if (z <= 1) {
    hipLaunchKernelGGL(g_t_kernel, dim3(gx), dim3(256), 0, s, G, rows, cols, T, k, Y, accumulate, cols, (int64_t)0);
    return hipGetLastError();
  }
  const int64_t chunks = (cols + kChunk - 1) / kChunk, col_part = (chunks + z - 1) / z * kChunk, stride = rows * (int64_t)k;
  hipLaunchKernelGGL(g_t_kernel, dim3(gx, (unsigned)z), dim3(256), 0, s, G, rows, cols, T, k, part, 0, col_part, stride);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_sum_parts(part, z, stride, stride, Y, 1.0f, accumulate, s);
}

size_t cloud_orth_scratch_doubles(int64_t rows, int k) {
  const int64_t parts = (rows + kGramRows - 1) / kGramRows;
  return (size_t)((parts < kGramMaxParts ? parts : kGramMaxParts) + 1) * (size_t)k * (size_t)k;
}

template <int NT>
static hipError_t orth_round(float* Y, int64_t rows, int k, int* dependent, double* scratch, hipStream_t s) {
  const int64_t chunks = (rows + kGramRows - 1) / kGramRows;
  const int64_t per = (chunks + kGramMaxParts - 1) / kGramMaxParts, parts = (chunks + per - 1) / per;
  double* fac = scratch + parts * k * k;
  hipLaunchKernelGGL(gram_kernel<NT>, dim3((unsigned)parts), dim3(256), 0, s, Y, rows, k, per * kGramRows, scratch);
  hipLaunchKernelGGL(cholesky_kernel, dim3(1), dim3(256), 0, s, scratch, (int)parts, k, fac, dependent);
  hipLaunchKernelGGL(substitute_kernel<NT>, dim3((unsigned)((rows + 63) / 64)), dim3(64), 0, s, Y, rows, k, fac);
  return hipGetLastError();
}

hipError_t launch_cloud_orth(float* Y, int64_t rows, int k, int* dependent, double* scratch, hipStream_t s) {
  for (int round = 0; round < 2; ++round) {                 // the count of the second round includes the first one's zero columns
    hipError_t e;
    switch ((k + 15) / 16) {
      case 1:  e = orth_round<1>(Y, rows, k, dependent, scratch, s); break;
      case 2:  e = orth_round<2>(Y, rows, k, dependent, scratch, s); break;
      case 3:  e = orth_round<3>(Y, rows, k, dependent, scratch, s); break;
      default: e = orth_round<4>(Y, rows, k, dependent, scratch, s); break;
    }
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_cloud_copy_basis(const float* Q, int64_t rows, int k, float* U, int ldu, hipStream_t s) {
  const int64_t n = rows * k;
  hipLaunchKernelGGL(copy_basis_kernel, dim3((unsigned)(n / 256 + 1 < 1024 ? n / 256 + 1 : 1024)), dim3(256), 0, s, Q, rows, k, U, ldu);
  return hipGetLastError();
}

hipError_t launch_cloud_residual(float* R, const float* Y, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(residual_kernel, dim3((unsigned)(n / 256 + 1 < 1024 ? n / 256 + 1 : 1024)), dim3(256), 0, s, R, Y, n);
  return hipGetLastError();
}

}  // namespace zgr
