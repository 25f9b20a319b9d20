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
// Each sweep reads every snapshot twice and is a pair of tall-skinny products (2 rows cols 4 bytes per
// snapshot and sweep); orth is Gram-Schmidt in matrix form (Cholesky-QR), taken twice, in pairs of doubles and in fp64.  The subspace converges like
// (sigma_{k+1} / sigma_k)^(2 n): the caller picks n_iter for the gap it expects.
#include "internal.h"
#include <type_traits>

namespace zgr {

namespace {

// Both products run on the fp32 matrix instruction (16x16x4), a wave owning a 64 x 64 piece of the result and a share of the
// sum, with the operands loaded from global memory straight into the layout the instruction takes: lane (i = lane % 16,
// kg = lane / 16) supplies element i of the free index and element kg of the summed one.  Nothing passes through LDS but the
// waves' partial results at the end.  At 8192 x 2048 and rank 64 a product reads 64 MB (13 us at the rate of a large copy) and
// multiplies 2.1 GFLOP (14 us on these matrix cores); on the vector unit, with both operands
// staged in LDS, it took 180 us; three snapshots together now take 63-66 us, 0.65 of the matrix cores' rate.
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kTile = 64;      // rows (or columns) of G and columns of the block a wave's result covers
constexpr int kStep = 16;      // terms of the sum a wave takes per step
constexpr int kWaves = 4;      // waves of a block: they take turns over the steps of the block's part of the sum

// Nothing is scheduled across this point: left to itself the compiler moves a step's loads down to where they are used.
__device__ __forceinline__ void in_this_order() {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_sched_barrier(0);
#endif
}

// A value all lanes agree on as a scalar (a wave's index, its number of steps): every address of its main loop is then a scalar base
// and a lane offset that stays the same (buffer addressing), and the loop holds loads, matrix instructions and scalar arithmetic
// only.  With vector instructions for the addresses each of them queued behind the matrix instructions of the SIMD's other waves:
// 111 us for 48 us of matrix instructions and 23 us of loads.
__device__ __forceinline__ int uniform(int v) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_readfirstlane(v);
#else
  return v;
#endif
}
// The float(s) `byte` bytes (< 2^32, a multiple of 4) past a scalar base.
__device__ __forceinline__ float load1_at(const float* base, uint32_t byte) {
#if defined(__HIP_DEVICE_COMPILE__)
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, 0xFFFFFFFFu, 0x00020000);
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, byte, 0, 0));
#else
  return base[byte / 4];
#endif
}
__device__ __forceinline__ f32x4 load4_at(const float* base, uint32_t byte) {
#if defined(__HIP_DEVICE_COMPILE__)
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, 0xFFFFFFFFu, 0x00020000);
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, byte, 0, 0));
#else
  return f32x4{base[byte / 4], base[byte / 4 + 1], base[byte / 4 + 2], base[byte / 4 + 3]};
#endif
}

// Adds the four waves' accumulators in a fixed order: ((0 + 2) + (1 + 3)), left in wave 0.
template <int NT> __device__ __forceinline__ void add_waves(f32x4 (&acc)[4][NT], float* lds, int wave, int lane) {
#pragma unroll
  for (int half = 2; half >= 1; half >>= 1) {
    __syncthreads();
    if (wave >= half && wave < 2 * half)
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int n = 0; n < NT; ++n) *reinterpret_cast<f32x4*>(lds + (((wave - half) * 4 * NT + t * NT + n) * 64 + lane) * 4) = acc[t][n];
    __syncthreads();
    if (wave < half)
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int n = 0; n < NT; ++n) acc[t][n] += *reinterpret_cast<const f32x4*>(lds + ((wave * 4 * NT + t * NT + n) * 64 + lane) * 4);
  }
}

// T[c][j] (+)= scale sum_r G[r][c] Q[r][j]: G [rows, cols] (row stride ldg), Q [rows, n] (row stride ldq), T row stride ldt.
// blockIdx.x: 64 columns c; blockIdx.y: NT 16 columns j, or, where one such tile is all (one_tile), the snapshot; blockIdx.z = part of the sum:
// rows [part row_part, (part + 1) row_part), result at T + (snapshot gridDim.z + part) t_part.  A lane's four consecutive columns of G feed four tiles: tile m holds the
// columns c0 + 4 i + m (a lane that would reach past the last column takes the last four instead).  NEAR: the lane offsets of a step fit
// 32 bits and there are four columns; the general form is for what is left.
template <int NT, bool NEAR>
__global__ void __launch_bounds__(64 * kWaves, 2) gt_q_kernel(CloudSnaps g, int one_tile, int64_t rows, int64_t cols, int64_t ldg, const float* __restrict__ Q, int n, int64_t ldq,
                                                           float* __restrict__ T, int64_t ldt, float scale, int accumulate, int64_t row_part, int64_t t_part) {
  __shared__ __attribute__((aligned(16))) float lds[2 * 4 * NT * 256];
  const int lane = threadIdx.x & 63, wave = uniform((int)threadIdx.x >> 6), i16 = lane & 15, kg = lane >> 4;
  const int snap = one_tile ? blockIdx.y : 0;
  const float* G = g.G[snap];
  const int64_t r_begin = (int64_t)blockIdx.z * row_part;
  const int64_t r_end = rows < r_begin + row_part ? rows : r_begin + row_part;
  const int64_t c0 = (int64_t)blockIdx.x * kTile;
  const int j0 = one_tile ? 0 : blockIdx.y * NT * 16;
  T += (int64_t)(snap * gridDim.z + blockIdx.z) * t_part;
  // a lane past the last column (of G or of Q) repeats columns that exist: its results are not stored
  auto first_col = [&](int i) { const int64_t c = c0 + 4 * i; return NEAR && c > cols - 4 ? cols - 4 : c; };
  const int64_t cl = first_col(i16), cb = first_col(0);      // cb <= cl: in a last strip of one to three columns the lanes start before c0
  int64_t cm[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) cm[m] = cl + m < cols ? cl + m : cols - 1;
  int jq[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) jq[t] = j0 + 16 * t + i16 < n ? j0 + 16 * t + i16 : n - 1;
  f32x4 acc[4][NT];
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[m][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  struct Operands { f32x4 a[kStep / 4]; float b[kStep / 4][NT]; };
  uint32_t go[kStep / 4], qo[kStep / 4][NT];            // byte offsets from the step's first row of G and of Q
#pragma unroll
  for (int s = 0; s < kStep / 4; ++s) {
    go[s] = (uint32_t)(4 * s + kg) * (uint32_t)ldg * 4u + (uint32_t)(cl - cb) * 4u;
#pragma unroll
    for (int t = 0; t < NT; ++t) qo[s][t] = ((uint32_t)(4 * s + kg) * (uint32_t)ldq + (uint32_t)jq[t]) * 4u;
  }
  auto fetch = [&](int64_t r0, Operands& o) {
    const float* gr = G + r0 * ldg + cb;
    const float* qr = Q + r0 * ldq;
#pragma unroll
    for (int s = 0; s < kStep / 4; ++s) {
      if (NEAR) o.a[s] = load4_at(gr, go[s]);
      else
#pragma unroll
        for (int m = 0; m < 4; ++m) o.a[s][m] = G[(r0 + 4 * s + kg) * ldg + cm[m]];
#pragma unroll
      for (int t = 0; t < NT; ++t) o.b[s][t] = NEAR ? load1_at(qr, qo[s][t]) : Q[(r0 + 4 * s + kg) * ldq + jq[t]];
    }
  };
  auto multiply = [&](const Operands& o) {
#pragma unroll
    for (int s = 0; s < kStep / 4; ++s)
#pragma unroll
      for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(o.a[s][m], o.b[s][t], acc[m][t], 0, 0, 0);
  };
  // Whole steps: the operands of the wave's next one travel while this one is multiplied (behind the last, it is read again).
  const int64_t r_full = r_begin + (r_end - r_begin) / kStep * kStep;
  int64_t r0 = r_begin + wave * kStep;
  const int steps = uniform(r0 < r_full ? (int)((r_full - r0 + kWaves * kStep - 1) / (kWaves * kStep)) : 0);
  if (steps > 0) {
    Operands o0, o1;
    auto step = [&](int i) { return r0 + (int64_t)(i < steps ? i : steps - 1) * (kWaves * kStep); };
    int i = 0;
    if (steps & 1) { fetch(r0, o0); multiply(o0); i = 1; }
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
    r0 += (int64_t)steps * (kWaves * kStep);
  }
  if (r0 == r_full && r_full < r_end) {                 // the rows left over: zeros past the end
    Operands o;
#pragma unroll
    for (int s = 0; s < kStep / 4; ++s) {
      const int64_t r = r0 + 4 * s + kg;
      const bool ok = r < r_end;
#pragma unroll
      for (int m = 0; m < 4; ++m) o.a[s][m] = ok ? G[r * ldg + cm[m]] : 0.f;
#pragma unroll
      for (int t = 0; t < NT; ++t) o.b[s][t] = ok ? Q[r * ldq + jq[t]] : 0.f;
    }
    multiply(o);
  }
  add_waves<NT>(acc, lds, wave, lane);
  if (wave != 0) return;
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t c = first_col(4 * kg + v) + m;
        const int j = j0 + 16 * t + i16;
        if (c >= c0 + 4 * (4 * kg + v) && c < cols && j < n) { float* o = T + c * ldt + j; *o = (accumulate ? *o : 0.f) + scale * acc[m][t][v]; }
      }
}

// Y[r][j] (+)= sum_c G[r][c] T[c][j], j < k <= 64: G [rows, cols], T [cols, k] (that of snapshot z at T + z t_snap), Y [rows, k].
// blockIdx.x: 64 rows, blockIdx.y = part of the sum: columns [part col_part, (part + 1) col_part), blockIdx.z = snapshot,
// result at Y + (snapshot gridDim.y + part) y_part.
// A lane's four consecutive columns of G are its terms of four matrix instructions: the step's terms are taken in the order
// c = 4 kg + s, which the rows of T are read in as well.
template <int NT, bool NEAR>
__global__ void __launch_bounds__(64 * kWaves, 2) g_t_kernel(CloudSnaps g, int64_t rows, int64_t cols, const float* __restrict__ T, int64_t t_snap, int k,
                                                          float* __restrict__ Y, int accumulate, int64_t col_part, int64_t y_part) {
  __shared__ __attribute__((aligned(16))) float lds[2 * 4 * NT * 256];
  const int lane = threadIdx.x & 63, wave = uniform((int)threadIdx.x >> 6), i16 = lane & 15, kg = lane >> 4;
  const float* G = g.G[blockIdx.z];
  T += blockIdx.z * t_snap;
  const int64_t c_begin = (int64_t)blockIdx.y * col_part;
  const int64_t c_end = cols < c_begin + col_part ? cols : c_begin + col_part;
  const int64_t r0 = (int64_t)blockIdx.x * kTile;
  Y += (int64_t)(blockIdx.z * gridDim.y + blockIdx.y) * y_part;
  int64_t rt[4];                                        // a row past the last repeats it: not stored
#pragma unroll
  for (int t = 0; t < 4; ++t) rt[t] = r0 + 16 * t + i16 < rows ? r0 + 16 * t + i16 : rows - 1;
  int jt[NT];
#pragma unroll
  for (int n = 0; n < NT; ++n) jt[n] = 16 * n + i16 < k ? 16 * n + i16 : k - 1;
  f32x4 acc[4][NT];
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int n = 0; n < NT; ++n) acc[t][n] = f32x4{0.f, 0.f, 0.f, 0.f};
  struct Operands { f32x4 a[4]; float b[4][NT]; };
  uint32_t go[4], to[4][NT];                            // byte offsets from the step's first column of G and row of T
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    go[t] = ((uint32_t)(rt[t] - r0) * (uint32_t)cols + 4u * kg) * 4u;
#pragma unroll
    for (int n = 0; n < NT; ++n) to[t][n] = (uint32_t)((4 * kg + t) * k + jt[n]) * 4u;
  }
  auto fetch = [&](int64_t c0, Operands& o) {
    const float* gr = G + r0 * cols + c0;
    const float* tr = T + c0 * k;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      if (NEAR) o.a[t] = load4_at(gr, go[t]);
      else
#pragma unroll
        for (int s = 0; s < 4; ++s) o.a[t][s] = G[rt[t] * cols + c0 + 4 * kg + s];
    }
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int n = 0; n < NT; ++n) o.b[s][n] = load1_at(tr, to[s][n]);
  };
  auto multiply = [&](const Operands& o) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int n = 0; n < NT; ++n) acc[t][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(o.a[t][s], o.b[s][n], acc[t][n], 0, 0, 0);
  };
  const int64_t c_full = c_begin + (c_end - c_begin) / kStep * kStep;
  int64_t c0 = c_begin + wave * kStep;
  const int steps = uniform(c0 < c_full ? (int)((c_full - c0 + kWaves * kStep - 1) / (kWaves * kStep)) : 0);
  if (steps > 0) {
    Operands o0, o1;
    auto step = [&](int i) { return c0 + (int64_t)(i < steps ? i : steps - 1) * (kWaves * kStep); };
    int i = 0;
    if (steps & 1) { fetch(c0, o0); multiply(o0); i = 1; }
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
    c0 += (int64_t)steps * (kWaves * kStep);
  }
  if (c0 == c_full && c_full < c_end) {
    Operands o;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int64_t c = c0 + 4 * kg + s;
      const bool ok = c < c_end;
#pragma unroll
      for (int t = 0; t < 4; ++t) o.a[t][s] = ok ? G[rt[t] * cols + c] : 0.f;
#pragma unroll
      for (int n = 0; n < NT; ++n) o.b[s][n] = ok ? T[c * k + jt[n]] : 0.f;
    }
    multiply(o);
  }
  add_waves<NT>(acc, lds, wave, lane);
  if (wave != 0) return;
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t r = r0 + 16 * t + 4 * kg + v;
        const int j = 16 * n + i16;
        if (r < rows && j < k) { float* y = Y + r * k + j; *y = (accumulate ? *y : 0.f) + acc[t][n][v]; }
      }
}

// In-place orthonormalisation of the k columns of Y [rows, k] (row stride k), in the order of the columns: Gram-Schmidt in its
// matrix form, Cholesky-QR, taken twice where the columns are the result and once where a sweep only needs their span.  One round is
//     W = Y^T Y        (one partial W per block of rows: gram_kernel)
//     W = L L^T        (sum_gram_kernel adds the partial W in their order, cholesky_kernel factorises: one workgroup)
//     Y <- Y L^-T      (fp64: apply_factor_kernel)
// Column j becomes y_j minus its projection on the earlier columns, divided by the norm that is left.  A column of which the earlier
// ones leave less than 1e-6 of its norm is stored as zeros and counted in *dependent.
// The pivot of column j is the square of what is left of it, a difference of sums c^2 times as large, c being the size of the
// coefficients with which the earlier columns make up y_j.  With columns that resemble each other c reaches 1e5 and more while each
// column still leaves 1e-3 of itself: in fp64 the difference is rounding then, and whole columns were taken for dependent (64
// overlapping bumps: 40 columns lost).  So the first round forms W and its pivots in pairs of doubles (106 bits: exact products of
// fp32 entries, two-term sums), which decides as the residuals themselves do up to c of 1e8.  At 8192 x 64 that costs 15 us instead of
// 10 for W and 40 instead of 25 for the factor.  The second round takes out what rounding of the coefficients and of Y to fp32 left of the earlier columns; its
// columns are orthonormal to a few per cent already, and fp64 is enough: the result is orthonormal to the rounding of its entries.
// The column-by-column form needs 3 k dependent sweeps over the rows, which one workgroup has to make: 33 ms for
// 8192 x 64, waiting for the L2 in every sweep.  This form reads the block twice per round, spread over all the rows'
// blocks, and what is serial (k pivots, one barrier each) stays inside one workgroup.
// Between sweeps the first round is enough: it fixes the span and which columns are dependent, and the next product takes columns that are orthonormal
// to a few per cent as well as better ones (8192 x 64, three sweeps: four second rounds of 53 us each became one, the whole basis 1000 us -> 847;
// the distance to an fp64 computation is the same over sizes, ranks and spectra decaying by up to 1e6).  Where a spectrum runs through the 1e-6 line rounding decides which of the
// columns next to it count as dependent, here as with two rounds: of 160 such bases 28 differ by a column or two from fp64's count either way, 8 from each other.  (Second rounds
// only where a column is left under 1e-4 agree in all 160, but cost 39 us of launches that leave at once, and let a later column decide on an earlier one's last bits.)
constexpr int kGramRows = 64;        // rows staged at a time
constexpr int kGramMaxParts = 128;   // partial W at most

// A number as the sum of two doubles, |lo| <= ulp(hi).  The operations follow Knuth's two-sum and the exact product by fma; nothing in them
// may be contracted or reordered.
struct Pair { double hi, lo; };
__device__ __forceinline__ Pair add_exact(double a, double b) {       // a + b = hi + lo
#pragma clang fp contract(off)
  const double s = a + b, t = s - a;
  return {s, (a - (s - t)) + (b - t)};
}
__device__ __forceinline__ Pair add_pair(Pair a, Pair b) {
#pragma clang fp contract(off)
  const Pair s = add_exact(a.hi, b.hi);
  const double lo = s.lo + (a.lo + b.lo), hi = s.hi + lo;
  return {hi, lo - (hi - s.hi)};
}
__device__ __forceinline__ Pair mul_pair(Pair a, Pair b) {
#pragma clang fp contract(off)
  const double p = a.hi * b.hi;
  return {p, __builtin_fma(a.lo, b.hi, __builtin_fma(a.hi, b.lo, __builtin_fma(a.hi, b.hi, -p)))};
}

// part[p][i k + j] = sum over the rows of part p of Y[r][i] Y[r][j], for every i >= j (16 x 16 tiles on and below the diagonal); with PAIRS
// the low halves follow in the part's next k^2 entries.
// Thread (tx, ty) holds element (16 a + ty, 16 b + tx) of each tile (a, b).  NT = ceil(k / 16) tiles.  With PAIRS the arithmetic is what bounds it (seven
// operations an entry and row), and the rows of tiles are shared between two blocks of equal work: blockIdx.y = 0 takes those of first_half.
template <int NT> constexpr bool first_half(int a) { return a == NT - 1 || (NT == 4 && a == 0); }
template <int NT, bool PAIRS>
__global__ void __launch_bounds__(256) gram_kernel(const float* __restrict__ Y, int64_t rows, int k, int64_t rows_per_part, double* __restrict__ part) {
  __shared__ float Ys[kGramRows][NT * 16 + 1];
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  const int64_t r_begin = (int64_t)blockIdx.x * rows_per_part;
  const int64_t r_end = rows < r_begin + rows_per_part ? rows : r_begin + rows_per_part;
  Pair acc[NT][NT];
#pragma unroll
  for (int a = 0; a < NT; ++a)
#pragma unroll
    for (int b = 0; b <= a; ++b) acc[a][b] = {0.0, 0.0};
  for (int64_t r0 = r_begin; r0 < r_end; r0 += kGramRows) {
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kGramRows * NT * 16 / 256; ++u) {
      const int i = tid + 256 * u, rr = i / (NT * 16), c = i % (NT * 16);
      Ys[rr][c] = (r0 + rr < r_end && c < k) ? Y[(r0 + rr) * k + c] : 0.f;
    }
    __syncthreads();
    auto add_rows = [&](auto half) {
#pragma unroll 2
      for (int rr = 0; rr < kGramRows; ++rr) {
        double yi[NT], yj[NT];
#pragma unroll
        for (int a = 0; a < NT; ++a) { yi[a] = (double)Ys[rr][16 * a + ty]; yj[a] = (double)Ys[rr][16 * a + tx]; }
#pragma unroll
        for (int a = 0; a < NT; ++a)
#pragma unroll
          for (int b = 0; b <= a; ++b) {
            if (PAIRS) {
#pragma clang fp contract(off)
              if (first_half<NT>(a) != decltype(half)::value) continue;
              const Pair s = add_exact(acc[a][b].hi, yi[a] * yj[b]);     // the product of two fp32 numbers is exact
              acc[a][b] = {s.hi, acc[a][b].lo + s.lo};
            } else {
              acc[a][b].hi = __builtin_fma(yi[a], yj[b], acc[a][b].hi);
            }
          }
      }
    };
    if (PAIRS && blockIdx.y) add_rows(std::false_type{}); else add_rows(std::true_type{});
  }
  const int n = k * k;
  double* out = part + (int64_t)blockIdx.x * n * (PAIRS ? 2 : 1);
#pragma unroll
  for (int a = 0; a < NT; ++a)
#pragma unroll
    for (int b = 0; b <= a; ++b) {
      const int i = 16 * a + ty, j = 16 * b + tx;
      const bool here = !PAIRS || first_half<NT>(a) == (blockIdx.y == 0);
      if (here && i < k && j <= i) { out[i * k + j] = acc[a][b].hi; if (PAIRS) out[n + i * k + j] = acc[a][b].lo; }
    }
}

// W[e] = sum over p of part[p][e] (n entries each, or n high and n low halves): 64 entries per block, four threads per entry, each
// adding a quarter of the parts in order.
template <bool PAIRS>
__global__ void __launch_bounds__(256) sum_gram_kernel(const double* __restrict__ part, int n_parts, int n, double* __restrict__ W) {
  __shared__ double sums[PAIRS ? 2 : 1][4][64];
  const int i64 = threadIdx.x & 63, e = blockIdx.x * 64 + i64, q = threadIdx.x >> 6, per = (n_parts + 3) / 4;
  const int64_t stride = (int64_t)n * (PAIRS ? 2 : 1);
  Pair v{0.0, 0.0};
  if (e < n) {
    const int end = n_parts < (q + 1) * per ? n_parts : (q + 1) * per;
#pragma unroll 8
    for (int p = q * per; p < end; ++p) {
      if (PAIRS) v = add_pair(v, {part[p * stride + e], part[p * stride + n + e]});
      else v.hi += part[p * stride + e];
    }
  }
  sums[0][q][i64] = v.hi;
  if (PAIRS) sums[PAIRS ? 1 : 0][q][i64] = v.lo;
  __syncthreads();
  if (q != 0 || e >= n) return;
  if (PAIRS) {
    auto of = [&](int i) { return Pair{sums[0][i][i64], sums[PAIRS ? 1 : 0][i][i64]}; };
    v = add_pair(add_pair(of(0), of(1)), add_pair(of(2), of(3)));
    W[e] = v.hi;
    W[n + e] = v.lo;
  } else {
    W[e] = (sums[0][0][i64] + sums[0][1][i64]) + (sums[0][2][i64] + sums[0][3][i64]);
  }
}

// Factorises W [k][k] (its lower triangle is read) and inverts the factor: fac[i k + j] = (L^-1)_ji for i <= j, 0 otherwise and for
// a dependent column j.  W = U D U^T with U unit lower triangular; X = U^-1 grows row by row under the same eliminations.
// Thread (tx, ty) keeps the entries (16 a + ty, 16 b + tx) of what is left of W in registers (W in pairs when PAIRS, X in fp64: the second round
// takes up what that rounds), those of the tiles a pivot still reaches being updated; the pivot's column and X's row go round through
// LDS, one barrier per pivot.
// What bounds it is that chain of k barriers, LDS reads and reciprocals (0.4 us each at k = 64, 0.6 with pairs).
template <int NT, bool PAIRS>
__global__ void __launch_bounds__(256) cholesky_kernel(const double* __restrict__ W, int k, double* __restrict__ fac, int* __restrict__ dependent) {
  __shared__ double col[2][PAIRS ? 2 : 1][NT * 16], row[2][NT * 16], pivots[NT * 16], norm0[NT * 16], inv[NT * 16];
  __shared__ int n_dep;
  constexpr int LO = PAIRS ? 1 : 0;
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  Pair w[NT][NT];
  double x[NT][NT];
#pragma unroll
  for (int a = 0; a < NT; ++a)
#pragma unroll
    for (int b = 0; b < NT; ++b) {
      const int i = 16 * a + ty, j = 16 * b + tx, e = i >= j ? i * k + j : j * k + i;
      const bool inside = i < k && j < k;
      x[a][b] = i == j ? 1.0 : 0.0;
      w[a][b] = {inside ? W[e] : 0.0, PAIRS && inside ? W[k * k + e] : 0.0};
      if (i == j) norm0[j] = w[a][b].hi;              // the column's size before anything is taken out
    }
  if (tid == 0) n_dep = 0;
#pragma unroll
  for (int b = 0; b < NT; ++b)
    for (int jj = 0; jj < 16; ++jj) {
      const int j = 16 * b + jj;
      if (j >= k) break;                              // uniform
      if (tx == jj)
#pragma unroll
        for (int a = b; a < NT; ++a) { col[j & 1][0][16 * a + ty] = w[a][b].hi; if (PAIRS) col[j & 1][LO][16 * a + ty] = w[a][b].lo; }
      if (ty == jj)
#pragma unroll
        for (int c = 0; c <= b; ++c) row[j & 1][16 * c + tx] = x[b][c];
      __syncthreads();
      auto col_at = [&](int i) { return Pair{col[j & 1][0][i], PAIRS ? col[j & 1][LO][i] : 0.0}; };
      const Pair pivot = col_at(j);
      const bool dep = !(pivot.hi > 1e-12 * norm0[j]) || !(pivot.hi > 0.0);
      if (tid == 0) pivots[j] = dep ? 0.0 : pivot.hi;
      Pair ip{__builtin_amdgcn_rcp(pivot.hi), 0.0};   // two Newton steps take the estimate to fp64 rounding, a third gives the low half
      ip.hi = __builtin_fma(__builtin_fma(-pivot.hi, ip.hi, 1.0), ip.hi, ip.hi);
      ip.hi = __builtin_fma(__builtin_fma(-pivot.hi, ip.hi, 1.0), ip.hi, ip.hi);
      if (PAIRS) ip.lo = __builtin_fma(-pivot.lo, ip.hi, __builtin_fma(-pivot.hi, ip.hi, 1.0)) * ip.hi;
      if (dep) ip = {0.0, 0.0};
      Pair g[NT];
      double h[NT];
#pragma unroll
      for (int c = b; c < NT; ++c) g[c] = col_at(16 * c + tx);
#pragma unroll
      for (int c = 0; c <= b; ++c) h[c] = row[j & 1][16 * c + tx];
#pragma unroll
      for (int a = b; a < NT; ++a) {
        if (a == b && ty <= jj) continue;             // rows up to the pivot's are finished (and a factor of zero would not spare them a NaN)
        Pair f = col_at(16 * a + ty);
        if (PAIRS) f = mul_pair({-f.hi, -f.lo}, ip); else f.hi = -f.hi * ip.hi;
#pragma unroll
        for (int c = b; c <= a; ++c) {                // on and below the diagonal: nothing above it is read
          if (PAIRS) w[a][c] = add_pair(w[a][c], mul_pair(f, g[c]));
          else w[a][c].hi = __builtin_fma(f.hi, g[c].hi, w[a][c].hi);
        }
#pragma unroll
        for (int c = 0; c <= b; ++c) x[a][c] = __builtin_fma(f.hi, h[c], x[a][c]);
      }
    }
  __syncthreads();
  if (tid < k) {
    inv[tid] = pivots[tid] > 0.0 ? 1.0 / sqrt(pivots[tid]) : 0.0;
    if (!(pivots[tid] > 0.0)) atomicAdd(&n_dep, 1);
  }
  __syncthreads();
#pragma unroll
  for (int a = 0; a < NT; ++a)
#pragma unroll
    for (int b = 0; b < NT; ++b) {
      const int j = 16 * a + ty, i = 16 * b + tx;
      if (i < k && j < k) fac[i * k + j] = i <= j ? x[a][b] * inv[j] : 0.0;
    }
  if (tid == 0) *dependent = n_dep;
}

// Y <- Y fac: row q_j = sum_{i<=j} y_i fac[i][j] in fp64, 32 rows per block; thread (tx, ty) holds rows ty, 16 + ty and columns 16 b + tx.
// (Forward substitution with a row per lane, everything unrolled, took 45 us at 8192 x 64: 30 KB of code fetched once.)
constexpr int kApplyRows = 32;
template <int NT>
__global__ void __launch_bounds__(256) apply_factor_kernel(float* __restrict__ Y, int64_t rows, int k, const double* __restrict__ fac) {
  constexpr int KP = NT * 16;
  __shared__ double F[KP][KP];
  __shared__ float Ys[kApplyRows][KP + 1];
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  const int64_t r0 = (int64_t)blockIdx.x * kApplyRows;
#pragma unroll
  for (int u = 0; u < KP * KP / 256; ++u) { const int e = tid + 256 * u, i = e / KP, j = e % KP; F[i][j] = (i < k && j < k) ? fac[i * k + j] : 0.0; }
#pragma unroll
  for (int u = 0; u < kApplyRows * KP / 256; ++u) { const int e = tid + 256 * u, r = e / KP, c = e % KP; Ys[r][c] = (r0 + r < rows && c < k) ? Y[(r0 + r) * k + c] : 0.f; }
  __syncthreads();
  double acc[2][NT];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < NT; ++b) acc[a][b] = 0.0;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll 4
    for (int i = 16 * t; i < 16 * t + 16; ++i) {
      const double y0 = (double)Ys[ty][i], y1 = (double)Ys[16 + ty][i];
      // in the tile on the diagonal the factor's zeros are skipped: a later column that is not finite must not reach an earlier one
      const bool up = i <= 16 * t + tx;
#pragma unroll
      for (int b = t; b < NT; ++b) {
        const double f = F[i][16 * b + tx];
        acc[0][b] = __builtin_fma(b > t || up ? y0 : 0.0, f, acc[0][b]);
        acc[1][b] = __builtin_fma(b > t || up ? y1 : 0.0, f, acc[1][b]);
      }
    }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < NT; ++b) {
      const int64_t r = r0 + 16 * a + ty;
      const int j = 16 * b + tx;
      if (r < rows && j < k) Y[r * k + j] = (float)acc[a][b];
    }
}

// out[i] = (accumulate ? out[i] : 0) + part[0][i] + part[1][i] + ...: the parts of a split sum, added in their order.
// blockIdx.y = y: parts y n_parts ... of the buffer into out + y n.
__global__ void __launch_bounds__(256) sum_parts_kernel(const float* __restrict__ part, int n_parts, int64_t n, float* __restrict__ out, int accumulate) {
  part += (int64_t)blockIdx.y * n_parts * n;
  out += (int64_t)blockIdx.y * n;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    float v = 0.f;
#pragma unroll 4
    for (int z = 0; z < n_parts; ++z) v += part[(int64_t)z * n + i];
    out[i] = (accumulate ? out[i] : 0.f) + v;
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

// How many parts to split a sum over `span` terms into when `blocks` blocks take it undivided: three blocks per CU, which is
// what the kernels' registers admit (G^T Q of three 8192 x 2048 snapshots at rank 64: 63 us with 768 blocks, 88 with 384), each part
// at least two steps per wave, at most max_parts.
static int cloud_sum_parts(int64_t blocks, int64_t span, int64_t max_parts) {
  int64_t z = blocks > 0 ? 768 / blocks : 1;
  const int64_t longest = span / (2 * kWaves * kStep);
  if (z > longest) z = longest;
  if (z > max_parts) z = max_parts;
  return z < 1 ? 1 : (int)z;
}

static hipError_t launch_sum_parts(const float* part, int n_parts, int64_t n, int n_out, float* out, int accumulate, hipStream_t s) {
  hipLaunchKernelGGL(sum_parts_kernel, dim3((unsigned)(n / 256 + 1 < 1024 ? n / 256 + 1 : 1024), (unsigned)n_out), dim3(256), 0, s, part, n_parts, n, out, accumulate);
  return hipGetLastError();
}

// Whether the byte offsets within a step fit 32 bits (64 rows or 16, of at most `ld` floats) and a row holds the four columns a lane loads.
static bool near_rows(int64_t cols, int64_t ld) { return cols >= 4 && ld < ((int64_t)1 << 24); }

static int column_tiles(int n) { return n >= kTile ? 4 : (n + 15) / 16; }

// The variant of a product kernel for NT = nt column tiles.
#define ZGR_CLOUD_LAUNCH(KERNEL, nt, near, grid, ...)                                                                                                \
  switch ((nt) * 2 + ((near) ? 1 : 0)) {                                                                                                             \
    case 2: hipLaunchKernelGGL((KERNEL<1, false>), grid, dim3(64 * kWaves), 0, __VA_ARGS__); break;                                                  \
    case 3: hipLaunchKernelGGL((KERNEL<1, true>), grid, dim3(64 * kWaves), 0, __VA_ARGS__); break;                                                   \
    case 4: hipLaunchKernelGGL((KERNEL<2, false>), grid, dim3(64 * kWaves), 0, __VA_ARGS__); break;                                                  \
    case 5: hipLaunchKernelGGL((KERNEL<2, true>), grid, dim3(64 * kWaves), 0, __VA_ARGS__); break;                                                   \
    case 6: hipLaunchKernelGGL((KERNEL<3, false>), grid, dim3(64 * kWaves), 0, __VA_ARGS__); break;                                                  \
    case 7: hipLaunchKernelGGL((KERNEL<3, true>), grid, dim3(64 * kWaves), 0, __VA_ARGS__); break;                                                   \
    case 8: hipLaunchKernelGGL((KERNEL<4, false>), grid, dim3(64 * kWaves), 0, __VA_ARGS__); break;                                                  \
    default: hipLaunchKernelGGL((KERNEL<4, true>), grid, dim3(64 * kWaves), 0, __VA_ARGS__); break;                                                  \
  }

hipError_t launch_cloud_gt_q(const float* G, int64_t rows, int64_t cols, int64_t ldg, const float* Q, int n, int64_t ldq, float* T, int64_t ldt, float scale,
                             int accumulate, hipStream_t s) {
  const CloudSnaps g{{G}};
  const int nt = column_tiles(n);
  const dim3 grid((unsigned)((cols + kTile - 1) / kTile), (unsigned)((n + 16 * nt - 1) / (16 * nt)), 1);
  ZGR_CLOUD_LAUNCH(gt_q_kernel, nt, near_rows(cols, ldg > ldq ? ldg : ldq), grid, s, g, 0, rows, cols, ldg, Q, n, ldq, T, ldt, scale, accumulate, rows, (int64_t)0)
  return hipGetLastError();
}

hipError_t launch_cloud_gt_q_all(const CloudSnaps& g, int n_snap, int64_t rows, int64_t cols, const float* Q, int k, float* T, float* part, int64_t part_floats, hipStream_t s) {
  const int nt = column_tiles(k);
  const int64_t strips = (cols + kTile - 1) / kTile, n = cols * k;
  const int z = cloud_sum_parts(strips * n_snap, rows, part_floats / n / n_snap);
  const int64_t steps = (rows + kStep - 1) / kStep, row_part = (steps + z - 1) / z * kStep;
  const dim3 grid((unsigned)strips, (unsigned)n_snap, (unsigned)z);
  ZGR_CLOUD_LAUNCH(gt_q_kernel, nt, near_rows(cols, cols), grid, s, g, 1, rows, cols, cols, Q, k, (int64_t)k, z > 1 ? part : T, (int64_t)k, 1.0f, 0, row_part, n)
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || z == 1) return e;
  return launch_sum_parts(part, z, n, n_snap, T, 0, s);
}

hipError_t launch_cloud_g_t_all(const CloudSnaps& g, int n_snap, int64_t rows, int64_t cols, const float* T, int64_t t_snap, int k, float* Y, int accumulate, float* part, int64_t part_floats,
                                hipStream_t s) {
  const int nt = column_tiles(k);
  const int64_t strips = (rows + kTile - 1) / kTile, n = rows * k;
  const int z = cloud_sum_parts(strips * n_snap, cols, part_floats / n / n_snap);
  const int64_t steps = (cols + kStep - 1) / kStep, col_part = (steps + z - 1) / z * kStep;
  const bool whole = n_snap * z == 1;
  const dim3 grid((unsigned)strips, (unsigned)z, (unsigned)n_snap);
  ZGR_CLOUD_LAUNCH(g_t_kernel, nt, near_rows(cols, cols), grid, s, g, rows, cols, T, t_snap, k, whole ? Y : part, whole ? accumulate : 0, col_part, n)
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || whole) return e;
  return launch_sum_parts(part, n_snap * z, n, 1, Y, accumulate, s);
}
#undef ZGR_CLOUD_LAUNCH

template <int NT, bool PAIRS>
static hipError_t orth_round(float* Y, int64_t rows, int k, int* dependent, double* scratch, hipStream_t s) {
  const int64_t chunks = (rows + kGramRows - 1) / kGramRows;
  const int64_t per = (chunks + kGramMaxParts - 1) / kGramMaxParts, parts = (chunks + per - 1) / per;
  const int n = k * k;
  constexpr int halves = PAIRS ? 2 : 1;
  double* W = scratch + parts * n * halves;
  double* fac = W + n * halves;
  hipLaunchKernelGGL((gram_kernel<NT, PAIRS>), dim3((unsigned)parts, PAIRS && NT > 1 ? 2 : 1), dim3(256), 0, s, Y, rows, k, per * kGramRows, scratch);
  hipLaunchKernelGGL(sum_gram_kernel<PAIRS>, dim3((unsigned)((n + 63) / 64)), dim3(256), 0, s, scratch, (int)parts, n, W);
  hipLaunchKernelGGL((cholesky_kernel<NT, PAIRS>), dim3(1), dim3(256), 0, s, W, k, fac, dependent);
  hipLaunchKernelGGL(apply_factor_kernel<NT>, dim3((unsigned)((rows + kApplyRows - 1) / kApplyRows)), dim3(256), 0, s, Y, rows, k, fac);
  return hipGetLastError();
}

template <int NT>
static hipError_t orth(float* Y, int64_t rows, int k, bool last, int* dependent, double* scratch, hipStream_t s) {
  const hipError_t e = orth_round<NT, true>(Y, rows, k, dependent, scratch, s);
  if (k == 1 || !last) return e;                                // one column has nothing left of earlier ones to take out (16 x 16, one sweep: 97 us a call, 118 with a second round)
  return e != hipSuccess ? e : orth_round<NT, false>(Y, rows, k, dependent, scratch, s);      // its count includes the first round's zero columns
}

hipError_t launch_cloud_orth(float* Y, int64_t rows, int k, bool last, int* dependent, double* scratch, hipStream_t s) {
  switch ((k + 15) / 16) {
    case 1:  return orth<1>(Y, rows, k, last, dependent, scratch, s);
    case 2:  return orth<2>(Y, rows, k, last, dependent, scratch, s);
    case 3:  return orth<3>(Y, rows, k, last, dependent, scratch, s);
    default: return orth<4>(Y, rows, k, last, dependent, scratch, s);
  }
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
