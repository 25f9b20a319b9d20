// Host-callable launchers of the backward-pass kernels (backward.hip): the cloud block of Algorithm 1.
// dtype / b_dtype: 0 = fp32 storage, 1 = bf16 storage.  All pointers are device memory; gradients are fp32.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace zgr {

constexpr int kBackwardMaxSeq = 2048;      // keys one wave of the attention rule holds

// Sums over rows (bias and LayerNorm gradients) run in two stages: their kernels leave chunk sums in an arena, and one launch adds up those of
// many, a row of blocks each (one launch per sum: 73 of 3.9 us in the backward pass of a 12-block decoder).  flush() before the results are read.
constexpr int kSumJobs = 64;
struct SumJob { const float* part; float* out; int64_t stride; int parts, n; };      // out[c] = sum over p of part[p stride + c], c < n
struct SumJobs { SumJob job[kSumJobs]; };
class SumQueue {
 public:
  SumQueue(float* arena, size_t floats, hipStream_t s) : arena_(arena), floats_(floats), s_(s) {}
  hipError_t take(size_t floats, int n_jobs, float** part);      // room for the chunk sums of the next n_jobs sums
  void add(const SumJob& j) { if (j.n > widest_) widest_ = j.n; jobs_.job[count_++] = j; }
  hipError_t flush();
 private:
  float* arena_; size_t floats_, used_ = 0;
  hipStream_t s_;
  SumJobs jobs_{};
  int count_ = 0, widest_ = 0;
};

// bf16 operands for the matrix-core products: out [cols, rows] (row stride ld_out, a multiple of 64) = in [rows, cols]^T in bf16 (row
// stride ld_in, a multiple of 4), zeros between rows and ld_out
hipError_t launch_bw_transpose_bf16(const void* in, int rows, int cols, int64_t ld_in, void* out, int64_t ld_out, hipStream_t s);
// several whole matrices at once, in [rows, cols] and out [cols, rows] (rows and cols multiples of 64)
constexpr int kTransposeJobs = 8;
struct TransposeJob { const void* in; void* out; int rows, cols; };
struct TransposeJobs { TransposeJob job[kTransposeJobs]; int count = 0; };
hipError_t launch_bw_transposes_bf16(const TransposeJobs& jobs, hipStream_t s);
// a gradient dy [M, N] (both multiples of 64) as both operands, cols_out [N, M] and rows_out [M, N] in bf16, and its column sums: dbias[i] gets
// those of the i-th of n_bias equal column blocks.  With u != NULL it is dy act'(u) that is taken.
hipError_t launch_bw_gradient_operands(const float* dy, const float* u, int relu, int M, int N, void* cols_out, void* rows_out, float* const* dbias, int n_bias, SumQueue& sums, hipStream_t s);
// A gradient dy [M, N] in fp32 (any M, N a multiple of 64) as the first operand of a product group with fold = 3, cols_out [N, 3 x M rounded up to a multiple
// of 64], and its column sums as above.  With u != NULL dy <- dy act'(u) first.  The second operand as well: x [M, x_cols] in bf16, x_out [x_cols, M rounded up].
hipError_t launch_bw_gradient_planes(float* dy, const float* u, int relu, int M, int N, void* cols_out, const void* x, int x_cols, void* x_out, float* const* dbias, int n_bias, SumQueue& sums,
                                     hipStream_t s);
// the largest room one column sum or LayerNorm rule takes of the arena, floats
size_t     bw_scratch_floats(int d, int n_widest);
size_t     bw_layernorm_floats(int M, int d);      // chunk sums that launch_bw_layernorm takes from the queue, and what launch_bw_gradient_operands takes for n columns in
size_t     bw_bias_floats(int M, int n);           // up to four calls
hipError_t launch_bw_fill(float* p, int64_t n, float v, hipStream_t s);
// row_loss of logits [rows, n] (0 where the target is negative), and (softmax - onehot(target)) inv_count in place of the logits or, with d16,
// in bf16 at d16 [rows, ld16] with zeros past n; rows with a target outside [0, n) become zeros
hipError_t launch_bw_cross_entropy(float* logits, const int32_t* targets, int rows, int n, float inv_count, float* row_loss, void* d16, int64_t ld16, hipStream_t s);
// y = LayerNorm(x) g + b: dx_out = (add ? add : 0) + dL/dx (dx_out may be add or dy), dg, db from dy; stats: 2 M floats of scratch.  dy: the sum of dy_parts parts of M d
// floats each, one behind the other (more than one where bw_layernorm_adds_parts).
bool       bw_layernorm_adds_parts(int d);
hipError_t launch_bw_layernorm(int dtype, const float* x, const void* g, const float* dy, const float* add, float* dx_out, float* stats, float* dg, float* db,
                               SumQueue& sums, int M, int d, float eps, hipStream_t s, int dy_parts = 1);
// f = act(u) in the storage type (erf-GELU, or ReLU when relu != 0); df <- df act'(u); dst += src
hipError_t launch_bw_act_forward(int dtype, int relu, const float* u, void* f, int64_t n, hipStream_t s);
hipError_t launch_bw_act(int relu, const float* u, float* df, int64_t n, hipStream_t s);
hipError_t launch_bw_add(float* dst, const float* src, int64_t n, hipStream_t s);
// dqkv [B T, 3 d] from dctx [B T, d]; scratch: bw_attention_scratch floats, which grow with batch and with seq
size_t     bw_attention_scratch(int dtype, int d, int n_head, int batch, int seq, int causal);
hipError_t launch_bw_attention(int dtype, const void* qkv, const float* dctx, const int32_t* lengths, int batch, int seq, int d, int n_head, int causal,
                               float* scratch, float* dqkv, hipStream_t s);
// dE [vocab, d] += rows of dx by token, dPe [max_pos, d] = sums of dx by position
hipError_t launch_bw_embedding(const int32_t* tok, const float* dx, int M, int seq, int d, int vocab, float* dE, float* dPe, int max_pos, hipStream_t s);

}  // namespace zgr
