// Host-callable launchers of the backward-pass kernels (backward.hip): the cloud block of Algorithm 1.
// dtype / b_dtype: 0 = fp32 storage, 1 = bf16 storage.  All pointers are device memory; gradients are fp32.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace zgr {

constexpr int kBackwardMaxSeq = 2048;      // keys one wave of the attention rule holds

// bf16 operands for the matrix-core products: out [cols, rows] (row stride ld_out, a multiple of 64) = in [rows, cols]^T in bf16 (row
// stride ld_in, a multiple of 4), zeros between rows and ld_out
hipError_t launch_bw_transpose_bf16(const void* in, int rows, int cols, int64_t ld_in, void* out, int64_t ld_out, hipStream_t s);
// a gradient dy [M, N] (both multiples of 64) as both operands, cols_out [N, M] and rows_out [M, N] in bf16, and its column sums: dbias[i] gets
// those of the i-th of n_bias equal column blocks.  With u != NULL it is dy act'(u) that is taken.
hipError_t launch_bw_gradient_operands(const float* dy, const float* u, int relu, int M, int N, void* cols_out, void* rows_out, float* const* dbias, int n_bias, float* part, hipStream_t s);
// `part` of the column sums and of the LayerNorm rule: scratch of bw_scratch_floats(d, widest N) floats
size_t     bw_scratch_floats(int d, int n_widest);
hipError_t launch_bw_fill(float* p, int64_t n, float v, hipStream_t s);
// row_loss of logits [rows, n] (0 where the target is negative), and (softmax - onehot(target)) inv_count in place of the logits or, with d16,
// in bf16 at d16 [rows, ld16] with zeros past n; rows with a target outside [0, n) become zeros
hipError_t launch_bw_cross_entropy(float* logits, const int32_t* targets, int rows, int n, float inv_count, float* row_loss, void* d16, int64_t ld16, hipStream_t s);
// y = LayerNorm(x) g + b: dx_out = (add ? add : 0) + dL/dx (dx_out may be add or dy), dg, db from dy; stats: 2 M floats of scratch
hipError_t launch_bw_layernorm(int dtype, const float* x, const void* g, const float* dy, const float* add, float* dx_out, float* stats, float* dg, float* db,
                               float* part, int M, int d, float eps, hipStream_t s);
// f = act(u) in the storage type (erf-GELU, or ReLU when relu != 0); df <- df act'(u); dst += src
hipError_t launch_bw_act_forward(int dtype, int relu, const float* u, void* f, int64_t n, hipStream_t s);
hipError_t launch_bw_act(int relu, const float* u, float* df, int64_t n, hipStream_t s);
hipError_t launch_bw_add(float* dst, const float* src, int64_t n, hipStream_t s);
// dqkv [B T, 3 d] from dctx [B T, d]; scratch: P of 3 B n_head floats for T rounded up to a multiple of 32, or, where the rule needs [T, T] buffers (heads of 8), P and dS of B n_head T T
// floats each
bool       bw_attention_buffers(int d, int n_head);
hipError_t launch_bw_attention(int dtype, const void* qkv, const float* dctx, const int32_t* lengths, int batch, int seq, int d, int n_head, int causal,
                               float* P, float* dS, float* dqkv, hipStream_t s);
// dE [vocab, d] += rows of dx by token, dPe [max_pos, d] = sums of dx by position
hipError_t launch_bw_embedding(const int32_t* tok, const float* dx, int M, int seq, int d, int vocab, float* dE, float* dPe, int max_pos, hipStream_t s);

}  // namespace zgr
