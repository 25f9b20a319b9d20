// Matrix products with fp32 accumulation on operands as they lie in memory (product.hip): the fp32 and the
// odd-sized products of the cloud's backward pass, and the small projections of fp32 models.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace zgr {

// C[i][j] = epilogue(alpha sum_k A[i][k] B[k][j] + bias[j]) for every batch z: operand X of batch z starts at X + (z / zdiv) x_outer + (z % zdiv) x_inner elements.
// An operand is fp32 or bf16 (dtype 0 / 1) and contiguous along k or along its other index; ld is the stride of the one that is not.
struct ProductArgs {
  const void* A = nullptr; int a_dtype = 0; bool a_k = true; int64_t lda = 0;       // a_k: A[i][k] at A + i lda + k, else A + k lda + i
  const void* B = nullptr; int b_dtype = 0; bool b_k = true; int64_t ldb = 0;       // b_k: B[k][j] at B + j ldb + k, else B + k ldb + j
  float* C = nullptr; int64_t ldc = 0;
  int M = 0, N = 0, K = 0;
  float alpha = 1.0f;
  int epilogue = 0;                 // forward.h: EPI_STORE (or EPI_F32), EPI_GELU, EPI_RELU, EPI_RESID (C += ...)
  const float* bias = nullptr;      // fp32 [N], may be NULL; bias_outer floats further on for each next batch (per outer step)
  int64_t bias_outer = 0;
  float* a_sums = nullptr;          // when not NULL: a_sums[i] = sum_k A[i][k] (fp32 A contiguous along i, one batch)
  int batches = 1, zdiv = 1;
  int64_t a_outer = 0, a_inner = 0, b_outer = 0, b_inner = 0, c_outer = 0, c_inner = 0;
  int models = 1;                   // the batches are those of that many models on the same inputs; each one's sums take the order they take by themselves
  int row_blocks = 1;               // M is that many equal blocks of rows; each one's sums take the order they take in a product of its own
  float* scratch = nullptr; size_t scratch_floats = 0;    // for the parts of a split sum; without it sums are split inside workgroups only
  int* parts_left = nullptr;        // when not NULL (one batch, EPI_STORE, alpha = 1, no bias): a sum in several parts is left to the reader, who adds parts of M N floats
                                    // each from scratch on, in their order: *parts_left of them, or 1, and C holds the result
};
hipError_t launch_product(const ProductArgs& p, hipStream_t s);

}  // namespace zgr
