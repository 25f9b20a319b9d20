// Host-callable launchers of the forward-pass kernels (forward.hip).
// dtype: 0 = fp32 storage, 1 = bf16 storage.  All pointers are device memory.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace zgr {

enum { EPI_STORE = 0, EPI_GELU = 1, EPI_RESID = 2, EPI_F32 = 3, EPI_CE = 4, EPI_RELU = 5 };

// Two models on the same batch in one launch (the two loss evaluations of a step): the second's parameters lie w bytes behind the first's, and
// in every activation and loss its rows follow the first's; its row losses start row_loss floats behind the first's.  M and batch below count one model's rows.  Half the launches, each with twice the blocks: steps of
// 125M parameters 3.21 -> 2.45 ms (with the tiles' order below), in fp32 4.46 -> 3.56 (kernels chosen by both models' tiles, as they no longer are), of 350M 9.07 -> 7.83, of 1.3B 26.1 -> 24.4, of a small decoder 245 -> 164 us.
// Every result has the bits that one model's launch gives it: whatever decides the order of a sum looks at one model's sizes.  (bf16 tiles, all of which take the terms in the
// same order, are chosen by the tiles of both.)
struct Twin { int models = 1; int64_t w = 0; int64_t row_loss = 0; };

// targets (may be NULL): the next token of each of the M rows, -1 at the end of a sequence
hipError_t launch_embed(int dtype, const int32_t* tok, const void* E, const void* Pe, float* x, int M, int seq, int d, int vocab, int32_t* targets, hipStream_t s, Twin tw = {});
// out (storage type) = LayerNorm(x) g + b; xout, when not NULL, receives the same values in fp32 (it may be x itself)
hipError_t launch_layernorm(int dtype, const float* x, const void* g, const void* b, void* out, int M, int d, float eps, hipStream_t s, float* xout = nullptr, Twin tw = {});
// keep_order (launch_gemm, launch_attention): sums in the order in which the large tiles, and attention key by key, take them at every size.
// The forward half of the cloud's backward pass asks for it: a ReLU's slope jumps where its argument changes sign, so sums taken in
// another order there move the gradients of bf16 ReLU models by far more than their rounding (4e-3 of their norm on a 13-block model with head
// size 32), while a loss, which is all the client's forward returns, follows smoothly.  Neither order is the more accurate one: what this keeps is
// that gradients stay as they were.  It is asked for with every model, though fp32 and GELU models have no such jump.
// out = epilogue(A[M,K] W[N,K]^T + bias); bf16 storage needs K % 64 == 0.  scratch (may be NULL): floats a split sum may be kept in meanwhile.
// shared_a: both models read the same A.  resid: what EPI_RESID adds to, where that is not out itself (sums in the order of the tiles then).
hipError_t launch_gemm(int dtype, const void* A, const void* W, const void* bias, void* out, int epi, int M, int N, int K, hipStream_t s, float* scratch = nullptr,
                       size_t scratch_floats = 0, bool keep_order = false, Twin tw = {}, bool shared_a = false, const float* resid = nullptr);
// Several bf16 products out = A W^T in one launch, out [M, N] in fp32, A's rows of K and W's of K / fold terms, lda and ldw entries apart.  fold = 3: A's rows hold three runs (the
// planes of fp32 numbers, planes.h), each of which is multiplied with W's row.  K a multiple of 64 fold, rows on 16 bytes.
constexpr int kGroupedProducts = 6;
struct GroupedProduct { const void* A; const void* W; float* out; int M, N, K, lda, ldw; };
struct ProductGroup { GroupedProduct job[kGroupedProducts]; int count = 0, fold = 1; };
hipError_t launch_product_group(const ProductGroup& g, hipStream_t s);
// One such product with its sum in slices, which leave parts of M N floats one behind the other for the reader to add up in their order; as many of them as pay, at most `most`.
int        product_slices(int M, int N, int K, int most);
hipError_t launch_product_slices(const void* A, const void* W, float* out, int M, int N, int K, int slices, hipStream_t s);
// The kernel of an fp32 projection (zgr.h, zgr_debug_gemm_form).  whole_rows: K % 4 == 0 and 16-byte aligned operands.
enum { F32_PLANES_128 = 0, F32_PLANES_64 = 1, F32_TILES_128 = 2, F32_TILES_64 = 3, F32_PRODUCT = 4, F32_VECTOR = 5 };
int        fp32_projection_form(int M, int N, int K, bool whole_rows, bool keep_order);
// bf16 vocabulary projection fused with cross-entropy: row_loss[m] = logsumexp(A[m] W^T) - (A[m] W^T)[targets[m]] (0 where targets[m] < 0).
int        ce_partials_per_row(int N);
hipError_t launch_gemm_ce_bf16(const void* A, const void* W, const int32_t* targets, void* part, float* tlogit, float* row_loss, int M, int N, int K, hipStream_t s, Twin tw = {});
hipError_t launch_attention(int dtype, const void* qkv, void* ctx, const int32_t* lengths, int batch, int seq, int d, int n_head, int causal, hipStream_t s,
                            bool keep_order = false, int models = 1);
bool       attention_head_dim_supported(int dh);
hipError_t launch_ce_rows(const float* logits, const int32_t* targets, float* row_loss, int M, int n, hipStream_t s, Twin tw = {});
hipError_t launch_mean_f64(const float* row_loss, int n, double inv_count, double* out, hipStream_t s, Twin tw = {});
hipError_t launch_cls_head(int dtype, const void* h, const void* Wc, const void* bc, float* logits, int batch, int seq, int d, int n_class, hipStream_t s, Twin tw = {});
// row losses and, at out (one per model), their mean
bool       lsq_in_one_block(int batch, int n_out);
hipError_t launch_lsq_loss(const float* pred, const float* Y, float* row_loss, int batch, int n_out, double* out, hipStream_t s, Twin tw = {});

}  // namespace zgr
