/* Entry points of libqdelta.so that only the autograd layer
 * (paper_2606_08804_amd/layer.py) calls: the chunk forward and backward on
 * the rows of its fused projection, and its gates.  They return the status codes of qdelta.h
 * and follow its conventions (device pointers, 16-byte alignment,
 * asynchronous on the caller's stream). */
#ifndef QDELTA_LAYER_H
#define QDELTA_LAYER_H

#include "qdelta.h"

#ifdef __cplusplus
extern "C" {
#endif

/* qkv [tokens, H, 2 Dk + Dv] (dtype), one row q | k | v per token and head;
 * q and k are L2-normalised per row into q, k [tokens, H, Dk] (written, with
 * 1 / |row| in rnorm_q, rnorm_k [tokens, H] as by qdelta_l2norm_fwd), v is
 * read in place.  cu_seqlens NULL: B sequences of T tokens; else B is ignored
 * and N sequences share T tokens.  The rest as qdelta_chunk_fwd. */
int qdelta_layer_fwd(int32_t B, int32_t T, int32_t N, const int32_t* cu_seqlens, int32_t H, int32_t Dk, int32_t Dv,
                     int32_t dtype, const void* qkv, const float* beta, const float* lam, float lam_scalar,
                     const float* log_alpha, const float* initial_state, void* q, void* k, float* rnorm_q,
                     float* rnorm_k, void* o, float* final_state, void* saved, void* ws, size_t ws_bytes,
                     hipStream_t stream);

/* The gradients of qdelta_layer_fwd from its saved context: dqkv like qkv
 * (the normalisation's backward applied to the q and k parts), the rest as
 * qdelta_chunk_bwd (workspace of qdelta_chunk_workspace_bytes with is_bwd). */
int qdelta_layer_bwd(int32_t B, int32_t T, int32_t N, const int32_t* cu_seqlens, int32_t H, int32_t Dk, int32_t Dv,
                     int32_t dtype, const void* qkv, const void* q, const void* k, const float* rnorm_q,
                     const float* rnorm_k, const float* beta, const float* lam, float lam_scalar,
                     const float* log_alpha, const float* initial_state, const void* saved, const void* d_o,
                     const float* d_final_state, void* dqkv, float* dbeta, float* dlam, float* dlog_alpha,
                     float* d_initial_state, void* ws, size_t ws_bytes, hipStream_t stream);

/* Gates from logits [tokens, n H] (dtype; contiguous rows of beta, then lambda
 * and alpha where lam and log_alpha are not NULL): beta = sigmoid(x),
 * lam = sigmoid(x + *bias) (one value of bias_dtype), log_alpha =
 * logsigmoid(x), each [tokens, H] fp32. */
int qdelta_layer_gates_fwd(int64_t tokens, int32_t H, int32_t dtype, int32_t bias_dtype, const void* logits,
                           const void* bias, float* beta, float* lam, float* log_alpha, hipStream_t stream);

/* Backward, from the gates themselves: dlogits like logits, *dbias the bias's
 * gradient (when lam is not NULL; parts: qdelta_layer_gate_parts floats of
 * workspace).  A NULL dbeta, dlam or dlog_alpha is a gradient of zeros. */
int32_t qdelta_layer_gate_parts(int64_t tokens, int32_t H);
int qdelta_layer_gates_bwd(int64_t tokens, int32_t H, int32_t dtype, int32_t bias_dtype, const float* beta,
                           const float* lam, const float* log_alpha, const float* dbeta, const float* dlam,
                           const float* dlog_alpha, void* dlogits, float* parts, void* dbias, hipStream_t stream);

#ifdef __cplusplus
}
#endif

#endif /* QDELTA_LAYER_H */
