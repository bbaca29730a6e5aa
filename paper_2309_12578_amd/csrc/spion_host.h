// Entry points of libspion that its own Python front end uses besides those of include/spion.h.
#ifndef SPION_HOST_H_
#define SPION_HOST_H_

#include <stddef.h>
#include <stdint.h>

#include "../../include/spion.h"

#ifdef __cplusplus
extern "C" {
#endif

// spion_pattern, then waits for it on the host; *nnzb_out (HOST) receives nnzb.
int spion_pattern_wait(const float* A_s, const spion_pattern_params* p, uint8_t* fl_out, int32_t* row_ptr,
                       int32_t* col_idx, int32_t* col_ptr, int32_t* row_idx, int32_t* bsr_pos, int32_t* nnzb,
                       int64_t* pool_sum, void* workspace, size_t workspace_bytes, void* hip_stream,
                       int32_t* nnzb_out);

// dW [N, M] = dY^T X for bf16 dY [rows, N] and X [rows, M], all contiguous, N and M multiples of 8; fp32 sums.
size_t spion_weight_grad_workspace_bytes(int32_t rows, int32_t N, int32_t M);
int spion_weight_grad(const void* dY, const void* X, void* dW, int32_t rows, int32_t N, int32_t M, void* workspace,
                      size_t workspace_bytes, void* hip_stream);

// LayerNorm over contiguous rows of D elements (a multiple of 64, at most 2048), fp32 or bf16; mean and rstd [rows], fp32.
int spion_layer_norm(const void* x, const void* w, const void* b, void* y, float* mean, float* rstd, int32_t rows, int32_t D,
                     float eps, int32_t dtype, void* hip_stream);
size_t spion_layer_norm_workspace_bytes(int32_t rows, int32_t D);
// dr: added to dx (the gradient of a residual that leaves from x), or NULL.
int spion_layer_norm_grad(const void* dy, const void* dr, const void* x, const void* w, const float* mean, const float* rstd,
                          void* dx, void* dw, void* db, int32_t rows, int32_t D, int32_t dtype, void* workspace,
                          size_t workspace_bytes, void* hip_stream);

// Head split (split != 0) or merge: merged [B, L, n, H, 64] <-> tensors t[0 .. n - 1] [B, H, L, 64], n = 1 or 3, fp32 or
// bf16, L a multiple of 4, fewer than 2^31 vectors of 16 bytes.
int spion_heads(int32_t split, void* merged, void* const* t, int32_t B, int32_t L, int32_t H, int32_t n, int32_t dtype,
                void* hip_stream);

// spion_attn_fwd with room for the pieces of long block rows (0 bytes: none are cut), which only these two calls' kernels
// use; room == NULL: as spion_attn_fwd.  Aligned to 256 bytes.
size_t spion_attn_fwd_room_bytes(const spion_attn_params* p, int32_t nnzb);
int spion_attn_fwd_room(const void* Q, const void* K, const void* V, void* O, float* LSE, const int32_t* row_ptr,
                        const int32_t* col_idx, int32_t nnzb, const spion_attn_params* p, void* room, size_t room_bytes,
                        void* hip_stream);

// spion_attn_fwd_room / spion_attn_bwd (p, room, workspace and index as there) on the sub-layer's own tensors: qkv and dqkv
// [B, L, 3, H, 64], S = O and dS [B, L, H, 64], LSE [B, H, L].  bf16 and block 32 or 64 only (else SPION_ERR_DTYPE,
// SPION_ERR_SHAPE), tensors aligned to 16 bytes.
int spion_heads_attn_fwd(const void* qkv, void* S, float* LSE, const int32_t* row_ptr, const int32_t* col_idx, int32_t nnzb,
                         const spion_attn_params* p, void* room, size_t room_bytes, void* hip_stream);
int spion_heads_attn_bwd(const void* qkv, const void* S, const void* dS, const float* LSE, void* dqkv, const int32_t* row_ptr,
                         const int32_t* col_idx, const int32_t* col_ptr, const int32_t* row_idx, int32_t nnzb,
                         const spion_attn_params* p, void* workspace, size_t workspace_bytes, void* hip_stream);

#ifdef __cplusplus
}
#endif
#endif
