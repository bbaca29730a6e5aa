// Internal launcher declarations shared by the translation units of libspion (not installed).
#ifndef SPION_INTERNAL_H_
#define SPION_INTERNAL_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace spion {

// pattern_kernels.hip
// part: the seven slot sums of every input block (pattern_part_bytes), written by launch_conv_pool and added
// up by launch_pool_gather / launch_pattern_finish into pool[nb * nb].  launch_pattern_finish with
// from_part == false starts from a given pool[]; part is scratch of the larger grids either way, and so is
// aux (pattern_aux_bytes).  nnzb_host: nullptr, or a word of host memory that receives nnzb as well; with
// nb <= 64 it is the last store of the call.
size_t pattern_part_bytes(size_t nb);
size_t pattern_aux_bytes(size_t nb);
hipError_t launch_conv_pool(const float* A, int L, int bs, int p, long long* part, void* aux, hipStream_t st);
hipError_t launch_pool_gather(const long long* part, int nb, long long* pool, hipStream_t st);
hipError_t launch_pattern_finish(bool from_part, long long* part, long long* pool, int nb, int mode, long long k_rank,
                                 double kval, double t_abs, int no_fill, void* aux, uint8_t* fl, int* row_ptr,
                                 int* col_idx, int* col_ptr, int* row_idx, int* bsr_pos, int* nnzb, int* nnzb_host,
                                 hipStream_t st);

// producer_kernels.hip
hipError_t launch_index_check(const int* row_ptr, const int* col_idx, const int* col_ptr, const int* row_idx,
                              const int* bsr_pos, int nb, int nnzb, int err_code, int* status, hipStream_t st);
hipError_t launch_score_mean(const void* A, int is_bf16, int n_maps, size_t n, float* out, hipStream_t st);
hipError_t launch_copy_yardstick(const void* src, void* dst, size_t n_tiles, hipStream_t st);
size_t frobenius_workspace_bytes();
hipError_t launch_frobenius_distance(const float* a, const float* b, size_t n, double* out, void* workspace,
                                     hipStream_t st);

// attn_kernels.hip
// Of a counter of arrivals: as few as hold the parts of one row or column (attn_key_items.h), 128 at most, because its other
// bits are the tag that tells it from what was in the memory before.  With 40 bits of tag instead of 56 a counter is
// taken for begun, and its sums come from nobody, 2^16 times as often.
constexpr int kArriveBits = 8;

struct AttnShape {
    int BH, L, bs, nb;
    int is_bf16;
    float scale;        // resolved score scale (> 0)
    int paper_denom;    // Algorithm 6's extra denominator term
    int bwd_phases;     // bit 0: query side (dQ); bit 1: key side (dK, dV)
    int heads_beside;   // 0: tensors [B, H, L, 64]; else H, and rows as HeadRows<true> (bf16, block 32 and 64 only)
    void* fwd_room;     // forward: device memory of RowCut::room_bytes() for the pieces of long rows, or nullptr: rows stay whole
    bool bwd_room;      // backward: the workspace has the room of BwdWorkspace::with_rows; else long rows stay whole
    unsigned long long tag;       // of this call alone, below 2^(64 - kArriveBits) (see last_to_arrive)
};

// How the kernels cut long block rows (see attn_bf16_tiles.h), from what the host knows of a pattern.
struct RowCut {
    int piece = 0;     // kept blocks of a piece, at most, unless there are too many pieces (row_pieces())
    int longest = 0;   // a row of more is cut
    int slots = 0;     // pieces per head that there is room for; 0: no row is cut
    int helpers = 0;   // workgroups per head for the pieces behind the first of each row
    int groups = 0;    // of all heads, a multiple of 8
    unsigned long long tag = 0;
    unsigned long long* counters = nullptr;   // [head][slots] (fp32, block 16: [workgroup of a block row]), in use: that of a row's first piece
    float* parts = nullptr;                   // partial results, as many
    RowCut() = default;
    RowCut(const AttnShape& s, int nnzb);   // the forward's
    // piece, longest and slots, where each of the workgroups that run at once has `steps` to do; short_too: rows from
    // twice the mean on
    void decide(const AttnShape& s, int nnzb, long long steps, bool short_too = false);
    // Most: two rows of half the columns at 3 % kept blocks; 0.6 MB of room per head.  Patterns with more or longer ones have them in larger
    // pieces: 8 full rows among 128, 4 heads, block 64, forward 33 us (whole 72), backward 41 (97).
    static constexpr int kSlots = 32;
    size_t counter_bytes(int BH) const { return ((size_t)BH * slots * 4 * 8 + 255) / 256 * 256; }
    // O, maximum, sum; the kernels of fp32 and block 16 use 66 floats a row of these 72
    static constexpr size_t partial_bytes(int bs) { return (size_t)(bs / 16) * 64 * 18 * sizeof(float); }
    size_t room_bytes(int BH, int bs) const { return slots ? counter_bytes(BH) + (size_t)BH * slots * partial_bytes(bs) : 0; }
};

// attn_kernels.hip: the plan for fp32 and block 16, without its memory
RowCut generic_fwd_cut(const AttnShape& s, int nnzb);

hipError_t launch_attn_fwd(const AttnShape& s, const void* Q, const void* K, const void* V, void* O,
                           float* LSE, const int* row_ptr, const int* col_idx, int nnzb, hipStream_t st);
hipError_t launch_attn_bwd(const AttnShape& s, const void* Q, const void* K, const void* V,
                           const void* O, const void* dO, const float* LSE, void* dQ, void* dK,
                           void* dV, const int* row_ptr, const int* col_idx, const int* col_ptr,
                           const int* row_idx, int nnzb, void* workspace, hipStream_t st);

// The backward workspace: fp32 partial dK / dV tiles for block columns that are cut into several chunks and, behind them, dQ
// tiles for long block rows.  What a call must have is the first, and a workspace for more kept blocks serves it; the
// second is sized for one number of kept blocks, nothing where no row can be cut.
struct BwdWorkspace {
    int nnzb;
    int chunk;                       // most kept rows of a key-side work item
    int w_max, w_first;              // work items per head (upper bound); those that may be chunks come first
    int n_slots;                     // partial slots per head (upper bound)
    size_t counter_bytes;            // one per slot and 16 rows, at the workspace's start; the partial tiles behind them
    size_t total;                    // of the columns; the rows' counters (one for every 16 rows) start there
    int row_slots;                   // partial slots per head for pieces of rows
    size_t row_parts, with_rows;     // where their partial tiles start, and end
    // mid_first: unsplit columns to make room for among the items that come first
    BwdWorkspace(int BH, int bs, int nb, int nnzb, int key_chunk, int mid_first, int row_slots);
};
BwdWorkspace attn_bwd_workspace(const AttnShape& s, int nnzb);   // its sizes
// false when a backward launch for this shape would need more workgroups than a 1-D grid can hold
bool attn_bwd_grids_fit(int BH, int bs, int nb, int nnzb);

// norm_kernels.hip: LayerNorm over rows of D = 64 k <= 2048 elements
size_t layer_norm_workspace_bytes(int rows, int D);
hipError_t launch_layer_norm(const void* x, const void* w, const void* b, void* y, float* mean, float* rstd, int rows,
                             int D, float eps, bool is_bf16, hipStream_t st);
hipError_t launch_layer_norm_grad(const void* dy, const void* dr, const void* x, const void* w, const float* mean,
                                  const float* rstd, void* dx, void* dw, void* db, float* partial, int rows, int D, bool is_bf16, hipStream_t st);

// projection_kernels.hip: dW [N, M] = dY^T X over `rows` rows, bf16, N and M multiples of 8
size_t weight_grad_workspace_bytes(int rows, int N, int M);
hipError_t launch_weight_grad(const void* dY, const void* X, void* dW, int rows, int N, int M, void* workspace,
                              hipStream_t st);

// merged [B, L, n, H, 64] <-> n tensors [B, H, L, 64], n = 1 or 3, L a multiple of 4
hipError_t launch_heads(bool split, void* merged, void* const* t, int B, int L, int H, int n, bool is_bf16, hipStream_t st);

// attn_bf16_kernels.hip: tuned bf16 forward, BS in {32, 64}
template <int BS>
hipError_t fwd_bf16(const AttnShape& s, const void* Q, const void* K, const void* V, void* O, float* LSE,
                    const int* row_ptr, const int* col_idx, int nnzb, hipStream_t st);

// attn_bwd_bf16_kernels.hip: tuned bf16 backward, BS in {32, 64}; both sides in one launch; pieces of long rows per head, at most
int bwd_bf16_row_slots(const AttnShape& s, int nnzb);
template <int BS>
hipError_t bwd_bf16(const AttnShape& s, const void* Q, const void* K, const void* V, const void* O,
                    const void* dO, const float* LSE, void* dQ, void* dK, void* dV, const int* row_ptr,
                    const int* col_idx, const int* col_ptr, const int* row_idx, const BwdWorkspace& ws,
                    void* workspace, hipStream_t st);

}  // namespace spion
#endif
