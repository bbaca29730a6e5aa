// Key-side work items of the backward pass: how the block columns are cut, found from the index by every
// workgroup for itself.
#ifndef SPION_ATTN_KEY_ITEMS_H_
#define SPION_ATTN_KEY_ITEMS_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "attn_bf16_tiles.h"
#include "attn_common.h"
#include "../../include/spion.h"
#include "spion_internal.h"

namespace spion {

// ------------------------------------------------------------------------------------------------
// Vertical stripes give block columns with up to nb kept rows next to columns with one or two, so the key
// side does not take one column per workgroup.  The items are derived from col_ptr alone (the same list
// for every head).  A column with cnt kept rows is cut into nch = ceil(cnt / chunk) near-equal chunks if
// cnt > chunk, else it is one item (also when cnt == 0: its dK / dV must still be written as zeros).
// Items are numbered longest first, as far as that is cheap to find and worth it: the chunks of split columns in column
// order, then the unsplit columns, by length or in column order.  Chunk number w writes its fp32
// partial tiles to slot w; the last of a column's chunks to do so adds them up in chunk order (deterministic).
// ------------------------------------------------------------------------------------------------
constexpr int kChunk = 16;      // the shortest chunk that is cut; of the tuned kernel of block 64:
constexpr int kChunkLeast = 8;  // (partial tiles are sized for both)
constexpr int kChunkMax = 64;   // the longest
static_assert((SPION_MAX_NB + kChunkLeast - 1) / kChunkLeast < 1 << kArriveBits && RowCut::kSlots < 1 << kArriveBits,
              "a counter holds the parts of any column or row");

// Workgroups of the tuned backward that run at once: 134 to 160 VGPRs let three waves share a SIMD.
inline int bwd_resident(int bs) { return 256 * (bs == 64 ? 3 : 6); }

// Steps that each of them has to do in a balanced run, both sides, the fixed cost of a workgroup taken as one.
inline long long bwd_steps_per_slot(int BH, int bs, int nb, int nnzb) {
    return 2LL * BH * ((long long)nnzb + nb) / bwd_resident(bs);
}

// Most kept rows of a work item of the tuned backward.  A cut costs a partial tile written and read back for
// each piece; an uncut column is one chain of steps, which only has to end before the rest of the launch
// does: so as long as a balanced run.  Measured, backward call in us with chunks of 16 / 24 / 32 / 64:
// 16 heads x 4096, block 64, 328 blocks (16 steps a slot) 37 / 38 / 44 / 68; 32 heads, 410 blocks (39) 79 / 76 /
// 76 / 70, 852 blocks (76) 149 / 146 / 138 / 129 (121 with long rows first); 16 heads x 8192, block 32, 3277
// blocks (73) 143 / 136 / 130 / 98 (last with long rows first).
// Block 64 with less to do than that: down to 8, and twice the mean (columns of about the mean stay whole), so that the longest
// chain is shorter: 2 heads x 1024, 25 %, 17.2 -> 13.7, 8 x 1024 18.1 -> 14.7, 8 x 2048, 15 %, 23.4 -> 18.1, 1 x 8192, 5 %, 26.0 -> 23.8; 8 rows
// at a mean of 9.6, 2 x 4096, 15 %, 27.5 -> 30.0; block 32, whose steps are half as long, 8 x 4096, 5 %, 22.6 -> 25.0.
inline int key_chunk(int BH, int bs, int nb, int nnzb) {
    const long long c = bwd_steps_per_slot(BH, bs, nb, nnzb);
    const int twice = 2 * ((nnzb + nb - 1) / nb);
    const int least = bs != 64 || twice > kChunk ? kChunk : twice > kChunkLeast ? twice : kChunkLeast;
    return (int)(c < least ? least : c > kChunkMax ? kChunkMax : c);
}

struct KeyItem {
    int J;      // block column, -1: no such item
    int kb, ke; // BSC entries [kb, ke)
    int slot;   // partial slot, -1: the item covers its whole column and writes dK / dV itself
    int first, count;   // slot of the column's first chunk, its chunks
};

// The chunk number w of a split column, if it is one of those of this group of 64 columns; `run`: chunks of the groups before.
__device__ __forceinline__ bool chunk_of_group(KeyItem& it, int& run, int base, int c0, int cnt, int chunk, int w, int lane) {
    if (!__any(cnt > chunk)) return false;
    const int nch = cnt > chunk ? (cnt + chunk - 1) / chunk : 0;
    const int incl = wave_incl_scan(nch, lane);
    const int lo = run + incl - nch;
    const unsigned long long hit = __ballot(nch > 0 && w >= lo && w < lo + nch);
    if (hit) {
        const int src = __ffsll((long long)hit) - 1;
        const int c0s = __builtin_amdgcn_readlane(c0, src), cnts = __builtin_amdgcn_readlane(cnt, src);
        const int nchs = __builtin_amdgcn_readlane(nch, src);
        const int first = __builtin_amdgcn_readlane(lo, src);
        int ci = w - first;
        ci = ci < 0 ? 0 : (ci >= nchs ? nchs - 1 : ci);
        it = {base + src, c0s + (ci * cnts) / nchs, c0s + ((ci + 1) * cnts) / nchs, w, first, nchs};
        return true;
    }
    run += __builtin_amdgcn_readlane(incl, 63);
    return false;
}

// Units of length of the columns: a quarter of the mean, but `finest` blocks at least; 0: lengths do not count.
__device__ __forceinline__ float units_of_length(int nb, int nnzb, int finest) {
    return finest ? fminf(quarters_of_mean(nb, nnzb), __builtin_amdgcn_rcpf((float)finest)) : 0.f;
}

// All lanes of the calling wave must be active; the result is wave-uniform.  The unsplit columns longest first, lengths in units_of_length(),
// or (finest == 0) in their order.  Backward, columns of more than 8 rows first and so: fp32, 32 heads x 1024, block 64, 90.7 -> 84.0 us, 64 x 1024, block
// 32, 115 -> 111; bf16, block 64, 16 x 4096 36.7 -> 35.6.
template <int NG>
__device__ __forceinline__ KeyItem key_item(const int* __restrict__ col_ptr, int nb, int chunk, int finest, int w, int lane) {
    KeyItem it = {-1, 0, 0, -1, 0, 1};
    int c0[NG], cnt[NG];
#pragma unroll
    for (int k = 0; k < NG; ++k) {
        const int J = 64 * k + lane;
        c0[k] = J < nb ? col_ptr[J] : 0;
        cnt[k] = J < nb ? col_ptr[J + 1] - c0[k] : 0;
    }
    int run = 0;
#pragma unroll
    for (int k = 0; k < NG; ++k)
        if (chunk_of_group(it, run, 64 * k, c0[k], cnt[k], chunk, w, lane)) return it;
    const float quarters = units_of_length(nb, col_ptr[nb], finest);
    int key[NG];
    unsigned long long mask[NG];
#pragma unroll
    for (int k = 0; k < NG; ++k) {
        key[k] = length_key(cnt[k], quarters);
        mask[k] = __ballot(64 * k + lane < nb && cnt[k] <= chunk);
    }
    const int J = entry_by_length<NG>(key, mask, w - run, lane, finest > 0);
    if (J < 0) return it;
    int a = 0, n = 0;
#pragma unroll
    for (int k = 0; k < NG; ++k)
        if (J >> 6 == k) {
            a = __builtin_amdgcn_readlane(c0[k], J & 63);
            n = __builtin_amdgcn_readlane(cnt[k], J & 63);
        }
    return {J, a, a + n, -1, 0, 1};
}
// The same for any number of columns.
__device__ __forceinline__ KeyItem key_item_any(const int* __restrict__ col_ptr, int nb, int chunk, int finest, int w, int lane) {
    KeyItem it = {-1, 0, 0, -1, 0, 1};
    const float quarters = units_of_length(nb, col_ptr[nb], finest);
    EntriesByLength columns;
    int run = 0;
#pragma unroll 1
    for (int base = 0; base < nb; base += 256) {   // four groups whose loads are in flight together
        int c0[4], cnt[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int J = base + 64 * k + lane;
            c0[k] = J < nb ? col_ptr[J] : 0;
            cnt[k] = J < nb ? col_ptr[J + 1] - c0[k] : -1;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (chunk_of_group(it, run, base + 64 * k, c0[k], cnt[k], chunk, w, lane)) return it;
            columns.add(base / 64 + k, cnt[k] >= 0 && cnt[k] <= chunk, length_key(max(cnt[k], 0), quarters));
        }
    }
    const int J = columns.entry((nb + 63) / 64, w - run, lane);
    if (J < 0) return it;
    return {J, col_ptr[J], col_ptr[J + 1], -1, 0, 1};
}
__device__ __forceinline__ KeyItem key_item_lookup(const int* __restrict__ col_ptr, int nb, int chunk, int finest, int w, int lane) {
    if (nb <= (finest ? kChunkLeast : chunk)) {   // none is cut, all about alike
        if (w >= nb) return {-1, 0, 0, -1, 0, 1};
        return {w, col_ptr[w], col_ptr[w + 1], -1, 0, 1};
    }
    if (nb <= 64) return key_item<1>(col_ptr, nb, chunk, finest, w, lane);
    if (nb <= 128) return key_item<2>(col_ptr, nb, chunk, finest, w, lane);
    if (nb <= 256) return key_item<4>(col_ptr, nb, chunk, finest, w, lane);
    return key_item_any(col_ptr, nb, chunk, finest, w, lane);
}

}  // namespace spion
#endif
