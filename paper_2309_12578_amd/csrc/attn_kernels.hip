// Block-sparse attention forward and backward for gfx950 (Eq. 5 / Algorithm 5 lines 4-7 of the SPION
// paper, softmax as in Algorithm 6, gradient by the chain rule): fp32 with every block size, bf16 with
// block size 16, and the dispatch over all variants.
//
// One pattern (BSR, plus BSC for the backward) is shared by all batch items and heads.  A kept block
// is a dense bs x bs tile, so SDDMM and SpMM inside it are dense contractions and run on MFMA; the
// row softmax is fused between them and never touches HBM.
//
// Work split.  A wave owns 16 or 32 rows (queries on the query side, keys on the key side) and walks 16-row
// tiles of the other side that the index lists for them; up to four waves share the tiles of the same rows
// (wave w takes tiles w, w + 4, ...) and add up their accumulators through LDS once, at the end.  At the sizes that
// use these kernels the longest row's or column's chain of tiles is what takes the time (a pattern's one or two
// long rows are 4 times the average, and there are too few rows to fill the machine otherwise): four waves
// cut the chain by four, and since a tile belongs to one wave, nothing inside the loop needs a barrier.
// Measured against one wave per 16 rows with the tiles staged through LDS for the whole workgroup:
// fp32, 8 heads of 2048 tokens, block 32, 410 blocks: forward 70 -> 26 us, backward 179 -> 58 us (the
// products alone take 5.6 and 20 us at the matrix cores' fp32 rate); bf16, 9 heads of 1936, block 16, 1171
// blocks: 40 -> 12 and 67 -> 34 us.
//
// Operands come from global memory straight into registers.  Every product has the owned rows on the N
// index of a 16x16 MFMA tile: lane l = 16 g + r holds values of owned row r, which makes row statistics
// lane-uniform scalars, and makes an accumulator tile directly the B operand of the next product
// (element i of lane group g is contraction index 4 g + i).  The A operand of a product that contracts over d
// is a tile's rows (load_rows).  The A operand of a product that contracts over the tile's rows has, in lane
// (r, g), rows 4 g + i and some column set of its own for r: with columns 4 r + e (load_cols) these are
// 16 (8) contiguous bytes per row, i.e. whole rows per load instruction and no transpose; MFMA number e then
// yields output columns 4 m + e at M index m, so that a lane ends up with 16 consecutive columns.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "attn_bf16_tiles.h"
#include "attn_common.h"
#include "attn_key_items.h"
#include "spion_internal.h"

namespace spion {

namespace {

constexpr int kPatchLd = kD + 4;   // floats per row of the merge area: b128 accesses of 16 rows hit all banks evenly

// How a workgroup's waves share its work: WQ sets of 16 NQ owned rows, each with WT waves that take every WT-th
// step of the other side's tiles.
template <typename T, int BS, int NQ_, int WT_, int WQ_>
struct Split {
    static constexpr int NQ = NQ_, WT = WT_, WQ = WQ_, W = WT * WQ;
    static constexpr int OWN = 16 * NQ * WQ;          // rows of a workgroup
    static constexpr int PARTS = BS / OWN;            // workgroups per block row or column
    static_assert(WT == 1 || OWN % (4 * W) == 0, "the merge takes 4 W rows at a time, all of them the workgroup's");
    static constexpr int TPB = BS / 16;               // 16-row tiles per block
    static constexpr int KT = sizeof(T) == 2 ? 2 : 1; // tiles per step: a bf16 MFMA contracts over 32 rows
    static constexpr int STRIDE = WT * KT;            // tiles per step of all WT waves
    static constexpr int NDC = kD / Elem<T>::KC;
};
// The default, for rows long or few: every row's tiles over four waves (32 owned rows halve the tile traffic
// per product where the block has them).
template <typename T, int BS> using SplitFew = Split<T, BS, BS == 16 ? 1 : 2, 4, 1>;
// Many block rows of few tiles, see many_short_rows(): the start of a workgroup (index, owned rows) and its
// merge cost more than the tiles, so fewer waves share a row.
template <typename T, int BS> struct SplitMany;   // forward, backward, backward of rows with hardly more than one block
template <typename T> struct SplitMany<T, 16> {
    typedef Split<T, 16, 1, 2, 1> bwd, bwd_single;
};
template <typename T> struct SplitMany<T, 32> {
    typedef Split<T, 32, 1, 2, 2> fwd;
    typedef Split<T, 32, 2, 2, 1> bwd;
    typedef Split<T, 32, 2, 1, 1> bwd_single;
};
template <typename T> struct SplitMany<T, 64> {
    typedef Split<T, 64, 1, 1, 4> fwd;
    typedef Split<T, 64, 2, 2, 2> bwd;
    typedef Split<T, 64, 2, 1, 2> bwd_single;
};

// lane (r, g): elements g EPL .. of each d chunk of row r
template <typename T>
__device__ __forceinline__ void load_rows(typename Elem<T>::Frag (&f)[kD / Elem<T>::KC], const T* tile, int r, int g) {
#pragma unroll
    for (int c = 0; c < kD / Elem<T>::KC; ++c)
        f[c] = *reinterpret_cast<const typename Elem<T>::Frag*>(tile + r * kD + g * Elem<T>::EPL + c * Elem<T>::KC);
}
// lane (r, g): columns 4 r .. 4 r + 3 of rows 4 g + i
template <typename T>
__device__ __forceinline__ void load_cols(typename Elem<T>::Quad (&v)[4], const T* tile, int r, int g) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
        v[i] = *reinterpret_cast<const typename Elem<T>::Quad*>(tile + 4 * g * kD + 4 * r + i * kD);
}
template <typename V, int N>
__device__ __forceinline__ void clear(V (&v)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = V{};
}

// acc[e][M = m] += sum over the tiles' rows of tile[row][4 m + e] * x[row][owned]
template <int NQ, int KT>
__device__ __forceinline__ void mma_cols(f32x4 (&acc)[NQ][4], const f32x4 (&v)[KT][4], const f32x4 (&x)[NQ][KT]) {
#pragma unroll
    for (int j = 0; j < 4 * KT; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int h = 0; h < NQ; ++h)
                acc[h][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[j / 4][j % 4][e], x[h][j / 4][j % 4], acc[h][e], 0, 0, 0);
}
template <int NQ>
__device__ __forceinline__ void mma_cols(f32x4 (&acc)[NQ][4], const bf16x4 (&v)[2][4], const bf16x4 (&x)[NQ][2]) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const bf16x8 a = {v[0][0][e], v[0][1][e], v[0][2][e], v[0][3][e], v[1][0][e], v[1][1][e], v[1][2][e], v[1][3][e]};
#pragma unroll
        for (int h = 0; h < NQ; ++h) acc[h][e] = mma_d(acc[h][e], a, join(x[h][0], x[h][1]));
    }
}

template <int NQ>
__device__ __forceinline__ void clear_acc(f32x4 (&acc)[NQ][4]) {
#pragma unroll
    for (int h = 0; h < NQ; ++h) clear(acc[h]);
}

// A wave's accumulators into its part of the merge area (row-major, fp32).
template <int NQ>
__device__ __forceinline__ void put_patch(float* patch, const f32x4 (&acc)[NQ][4], int r, int g) {
#pragma unroll
    for (int h = 0; h < NQ; ++h)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            *reinterpret_cast<f32x4*>(patch + (h * 16 + r) * kPatchLd + 16 * g + 4 * i) =
                f32x4{acc[h][0][i], acc[h][1][i], acc[h][2][i], acc[h][3][i]};
}

// The same values as rows of the output, when no other wave holds a share of them.
template <typename T>
__device__ __forceinline__ void store_acc(T* row, const f32x4 (&acc)[4], float f, int g) {
#pragma unroll
    for (int i = 0; i < 4; ++i) store_quad<T>(row + 16 * g + 4 * i, f32x4{acc[0][i], acc[1][i], acc[2][i], acc[3][i]} * f);
}

// Block j of the list, lists of up to 64 blocks from the lanes of `head64` (no scalar load in the loop).
__device__ __forceinline__ int list_at(const int* list, int head64, int j) {
    return j < 64 ? __builtin_amdgcn_readlane(head64, j) : list[j];
}

// Work of a group of n items, dealt to the XCDs in contiguous eighths: items of one head share an L2.  The
// group takes 8 * ceil(n / 8) workgroups from a multiple of 8 on; -1: a workgroup past the end.
__device__ __forceinline__ int item_of_group(int id, int n) {
    const int item = (id & 7) * ((n + 7) >> 3) + (id >> 3);
    return item < n ? item : -1;
}
inline long long group_grid(long long n) { return (n + 7) / 8 * 8; }

// The block row that workgroup number l (all of a row's beside each other) takes when there are more than run at once.
// Heads that do not divide over the XCDs: the rows with more than twice the mean number of kept blocks first, of all the heads (a
// row of 80 blocks that starts last runs alone for as long as everything before it took), then head by
// head the others, so that neighbours in time share K and V in an L2; each of the two lists is shared out over the XCDs head by head.
// Patterns without a long row skip the second search, and the counts are loaded four groups at a time.  By length, on the XCDs
// as deal_heads() has them, which the bf16 kernels gain by, took as long: 96 shapes, forward 0.95 to 1.04 of the time, backward 0.95 to 1.11.
// All lanes of the calling wave must be active.
__device__ __forceinline__ ItemOfHead long_rows_first(const int* __restrict__ row_ptr, int nb, int heads, int l, int lane) {
    const int limit = 2 * row_ptr[nb] / nb;
    int n_long = 0, cnt_first = 0;   // rows 0 .. 63 are kept for the second search
    int base0 = 0;
    for (; base0 + 256 <= nb; base0 += 256) {   // four groups whose loads are in flight together
        int from[4], to[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            from[k] = row_ptr[base0 + 64 * k + lane];
            to[k] = row_ptr[base0 + 64 * k + lane + 1];
        }
        if (base0 == 0) cnt_first = to[0] - from[0];
#pragma unroll
        for (int k = 0; k < 4; ++k) n_long += __popcll(__ballot(to[k] - from[k] > limit));
    }
    for (int base = base0; base < nb; base += 64) {
        const int r = base + lane;
        const int cnt = r < nb ? row_ptr[r + 1] - row_ptr[r] : 0;
        if (base == 0) cnt_first = cnt;
        n_long += __popcll(__ballot(r < nb && cnt > limit));
    }
    const int longs = heads * n_long;
    const bool want_long = l < longs;
    int head, rank;
    if (want_long) {
        l = xcd_deal(l, 0, longs);
        head = l / n_long;
        rank = l % n_long;
    } else {
        l = xcd_deal(l, longs, heads * nb);
        head = l / (nb - n_long);
        rank = l % (nb - n_long);
    }
    if (n_long == 0) return {head, rank};
    for (int base = 0; base < nb; base += 64) {   // the counts are in the cache by now
        const int r = base + lane;
        int cnt = cnt_first;
        if (base != 0) cnt = r < nb ? row_ptr[r + 1] - row_ptr[r] : 0;
        const unsigned long long mine = __ballot(r < nb && (cnt > limit) == want_long);
        const int members = __popcll(mine);
        if (rank < members) {
            const unsigned long long hit = __ballot(((mine >> lane) & 1ull) && lanes_below(mine) == rank);
            return {head, base + __ffsll((long long)hit) - 1};
        }
        rank -= members;
    }
    return {head, 0};
}

// By length, all heads of an XCD together, where each XCD has whole heads: what starts last is short then.  Forward, long rows
// first and so: fp32, block 16, 16 x 2048 23.5 -> 22.5.
__device__ __forceinline__ ItemOfHead rows_in_order(const int* __restrict__ row_ptr, int nb, int heads, int l, int lane) {
    if (heads & 7) return long_rows_first(row_ptr, nb, heads, l, lane);
    const ItemOfHead mine = deal_heads(l, heads, false);
    return {mine.head, row_by_length(row_ptr, nb, mine.item, lane)};
}

}  // namespace

// ------------------------------------------------------------------------------------------------
// forward: workgroup = (head, S::OWN query rows)
// ------------------------------------------------------------------------------------------------
template <typename T, int BS, typename S, bool CUT>
__global__ __launch_bounds__(S::W * 64, 2) void attn_fwd_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, T* __restrict__ O,
    float* __restrict__ LSE, const int* __restrict__ row_ptr, const int* __restrict__ col_idx,
    CutOf<CUT> cut, int L, int nb, int total, int sort_rows, float scale_log2, int paper_denom) {
    typedef typename Elem<T>::Frag Frag;
    typedef typename Elem<T>::Quad Quad;
    constexpr int NQ = S::NQ, KT = S::KT, NDC = S::NDC, OWN = S::OWN;
    __shared__ __attribute__((aligned(16))) float o_s[S::WT][OWN * kPatchLd];
    __shared__ float m_s[S::WT][OWN], l_s[S::WT][OWN];

    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
    int bh, I, part, id = blockIdx.x;
    [[maybe_unused]] RowPieces cuts = {0, 1, 0, 0};
    [[maybe_unused]] int piece = 0;
    bool helper = false;
    if constexpr (CUT) {
        helper = id < cut.groups;
        if (!helper) id -= cut.groups;
    }
    if (helper) {   // a piece of a long row
        if constexpr (CUT) {
            const int i = (id >> 3) / S::PARTS * 8 + (id & 7), heads = total / (nb * S::PARTS), want = i / heads;
            if (want >= cut.helpers) return;
            cuts = row_pieces<false>(row_ptr, nb, cut, want, lane);
            if (cuts.row < 0) return;
            bh = i % heads;
            I = cuts.row;
            part = (id >> 3) % S::PARTS;
            piece = want - cuts.first + 1;
        }
    } else if (sort_rows) {
        const int row = (id >> 3) / S::PARTS * 8 + (id & 7);   // a row's workgroups on one XCD
        if (row >= total / S::PARTS) return;
        const ItemOfHead mine = rows_in_order(row_ptr, nb, total / (nb * S::PARTS), row, lane);
        bh = mine.head;
        I = mine.item;
        part = (id >> 3) % S::PARTS;
    } else {
        const int item = item_of_group(id, total);
        if (item < 0) return;
        bh = item / (nb * S::PARTS);
        I = item % (nb * S::PARTS) / S::PARTS;
        part = item % S::PARTS;
    }
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wt = wave % S::WT, own = wave / S::WT * (16 * NQ);
    const size_t head = (size_t)bh * L * kD;
    const int wg0 = I * BS + part * OWN, row0 = wg0 + own;   // rows of the workgroup, of the wave

    int jb = row_ptr[I];
    const int n_row = row_ptr[I + 1] - jb;
    int n = n_row;   // blocks of this workgroup
    if constexpr (CUT) if (n_row > cut.longest) {
        if (!helper) cuts = row_pieces<true>(row_ptr, nb, cut, I, lane);
        const int from = piece * n_row / cuts.count;
        n = (piece + 1) * n_row / cuts.count - from;
        jb += from;
    }
    const int nt = n * S::TPB;
    const int* cols = col_idx + jb;
    const int cols64 = n > 0 ? cols[lane < n ? lane : n - 1] : 0;
    Frag qf[NQ][NDC];
#pragma unroll
    for (int h = 0; h < NQ; ++h) load_rows<T>(qf[h], Q + head + (size_t)(row0 + 16 * h) * kD, r, g);
    auto tile_at = [&](int t) { return head + (size_t)(list_at(cols, cols64, t / S::TPB) * BS + t % S::TPB * 16) * kD; };
    // tile t + u of a step that starts at t; past the end: zeros
    auto load_k = [&](Frag (&k)[KT][NDC], int t) {
#pragma unroll
        for (int u = 0; u < KT; ++u) {
            if (u == 0 || t + u < nt) load_rows<T>(k[u], K + tile_at(t + u), r, g);
            else clear(k[u]);
        }
    };

    float m[NQ], limit[NQ], lsum[NQ];   // m: what a row's exponentials are taken against, log2 units
    f32x4 oacc[NQ][4];
#pragma unroll
    for (int h = 0; h < NQ; ++h) {
        m[h] = kLowest;
        limit[h] = -INFINITY;
        lsum[h] = 0.f;
    }
    clear_acc<NQ>(oacc);

    auto step = [&](const Frag (&kf)[KT][NDC], Frag (&knext)[KT][NDC], int t) {
        Quad vc[KT][4];
#pragma unroll
        for (int u = 0; u < KT; ++u) {
            if (u == 0 || t + u < nt) load_cols<T>(vc[u], V + tile_at(t + u), r, g);
            else clear(vc[u]);
        }
        if (t + S::STRIDE < nt) load_k(knext, t + S::STRIDE);
        __builtin_amdgcn_sched_barrier(0);
        // S^T: [tile row 4 g + i][query r]
        f32x4 s[NQ][KT];
        float mx[NQ];
        bool above = false;
#pragma unroll
        for (int h = 0; h < NQ; ++h) {
            mx[h] = -INFINITY;
#pragma unroll
            for (int u = 0; u < KT; ++u) {
                s[h][u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int c = 0; c < NDC; ++c) s[h][u] = mma_d(s[h][u], kf[u][c], qf[h][c]);
            }
        }
#pragma unroll
        for (int h = 0; h < NQ; ++h) {
#pragma unroll
            for (int u = 0; u < KT; ++u)
                if (u == 0 || t + u < nt)
#pragma unroll
                    for (int i = 0; i < 4; ++i) mx[h] = fmaxf(mx[h], s[h][u][i]);
            above |= mx[h] * scale_log2 > limit[h];
        }
        if (__any(above)) {   // always at a wave's first step
#pragma unroll
            for (int h = 0; h < NQ; ++h) {
                const float m_new = fmaxf(m[h], group_max(mx[h]) * scale_log2);
                const float alpha = exp2f(m[h] - m_new);
                m[h] = m_new;
                limit[h] = m_new + kRescaleSlack;
                lsum[h] *= alpha;
#pragma unroll
                for (int e = 0; e < 4; ++e) oacc[h][e] *= alpha;
            }
        }
        Quad pq[NQ][KT];
#pragma unroll
        for (int h = 0; h < NQ; ++h)
#pragma unroll
            for (int u = 0; u < KT; ++u) {
                f32x4 p;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    p[i] = exp2f(fmaf(s[h][u][i], scale_log2, -m[h]));
                    if (u > 0) p[i] = t + u < nt ? p[i] : 0.f;
                    lsum[h] += p[i];
                }
                pq[h][u] = to_quad<T>(p);
            }
        mma_cols(oacc, vc, pq);   // O^T += V^T P^T
    };
    {
        Frag ka[KT][NDC], kb[KT][NDC];
        int t = wt * KT;
        if (t < nt) load_k(ka, t);
        for (; t < nt; t += 2 * S::STRIDE) {
            step(ka, kb, t);
            if (t + S::STRIDE < nt) step(kb, ka, t + S::STRIDE);
        }
    }

    // Algorithm 6: every masked entry of the row counts as a score of 0 (a row that keeps nothing
    // has no entry to normalise and stays at O = 0, LSE = -inf).  The sums are up to 2^kRescaleSlack times what they
    // would be against the row's maximum.
    const float masked = paper_denom && n_row > 0 ? (float)(L - n_row * BS) : 0.f;
    if constexpr (S::WT == 1) {
#pragma unroll
        for (int h = 0; h < NQ; ++h) {
            const int q = row0 + h * 16 + r;
            const float mm = masked > 0.f ? fmaxf(m[h], 0.f) : m[h];
            float l = group_sum(lsum[h]);
            if (masked > 0.f) {
                l = scale_down(f32x4{l, 0.f, 0.f, 0.f}, m[h] - mm)[0] + masked * exp2f(-mm);
#pragma unroll
                for (int e = 0; e < 4; ++e) oacc[h][e] = scale_down(oacc[h][e], m[h] - mm);
            }
            store_acc<T>(O + head + (size_t)q * kD, oacc[h], l > 0.f ? 1.f / l : 0.f, g);
            if (g == 0) LSE[(size_t)bh * L + q] = l > 0.f ? (mm + log2f(l)) * kLn2 : -INFINITY;
        }
        return;
    }
    // the waves' shares of each row: rescaled to the row's largest m and added up in wave order
    put_patch<NQ>(&o_s[wt][own * kPatchLd], oacc, r, g);
#pragma unroll
    for (int h = 0; h < NQ; ++h) {
        const float l = group_sum(lsum[h]);
        if (g == 0) {
            m_s[wt][own + h * 16 + r] = m[h];
            l_s[wt][own + h * 16 + r] = l;
        }
    }
    __syncthreads();
    // four numbers of row q of this workgroup's blocks, the row's reference and sum
    auto merged = [&](int q, int d, float& mm, float& l) {
        mm = m_s[0][q];
#pragma unroll
        for (int w = 1; w < S::WT; ++w) mm = fmaxf(mm, m_s[w][q]);
        f32x4 o = f32x4{0.f, 0.f, 0.f, 0.f};
        l = 0.f;
        if (n > 0) {
#pragma unroll
            for (int w = 0; w < S::WT; ++w) {
                const float a = exp2f(m_s[w][q] - mm);
                l += l_s[w][q] * a;
                o += *reinterpret_cast<const f32x4*>(&o_s[w][q * kPatchLd + d]) * a;
            }
        }
        return o;
    };
    // [head][slot][part]: the rows' numbers, then their references and sums
    constexpr int kPart = OWN * (kD + 2);
    [[maybe_unused]] float* parts = nullptr;
    if constexpr (CUT) if (cuts.count > 1) {   // a long row in pieces: see attn_bf16_tiles.h
        __shared__ int flag;
        const size_t slot = ((size_t)bh * cut.slots + cuts.slot) * S::PARTS + part;
        parts = cut.parts + slot * kPart;
        float* const mine = parts + (size_t)piece * (S::PARTS * kPart);
#pragma unroll
        for (int p = 0; p < OWN; p += 4 * S::W) {
            const int q = p + (tid >> 4), d = (tid & 15) * 4;
            float mm, l;
            const f32x4 o = merged(q, d, mm, l);
            put_shared(mine + q * kD + d, o[0], o[1]);
            put_shared(mine + q * kD + d + 2, o[2], o[3]);
            if (d == 0) put_shared(mine + OWN * kD + 2 * q, mm, l);
        }
        if (!last_to_arrive(cut.counters + slot, cut.tag, cuts.count, &flag)) return;
    }
#pragma unroll
    for (int p = 0; p < OWN; p += 4 * S::W) {
        const int q = p + (tid >> 4), d = (tid & 15) * 4;
        float mm, l;
        f32x4 o;
        if (CUT && parts) {   // every piece has blocks, so that its references are finite
            mm = -INFINITY;
            l = 0.f;
            o = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
            for (int c = 0; c < cuts.count; ++c) {
                const float* const part = parts + (size_t)c * (S::PARTS * kPart);
                const float2 lo = get_shared(part + q * kD + d), hi = get_shared(part + q * kD + d + 2);
                const float2 ml = get_shared(part + OWN * kD + 2 * q);
                const float m_new = fmaxf(mm, ml.x), a = exp2f(mm - m_new), b = exp2f(ml.x - m_new);
                mm = m_new;
                l = l * a + ml.y * b;
                o = o * a + f32x4{lo.x, lo.y, hi.x, hi.y} * b;
            }
        } else {
            o = merged(q, d, mm, l);
        }
        if (masked > 0.f) {
            const float mp = fmaxf(mm, 0.f);
            o = scale_down(o, mm - mp);
            l = scale_down(f32x4{l, 0.f, 0.f, 0.f}, mm - mp)[0] + masked * exp2f(-mp);
            mm = mp;
        }
        const float inv = l > 0.f ? 1.f / l : 0.f;
        store_quad<T>(O + head + (size_t)(wg0 + q) * kD + d, o * inv);
        if (d == 0) LSE[(size_t)bh * L + wg0 + q] = l > 0.f ? (mm + log2f(l)) * kLn2 : -INFINITY;
    }
}

// ------------------------------------------------------------------------------------------------
// backward: one launch computes dQ, dK and dV.  Workgroup = (head, S::OWN rows of a block row) on the query
// side, or (head, S::OWN keys of a work item's block column) on the key side.  The sides share no data: the
// key side computes delta = rowsum(dO .* O) of the query rows it visits by itself.  Deterministic: sums over waves
// and chunks in fixed order.
// Grid: some of the long block rows, the long key items (chunks of split columns, long columns), the other block rows, the
// other key items; all heads in each.
// ------------------------------------------------------------------------------------------------
template <typename T, int BS, typename S, bool CUT>
__global__ __launch_bounds__(S::W * 64, 2) void attn_bwd_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, const T* __restrict__ O,
    const T* __restrict__ dO, const float* __restrict__ LSE, T* __restrict__ dQ, T* __restrict__ dK,
    T* __restrict__ dV, const int* __restrict__ row_ptr, const int* __restrict__ col_idx,
    const int* __restrict__ col_ptr, const int* __restrict__ row_idx, float* __restrict__ partial,
    unsigned long long* __restrict__ counters, unsigned long long tag, CutOf<CUT> cut, int n_slots, int BH, int L, int nb, int n_key_a,
    int n_rows, int n_key_c, int w_first, int chunk, int by_length, int early_rows, float scale, float scale_log2) {
    typedef typename Elem<T>::Frag Frag;
    typedef typename Elem<T>::Quad Quad;
    typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
    constexpr int NQ = S::NQ, KT = S::KT, NDC = S::NDC, OWN = S::OWN;
    __shared__ __attribute__((aligned(16))) float acc_s[S::WT][OWN * kPatchLd];
    __shared__ int flag;

    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wt = wave % S::WT, own = wave / S::WT * (16 * NQ);
    auto padded = [](int n) { return (n + 7) & ~7; };
    // early_rows > 0: rows by length (see launch_bwd), so many of them before everything else; a multiple of 8
    const int early = S::PARTS * early_rows;
    const int late = early_rows ? S::PARTS * padded(BH * n_rows) - early : padded(BH * n_rows * S::PARTS);
    int id = blockIdx.x, first = 0, first_row = 0;
    [[maybe_unused]] RowPieces cuts = {0, 1, 0, 0};
    [[maybe_unused]] int piece = 0;
    bool key_side = false, helper = false;
    if constexpr (CUT) {
        helper = id < cut.groups;
        if (!helper) id -= cut.groups;
    }
    if (!helper && id >= early) {
        id -= early;
        key_side = true;
        if (id >= BH * n_key_a * S::PARTS) {
            id -= padded(BH * n_key_a * S::PARTS);
            if (id < 0) return;
            key_side = false;
            first_row = early_rows;
            if (id >= late) {
                id -= late;
                first = w_first;
                key_side = true;
            }
        }
    }
    int bh, idx, sub;   // sub: the workgroup's rows within the block
    if (helper) {   // a piece of a long row
        if constexpr (CUT) {
            const int i = (id >> 3) / S::PARTS * 8 + (id & 7), want = i / BH;
            if (want >= cut.helpers) return;
            cuts = row_pieces<false>(row_ptr, nb, cut, want, lane);
            if (cuts.row < 0) return;
            bh = i % BH;
            idx = cuts.row;
            sub = (id >> 3) % S::PARTS * OWN;
            piece = want - cuts.first + 1;
        }
    } else if (key_side) {
        // The items of all heads together, longest first; heads keep to an XCD where that shares them out evenly.  (In
        // contiguous eighths, as the rows are, a few heads' long items met on a few XCDs: fp32, 3 x 4096, block 64, 75 -> 71.5 us;
        // 32 x 1024, block 64, 105 -> 96.)
        int x = 0, hpx = BH, l = id;
        if ((BH & 7) == 0) {
            x = id & 7;
            hpx = BH >> 3;
            l = id >> 3;
        }
        bh = x * hpx + l % hpx;
        idx = l / hpx;
        sub = idx % S::PARTS * OWN;
        idx = first + idx / S::PARTS;
        if (first && idx >= w_first + n_key_c) return;
    } else if (early_rows) {
        const int row = first_row + (id >> 3) / S::PARTS * 8 + (id & 7);   // a row's workgroups on one XCD
        if (row >= BH * n_rows) return;
        const ItemOfHead mine = rows_in_order(row_ptr, nb, BH, row, lane);
        bh = mine.head;
        idx = mine.item;
        sub = (id >> 3) % S::PARTS * OWN;
    } else {
        const int per_head = n_rows * S::PARTS, item = item_of_group(id, BH * per_head);
        if (item < 0) return;
        bh = item / per_head;
        idx = item % per_head / S::PARTS;
        sub = item % S::PARTS * OWN;
    }
    const size_t head = (size_t)bh * L * kD, vec = (size_t)bh * L;

    // adds up the waves' accumulators: row p + tid / 16, columns 4 (tid % 16) .. + 3
    auto merged = [&](int p) {
        const int o = (p + (tid >> 4)) * kPatchLd + (tid & 15) * 4;
        f32x4 v = *reinterpret_cast<const f32x4*>(&acc_s[0][o]);
#pragma unroll
        for (int w = 1; w < S::WT; ++w) v += *reinterpret_cast<const f32x4*>(&acc_s[w][o]);
        return v;
    };
    const int out = (sub + (tid >> 4)) * kD + (tid & 15) * 4;

    if (!key_side) {
        const int I = idx, row0 = I * BS + sub + own;
        int jb = row_ptr[I], n = row_ptr[I + 1] - jb;
        if constexpr (CUT) if (n > cut.longest) {
            if (!helper) cuts = row_pieces<true>(row_ptr, nb, cut, I, lane);
            const int from = piece * n / cuts.count;
            n = (piece + 1) * n / cuts.count - from;
            jb += from;
        }
        const int nt = n * S::TPB;
        const int* cols = col_idx + jb;
        const int cols64 = n > 0 ? cols[lane < n ? lane : n - 1] : 0;
        auto tile_at = [&](int t) { return head + (size_t)(list_at(cols, cols64, t / S::TPB) * BS + t % S::TPB * 16) * kD; };
        Frag kf[KT][NDC], vf[KT][NDC];
        Quad kc[KT][4];
        auto load_tiles = [&](int t) {   // tiles t, t + 1, ..; past the end: zeros
#pragma unroll
            for (int u = 0; u < KT; ++u) {
                if (u == 0 || t + u < nt) {
                    const size_t at = tile_at(t + u);
                    load_rows<T>(kf[u], K + at, r, g);
                    load_rows<T>(vf[u], V + at, r, g);
                    load_cols<T>(kc[u], K + at, r, g);
                } else {
                    clear(kf[u]);
                    clear(vf[u]);
                    clear(kc[u]);
                }
            }
        };
        Frag qf[NQ][NDC], dof[NQ][NDC];
        float delta[NQ], lse2[NQ];
        int t = wt * KT;
        if (t < nt) {   // a wave without tiles only takes part in the merge
            Frag of[NQ][NDC];
#pragma unroll
            for (int h = 0; h < NQ; ++h) {
                const size_t at = head + (size_t)(row0 + 16 * h) * kD;
                load_rows<T>(qf[h], Q + at, r, g);
                load_rows<T>(dof[h], dO + at, r, g);
                load_rows<T>(of[h], O + at, r, g);
                lse2[h] = LSE[vec + row0 + 16 * h + r] * kLog2e;
            }
            load_tiles(t);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int h = 0; h < NQ; ++h) {
                float dl = 0.f;
#pragma unroll
                for (int c = 0; c < NDC; ++c)
#pragma unroll
                    for (int e = 0; e < Elem<T>::EPL; ++e) dl = fmaf((float)dof[h][c][e], (float)of[h][c][e], dl);
                delta[h] = group_sum(dl);
            }
        }
        f32x4 dq[NQ][4];
        clear_acc<NQ>(dq);
        while (t < nt) {
            Quad dsq[NQ][KT];
#pragma unroll
            for (int h = 0; h < NQ; ++h)
#pragma unroll
                for (int u = 0; u < KT; ++u) {
                    // the accumulator starts at -delta: dP - delta comes out of the MFMA
                    f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f}, dp = f32x4{-delta[h], -delta[h], -delta[h], -delta[h]};
#pragma unroll
                    for (int c = 0; c < NDC; ++c) {
                        s = mma_d(s, kf[u][c], qf[h][c]);      // S^T = K Q^T
                        dp = mma_d(dp, vf[u][c], dof[h][c]);   // dP^T = V dO^T
                    }
                    f32x4 ds;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        ds[i] = exp2f(fmaf(s[i], scale_log2, -lse2[h])) * dp[i];
                        if (u > 0) ds[i] = t + u < nt ? ds[i] : 0.f;
                    }
                    dsq[h][u] = to_quad<T>(ds);
                }
            mma_cols(dq, kc, dsq);   // dQ^T += K^T dS^T
            t += S::STRIDE;
            if (t < nt) load_tiles(t);
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (S::WT == 1) {
#pragma unroll
            for (int h = 0; h < NQ; ++h) store_acc<T>(dQ + head + (size_t)(row0 + h * 16 + r) * kD, dq[h], scale, g);
            return;
        }
        put_patch<NQ>(&acc_s[wt][own * kPatchLd], dq, r, g);
        __syncthreads();
        if constexpr (CUT) if (cuts.count > 1) {   // a long row in pieces: see attn_bf16_tiles.h
            const size_t slot = ((size_t)bh * cut.slots + cuts.slot) * S::PARTS + sub / OWN;
            float* const parts = cut.parts + slot * (OWN * kD) + tid * 4;
            constexpr int kPiece = S::PARTS * OWN * kD;
#pragma unroll
            for (int p = 0; p < OWN; p += 4 * S::W) {
                const f32x4 v = merged(p);
                float* const mine = parts + (size_t)piece * kPiece + p * kD;
                put_shared(mine, v[0], v[1]);
                put_shared(mine + 2, v[2], v[3]);
            }
            if (!last_to_arrive(cut.counters + slot, cut.tag, cuts.count, &flag)) return;
#pragma unroll
            for (int p = 0; p < OWN; p += 4 * S::W) {
                f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
                for (int c = 0; c < cuts.count; ++c) {
                    const float* const part = parts + (size_t)c * kPiece + p * kD;
                    const float2 lo = get_shared(part), hi = get_shared(part + 2);
                    v += f32x4{lo.x, lo.y, hi.x, hi.y};
                }
                store_quad<T>(dQ + head + (size_t)(I * BS + p) * kD + out, v * scale);
            }
            return;
        }
#pragma unroll
        for (int p = 0; p < OWN; p += 4 * S::W)
            store_quad<T>(dQ + head + (size_t)(I * BS + p) * kD + out, merged(p) * scale);
        return;
    }

    const KeyItem it = key_item_lookup(col_ptr, nb, chunk, by_length, idx, lane);
    if (it.J < 0) return;
    const int n = it.ke - it.kb, nt = n * S::TPB, row0 = it.J * BS + sub + own;
    const int* rows = row_idx + it.kb;
    const int rows64 = n > 0 ? rows[lane < n ? lane : n - 1] : 0;
    auto row_at = [&](int t) { return list_at(rows, rows64, t / S::TPB) * BS + t % S::TPB * 16; };
    Frag kf[NQ][NDC], vf[NQ][NDC];
#pragma unroll
    for (int h = 0; h < NQ; ++h) {
        load_rows<T>(kf[h], K + head + (size_t)(row0 + 16 * h) * kD, r, g);
        load_rows<T>(vf[h], V + head + (size_t)(row0 + 16 * h) * kD, r, g);
    }
    f32x4 dk[NQ][4], dv[NQ][4];
    clear_acc<NQ>(dk);
    clear_acc<NQ>(dv);
    for (int t = wt * KT; t < nt; t += S::STRIDE) {
        Quad qc[KT][4], dc[KT][4];
        Quad pq[NQ][KT], dsq[NQ][KT];
#pragma unroll
        for (int u = 0; u < KT; ++u) {
            if (u == 0 || t + u < nt) {
                const int q0 = row_at(t + u);
                const size_t at = head + (size_t)q0 * kD;
                Frag qf[NDC], df[NDC], of[NDC];
                load_rows<T>(df, dO + at, r, g);
                load_rows<T>(of, O + at, r, g);
                load_rows<T>(qf, Q + at, r, g);
                const f32x4_any lse = *reinterpret_cast<const f32x4_any*>(LSE + vec + q0 + 4 * g);
                load_cols<T>(dc[u], dO + at, r, g);
                load_cols<T>(qc[u], Q + at, r, g);
                __builtin_amdgcn_sched_barrier(0);
                // -delta of rows 4 g + i in every lane: the lanes' shares of row r times a tile of ones
                float part = 0.f;
#pragma unroll
                for (int c = 0; c < NDC; ++c)
#pragma unroll
                    for (int e = 0; e < Elem<T>::EPL; ++e) part = fmaf((float)df[c][e], (float)of[c][e], part);
                const f32x4 ndelta = __builtin_amdgcn_mfma_f32_16x16x4f32(-part, 1.f, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
                for (int h = 0; h < NQ; ++h) {
                    f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f}, dp = ndelta;
#pragma unroll
                    for (int c = 0; c < NDC; ++c) {
                        s = mma_d(s, qf[c], kf[h][c]);     // S = Q K^T
                        dp = mma_d(dp, df[c], vf[h][c]);   // dP = dO V^T
                    }
                    f32x4 p, ds;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        p[i] = exp2f(fmaf(s[i], scale_log2, -lse[i] * kLog2e));
                        ds[i] = p[i] * dp[i];
                    }
                    pq[h][u] = to_quad<T>(p);
                    dsq[h][u] = to_quad<T>(ds);
                }
            } else {
                clear(dc[u]);
                clear(qc[u]);
#pragma unroll
                for (int h = 0; h < NQ; ++h) pq[h][u] = dsq[h][u] = Quad{};
            }
        }
        mma_cols(dv, dc, pq);    // dV^T += dO^T P
        mma_cols(dk, qc, dsq);   // dK^T += Q^T dS
    }
    // Final rows, or this chunk's fp32 partial tiles [head][slot][dK | dV][bs][64], unscaled: of a column's chunks, the
    // last to arrive with these rows adds all of them up, in their order (a launch for the sums took 4.3 to 5 us; these take
    // none to 2: bf16, 9 x 1936, 8 %, backward 28.8 + 4.7 -> 29.4 us, 24 x 1168, 8 %, 25.3 + 4.7 -> 27.1).
    constexpr int kPart = 2 * BS * kD;
    float* const parts = partial + ((size_t)bh * n_slots + it.first) * kPart;
    float* const pk = parts + (size_t)(it.slot - it.first) * kPart;   // read where slot >= 0
    const size_t column = head + (size_t)it.J * BS * kD;
    auto put = [&](float* p, f32x4 v) {
        put_shared(p, v[0], v[1]);
        put_shared(p + 2, v[2], v[3]);
    };
    auto last = [&] {
        return last_to_arrive(counters + ((size_t)bh * n_slots + it.first) * (BS / 16) + sub / OWN, tag, it.count, &flag);
    };
    // kInFlight parts are requested together: one by one, a trip past the L2 each, the sums took longer than a launch for them
    // would.  bf16, block 16, backward with the launch, one by one and so: 6 heads x 2016, five columns of 57 to 87 rows, 17.1 / 19.2 /
    // 17.0 us; 4 x 2624, 65 to 110 rows, 17.2 / 19.9 / 17.3.
    auto add_up = [&](int o) {   // four numbers of dK and of dV
        f32x4 ak = f32x4{0.f, 0.f, 0.f, 0.f}, av = f32x4{0.f, 0.f, 0.f, 0.f};
        constexpr int kInFlight = 8;
        for (int c = 0; c < it.count; c += kInFlight) {
            f32x4 k[kInFlight], v[kInFlight];
#pragma unroll
            for (int u = 0; u < kInFlight; ++u)
                if (c + u < it.count) {   // uniform
                    const float* p = parts + (size_t)(c + u) * kPart + o;
                    const float2 k0 = get_shared(p), k1 = get_shared(p + 2);
                    const float2 v0 = get_shared(p + BS * kD), v1 = get_shared(p + BS * kD + 2);
                    k[u] = f32x4{k0.x, k0.y, k1.x, k1.y};
                    v[u] = f32x4{v0.x, v0.y, v1.x, v1.y};
                }
#pragma unroll
            for (int u = 0; u < kInFlight; ++u)
                if (c + u < it.count) {
                    ak += k[u];
                    av += v[u];
                }
        }
        store_quad<T>(dK + column + o, ak * scale);
        store_quad<T>(dV + column + o, av);
    };
    if constexpr (S::WT == 1) {
        const int o = (sub + own + r) * kD;
        if (it.slot < 0) {
#pragma unroll
            for (int h = 0; h < NQ; ++h) {
                store_acc<T>(dK + column + (o + h * 16 * kD), dk[h], scale, g);
                store_acc<T>(dV + column + (o + h * 16 * kD), dv[h], 1.f, g);
            }
            return;
        }
#pragma unroll
        for (int h = 0; h < NQ; ++h)
#pragma unroll
            for (int i = 0; i < 4; ++i) {   // as store_acc
                float* const p = pk + o + h * 16 * kD + 16 * g + 4 * i;
                put(p, f32x4{dk[h][0][i], dk[h][1][i], dk[h][2][i], dk[h][3][i]});
                put(p + BS * kD, f32x4{dv[h][0][i], dv[h][1][i], dv[h][2][i], dv[h][3][i]});
            }
        if (!last()) return;
#pragma unroll
        for (int h = 0; h < NQ; ++h)
#pragma unroll
            for (int i = 0; i < 4; ++i) add_up(o + h * 16 * kD + 16 * g + 4 * i);
        return;
    }
#pragma unroll
    for (int which = 0; which < 2; ++which) {
        if (which) __syncthreads();
        put_patch<NQ>(&acc_s[wt][own * kPatchLd], which ? dv : dk, r, g);
        __syncthreads();
#pragma unroll
        for (int p = 0; p < OWN; p += 4 * S::W) {
            const f32x4 v = merged(p);
            const int o = p * kD + out;
            if (it.slot >= 0) put(pk + which * BS * kD + o, v);
            else store_quad<T>((which ? dV : dK) + column + o, which ? v : v * scale);
        }
    }
    if (it.slot < 0 || !last()) return;
#pragma unroll
    for (int p = 0; p < OWN; p += 4 * S::W) add_up(p * kD + out);
}

// ------------------------------------------------------------------------------------------------
// host launchers
// ------------------------------------------------------------------------------------------------
BwdWorkspace::BwdWorkspace(int BH, int bs, int nb, int nnzb_, int key_chunk, int mid_first, int row_slots_) {
    nnzb = nnzb_;
    row_slots = row_slots_;
    chunk = key_chunk;
    w_max = nnzb / chunk + nb;
    w_first = nnzb / chunk + 1 + mid_first;
    if (w_first > w_max) w_first = w_max;
    n_slots = 2 * (nnzb / chunk) + 2;
    // for the shortest chunks, so that a workspace for more kept blocks also serves fewer; multiples of 256
    int most = 2 * (nnzb / kChunk) + 2;
    if (bs == 64) {   // chunks shorter than kChunk are at least twice the mean: no more than nb / 2 of them in nnzb blocks
        const int least = 2 * (nnzb / kChunkLeast) + 2 < nb + 2 ? 2 * (nnzb / kChunkLeast) + 2 : nb + 2;
        if (least > most) most = least;
    }
    const size_t slots = (size_t)BH * most;
    counter_bytes = (slots * (bs / 16) * 8 + 255) / 256 * 256;
    total = counter_bytes + slots * 2 * bs * kD * sizeof(float);
    row_parts = total + ((size_t)BH * row_slots * (bs / 16) * 8 + 255) / 256 * 256;
    with_rows = row_parts + (size_t)BH * row_slots * bs * kD * sizeof(float);
}

// Rows with hardly more than one block each (the diagonal): no long chain to cut anywhere.
static bool single_block_rows(const AttnShape& s, int nnzb) { return 2 * (long long)nnzb < 3 * (long long)s.nb; }

// Block rows times rows of a head for every tile of its average row.
static double short_rows(const AttnShape& s, int nnzb) { return (double)s.BH * s.nb * s.nb / ((double)nnzb * (s.bs / 16)); }

// Whether a call has many block rows for every tile of its average row: 100.  Measured (fp32, and bf16 / block 16;
// patterns with a few long rows and columns, 2.4 to 9.6 blocks per row) the backward's crossing lies between 75
// and 200; without long rows it comes earlier, at 40 with the diagonal alone.
static bool many_short_rows(const AttnShape& s, int nnzb) { return short_rows(s, nnzb) >= (single_block_rows(s, nnzb) ? 40 : 100); }

// The backward's line of the larger blocks, with fp32 (the few's kernels' time over the many's, 110 shapes on both sides of the lines).  The diagonal alone:
// short_rows of 48 0.85, 63 to 127 0.98 to 1.17, above 1.2 to 1.3.  A few blocks besides: 40 to 96 0.69 to 0.99, 107 to 123 0.82 to 1.05, 124 to 147 0.89
// to 1.09 (1.03 on average), above 0.77 to 1.43.  More: up to 100 0.48 to 1.15 (0.83 on average).  From 100 on it takes rows that can be long and
// hardly more workgroups than run at once: up to 13 block rows 1.13 to 1.17 at 101 to 141 (30 x 352, block 32, 18.8 / 21.3 us), with over 2000 workgroups (of 32
// rows, both sides) 1.05 to 1.18 (16 x 2080, block 32, 62 / 74), the others 0.87 to 0.88 at 105 to 144 (42 x 544, block 32, 51 / 44) and
// 0.63 to 1.06 at 157 to 198.
static bool many_short_rows_bwd(const AttnShape& s, int nnzb) {
    if (s.bs == 16) return many_short_rows(s, nnzb);
    const bool can_be_long = s.nb >= 16 && 2ll * s.BH * s.nb * (s.bs / 32) <= 2000;
    return short_rows(s, nnzb) >= (10ll * nnzb < 11ll * s.nb ? 60 : single_block_rows(s, nnzb) ? 120 : can_be_long ? 150 : 100);
}

// What bwd_t takes, but for 16 rows a workgroup instead of 32: with these there are more workgroups and no more pieces.
struct GenericBwdSplit {
    int waves, waves_a_row, parts;   // of a workgroup, of them for the same rows; workgroups a block row
};
static GenericBwdSplit generic_bwd_split(const AttnShape& s, int nnzb) {
    if (!many_short_rows_bwd(s, nnzb)) return {4, 4, s.bs == 64 ? 2 : 1};
    const int wide = s.bs == 64 ? 2 : 1;
    return single_block_rows(s, nnzb) ? GenericBwdSplit{s.bs == 16 ? 2 : wide, s.bs == 16 ? 2 : 1, 1} : GenericBwdSplit{2 * wide, 2, 1};
}

// Workgroups of the generic backward that run at once: two (fp32) or three waves a SIMD.
static long long generic_bwd_resident(bool is_bf16, int waves) { return 256 * 4 * (is_bf16 ? 3 : 2) / waves; }

// Which of its query side's rows are cut, with the steps of both sides and as many helpers as the forward.
static void generic_bwd_decide(RowCut& cut, const AttnShape& s, int nnzb, int parts, long long resident) {
    cut.decide(s, nnzb, 2ll * s.BH * ((long long)nnzb + s.nb) * parts / resident);
    const long long most = 512 / ((long long)s.BH * parts);
    if (cut.slots > most) cut.slots = (int)most;
    if (cut.slots < 2) cut.slots = 0;
}

// Pieces of long rows per head, at most.
static int bwd_row_slots(const AttnShape& s, int nnzb) {
    if (s.is_bf16 && s.bs > 16) return bwd_bf16_row_slots(s, nnzb);
    RowCut cut;
    const GenericBwdSplit split = generic_bwd_split(s, nnzb);
    if (split.waves_a_row > 1) generic_bwd_decide(cut, s, nnzb, split.parts, generic_bwd_resident(s.is_bf16, split.waves));
    return cut.slots;
}

BwdWorkspace attn_bwd_workspace(const AttnShape& s, int nnzb) { return BwdWorkspace(s.BH, s.bs, s.nb, nnzb, kChunk, 0, bwd_row_slots(s, nnzb)); }

bool attn_bwd_grids_fit(int BH, int bs, int nb, int nnzb) {
    const BwdWorkspace ws(BH, bs, nb, nnzb, kChunk, 0, 0);
    const int64_t limit = 0x7fffffffll, parts = bs == 64 ? 2 : 1;
    return (int64_t)(ws.w_max + nb) * BH * parts + 24 <= limit &&
           (int64_t)(nb > kChunk ? nnzb / (kChunk + 1) : 0) * BH * (bs / 16) <= limit;   // rows of cut columns
}

// 16 rows a workgroup (32: half the tile traffic) until there are enough of them anyway: a row of many blocks is
// then shared by twice the compute units, whose matrix cores it fills.  fp32, 32 -> 16 rows: 2 heads x 8192, block
// 32, 3 %, 87 -> 54 us; 8 x 2048, 10 %, 24.3 -> 18.7; 4 x 1024, block 64, 20 %, 11.7 -> 7.8; 8 x 2048, 30 %, 37.5 -> 35.0;
// 32 x 2048, block 64 (2048 workgroups of 32 rows) 45.9 -> 47.3; 64 x 2048, block 32 (4096) 96.4 both.
// 0: many short rows, which waves do not share.
static int fwd_rows(const AttnShape& s, int nnzb) {
    if (s.bs == 16) return 16;
    if (many_short_rows(s, nnzb)) return 0;
    return s.bs > 16 && (long long)s.BH * s.L / 32 >= 2048 ? 32 : 16;
}

// Workgroups of four waves that run at once: four or three waves a SIMD.
static long long fwd_resident(int rows) { return 256 * (rows == 16 ? 4 : 3); }

// Whether there are half as many workgroups again as run at once, so that the order of the rows matters.
static bool fwd_many(const AttnShape& s, int rows) { return 2ll * s.BH * s.L / rows > 3 * fwd_resident(rows); }

// Rows in pieces, from twice the mean on as long as about all workgroups run at once (else the long ones start first, and
// have to outlast the launch from there to be cut).  Forward kernel, fp32, block 32: 2 heads x 8192, 3 %, 51 -> 23.4 us; 4 x 4096, 5 %, 28 -> 18.9; 8 x 2048, 10 %,
// 20.3 -> 17.7, 20 %, 28.6 -> 26; block 64, 3 x 4096, 10 %, 31.4 -> 26.8; block 16, 2 x 2048, 15.7 -> 12.  Patterns without a long row pay 2 to 7 %, at most
// (5 x 2368, block 64) 11.7 -> 13.2.  Cut where the rule leaves them whole, 16 x 2048: block 32 28.9 -> 30, block 16 22.7 -> 23.5, bf16 15.3 -> 16.1.
// Block 16, whose rows are short work: fp32, long rows, 64 block rows 4 heads 9.0 -> 9.8, 9 heads 15.1 -> 11.9; 65 9.0 -> 10.2, 12.3 -> 12.0; 80 10.3 -> 10.8,
// 14.6 -> 13.8; 110 and more 0.62 to 0.89 of the time.  bf16, a row of 65 to 70 blocks breaks even; uncut to cut on average over 12 patterns, 9 heads (more
// workgroups than run at once from 114 block rows on): 115 block rows 1.04, 121 1.00, 130 0.95, 144 0.93, 160 0.88; 4 heads: 121 1.11, 136 1.07, 144 1.02, 160
// 0.95, 180 0.94; 2 heads: 136 1.07, 144 1.02, 160 0.97.
RowCut generic_fwd_cut(const AttnShape& s, int nnzb) {
    RowCut cut;
    if (s.nb <= 32) return cut;   // decide() cuts none
    const int rows = fwd_rows(s, nnzb);
    if (rows == 0) return cut;
    const bool many = fwd_many(s, rows);
    // block 16: rows that can be long enough for what the pieces cost, 2 us
    const int least = !s.is_bf16 ? 64 : (long long)s.BH * s.nb > fwd_resident(16) ? 120 : 150;
    if (many ? s.BH > 8 : s.bs == 16 && s.nb <= least) return cut;   // rather no helpers that find nothing to do
    const int parts = s.bs / rows;
    cut.decide(s, nnzb, (many ? 2 : 1) * (long long)s.BH * nnzb * parts / fwd_resident(rows), !many);
    const long long most = 512 / ((long long)s.BH * parts);   // a helper for each piece, and not many that find nothing to do
    if (cut.slots > most) cut.slots = (int)most;
    if (cut.slots < 2) return RowCut{};
    cut.helpers = cut.slots - 1;
    cut.groups = parts * ((s.BH * cut.helpers + 7) & ~7);
    return cut;
}

template <typename T, int BS, typename S>
static hipError_t launch_fwd(const AttnShape& s, const void* Q, const void* K, const void* V, void* O,
                             float* LSE, const int* row_ptr, const int* col_idx, int nnzb, hipStream_t st) {
    const long long total = (long long)s.nb * s.BH * S::PARTS;
    // Rows by length or long ones first (rows_in_order), as in launch_bwd.  fp32, block 32: 32 heads x 2048, 10 %, 61.3 -> 48.3 us, 16 x 2048 33.3 -> 29.1; block 16, 16 x
    // 2048, 6 %, 27.2 -> 22.7; bf16, 17.2 -> 15.4.  The search costs half a microsecond to one: 9 x 1936 (few more than run at once)
    // 12.7 -> 13.2; up to 32 block rows no row is long enough, 32 x 1024, block 64, 28.2 -> 29.2.
    const int sort_rows = s.nb > 32 && (long long)nnzb * (BS / 16) >= 6ll * s.nb && fwd_many(s, S::OWN);
    const long long grid = sort_rows ? S::PARTS * group_grid((long long)s.nb * s.BH) : group_grid(total);
    if (grid > 0x7fffffffll) return hipErrorInvalidValue;
    auto launch = [&](auto kernel, auto cut_arg, int helpers) {
        kernel<<<dim3((unsigned)(helpers + grid)), dim3(S::W * 64), 0, st>>>(
            static_cast<const T*>(Q), static_cast<const T*>(K), static_cast<const T*>(V), static_cast<T*>(O), LSE, row_ptr, col_idx,
            cut_arg, s.L, s.nb, (int)total, sort_rows, s.scale * kLog2e, s.paper_denom);
    };
    RowCut cut;
    if (s.fwd_room) cut = RowCut(s, nnzb);
    if constexpr (S::WT > 2) {
        if (cut.slots && grid + cut.groups <= 0x7fffffffll) {
            launch(attn_fwd_kernel<T, BS, S, true>, cut, cut.groups);
            return hipGetLastError();
        }
    }
    launch(attn_fwd_kernel<T, BS, S, false>, NoCut{}, 0);
    return hipGetLastError();
}

// The query side's rows that are cut, with the steps of both sides.  Backward kernel, fp32, block 32: 2 heads x 8192, 3 %, rows of
// 80 blocks, 125 -> 61.8 us; 4 x 4096, 5 %, 61.6 -> 52.8; block 16, 2 x 2048, 8 %, 26.4 -> 21.3; patterns that are left whole, the same.
// Where two waves share a row (many_short_rows) its chain is twice as long: bf16, block 16, 9 x 1936, 8 %, rows of 65 blocks, 29.2 -> 26.5; fp32, block 16,
// 10 x 1408, 8 %, 35.1 -> 32.8; with rows that did not set the time 54.1 -> 54.6 (10 x 3200, 6 %), 22.2 -> 22.5 (12 x 1280, 10 %).
static RowCut generic_bwd_cut(const AttnShape& s, const BwdWorkspace& ws, int parts, long long resident, void* workspace) {
    RowCut cut;
    if (!s.bwd_room) return cut;
    generic_bwd_decide(cut, s, ws.nnzb, parts, resident);
    if (cut.slots > ws.row_slots) cut.slots = ws.row_slots;   // (it is not)
    if (cut.slots == 0) return cut;
    cut.helpers = cut.slots - 1;
    cut.groups = parts * ((s.BH * cut.helpers + 7) & ~7);
    cut.counters = reinterpret_cast<unsigned long long*>(static_cast<char*>(workspace) + ws.total);
    cut.parts = reinterpret_cast<float*>(static_cast<char*>(workspace) + ws.row_parts);
    return cut;
}

template <typename T, int BS, typename S>
static hipError_t launch_bwd(const AttnShape& s, const void* Q, const void* K, const void* V, const void* O,
                             const void* dO, const float* LSE, void* dQ, void* dK, void* dV, const int* row_ptr,
                             const int* col_idx, const int* col_ptr, const int* row_idx, const BwdWorkspace& ws,
                             void* workspace, hipStream_t st) {
    auto* const counters = static_cast<unsigned long long*>(workspace);
    float* const partial = reinterpret_cast<float*>(static_cast<char*>(workspace) + ws.counter_bytes);
    const bool rows = (s.bwd_phases & 1) != 0, keys = (s.bwd_phases & 2) != 0;
    const int n_key_a = keys ? ws.w_first : 0, n_rows = rows ? s.nb : 0, n_key_c = keys ? ws.w_max - ws.w_first : 0;
    const long long per_item = (long long)s.BH * S::PARTS;
    // Rows by length or long ones first (rows_in_order), where a quarter more workgroups than run at once (two or three waves a SIMD) follow:
    // one that starts late runs on alone.  fp32: 2 heads x 8192, block 32, 3 %, 161 -> 148 us; 3 x 4096, block 64, 10 %, 86 -> 76; 8 x 2048,
    // block 32, 15 %, 78 -> 71, 10 % 52.7 both; bf16, block 16: 10 x 4096, 4 %, 71 -> 67, 9 x 1936, 8 %, 31.3 -> 30.0; rows of fewer
    // than 6 tiles on average gain nothing and pay the search, up to 1 us (bf16, block 16, searched and not: 24 x 1168, 4 %, 19.5,
    // 18.8; 16 x 2048, 3 %, 25.1, 24.3, 5 %, 33.7, 34.1; 16 block rows, fp32, 16 x 512, 28.7, 27.5; fp32, block 32: 24 x 2336, 4 %, 81.2, 79.8; 16 x 1024, 10 %, 49.4, 50.9).
    const long long resident = generic_bwd_resident(sizeof(T) == 2, S::W);
    const int sort_rows = rows && (long long)ws.nnzb * (BS / 16) >= 6ll * s.nb &&
                          s.nb >= 32 && 4 * per_item * (n_key_a + n_rows + n_key_c) > 5 * resident;
    // and a row a head for every 32 of them before the key side's items too: there the long ones are.  2 heads x 8192: 136 -> 125;
    // 4 x 4096, 5 %, 70.6 -> 62.2.
    const long long row_items = group_grid((long long)s.BH * n_rows), some = group_grid((long long)s.BH * ((s.nb + 31) / 32));
    const int early_rows = (int)(!sort_rows ? 0 : some < row_items ? some : row_items);
    // Unsplit columns by length, so that long ones come before the rows, where half as many workgroups again as run at once make the order matter
    // (the search costs a workgroup a microsecond: 16 heads x 512, block 32, 29.1 -> 30.4).  fp32, block 32: 16 x 1024, 10 %, 46.4 -> 34.7,
    // 20 %, 68 -> 49.4; 64 x 1024, 15 %, 142 -> 113; 24 x 2336, 4 %, 74.6 -> 69; block 64, 32 x 1024, 20 %, 95.7 -> 87.3.
    const int by_length = 2 * per_item * (n_key_a + n_rows + n_key_c) > 3 * resident;
    const long long grid = group_grid(per_item * n_key_a) + (sort_rows ? S::PARTS * row_items : group_grid(per_item * n_rows)) +
                           group_grid(per_item * n_key_c);
    auto launch = [&](auto kernel, auto cut_arg, int helpers) {
        kernel<<<dim3((unsigned)(helpers + grid)), dim3(S::W * 64), 0, st>>>(
            static_cast<const T*>(Q), static_cast<const T*>(K), static_cast<const T*>(V), static_cast<const T*>(O),
            static_cast<const T*>(dO), LSE, static_cast<T*>(dQ), static_cast<T*>(dK), static_cast<T*>(dV), row_ptr,
            col_idx, col_ptr, row_idx, partial, counters, s.tag, cut_arg, ws.n_slots, s.BH, s.L, s.nb, n_key_a, n_rows, n_key_c,
            ws.w_first, ws.chunk, by_length, early_rows, s.scale, s.scale * kLog2e);
        return hipGetLastError();
    };
    if (grid <= 0) return hipSuccess;
    if constexpr (S::WT > 1) {
        const RowCut cut = rows ? generic_bwd_cut(s, ws, S::PARTS, resident, workspace) : RowCut{};
        if (cut.slots && grid + cut.groups <= 0x7fffffffll) return launch(attn_bwd_kernel<T, BS, S, true>, cut, cut.groups);
    }
    return launch(attn_bwd_kernel<T, BS, S, false>, NoCut{}, 0);
}

template <typename T, int BS>
static hipError_t fwd_t(const AttnShape& s, const void* Q, const void* K, const void* V, void* O,
                        float* LSE, const int* row_ptr, const int* col_idx, int nnzb, hipStream_t st) {
    if constexpr (sizeof(T) == 2 && BS >= 32) {
        return fwd_bf16<BS>(s, Q, K, V, O, LSE, row_ptr, col_idx, nnzb, st);
    } else {
        const int rows = fwd_rows(s, nnzb);
        if constexpr (BS > 16) {
            if (rows == 0) return launch_fwd<T, BS, typename SplitMany<T, BS>::fwd>(s, Q, K, V, O, LSE, row_ptr, col_idx, nnzb, st);
            if (rows == 32) return launch_fwd<T, BS, SplitFew<T, BS>>(s, Q, K, V, O, LSE, row_ptr, col_idx, nnzb, st);
        }
        return launch_fwd<T, BS, Split<T, BS, 1, 4, 1>>(s, Q, K, V, O, LSE, row_ptr, col_idx, nnzb, st);
    }
}

template <typename T, int BS>
static hipError_t bwd_t(const AttnShape& s, const void* Q, const void* K, const void* V, const void* O,
                        const void* dO, const float* LSE, void* dQ, void* dK, void* dV,
                        const int* row_ptr, const int* col_idx, const int* col_ptr, const int* row_idx,
                        int nnzb, void* workspace, hipStream_t st) {
    if constexpr (sizeof(T) == 2 && BS >= 32) {
        const BwdWorkspace ws(s.BH, s.bs, s.nb, nnzb, key_chunk(s.BH, BS, s.nb, nnzb), s.nb / 4, bwd_row_slots(s, nnzb));
        return bwd_bf16<BS>(s, Q, K, V, O, dO, LSE, dQ, dK, dV, row_ptr, col_idx, col_ptr, row_idx, ws, workspace, st);
    } else {
        const BwdWorkspace ws(s.BH, s.bs, s.nb, nnzb, kChunk, s.nb / 8, bwd_row_slots(s, nnzb));
        auto* launch = launch_bwd<T, BS, SplitFew<T, BS>>;
        // 16 rows or keys a workgroup instead of 32 while there are at most 800 of 32 (from six blocks a row on 760), of which 512 (of four waves) run at
        // once: the compute units that the second, short round of them leaves idle are worth more than the tiles' second reading.  fp32, backward
        // kernel, 32 -> 16 rows, block 32: 2 heads x 512, 20 %, 20.3 -> 14.5 us; 2 x 2048, 10 %, 35.0 -> 26.4; block 64: 1 x 4096 57.3 -> 42.5.
        // Where the line lies (the time with 32 rows over that with 16, 196 shapes): 450 to 640 workgroups 0.95 to 1.65 (1.25 on average), 640 to 720
        // 0.80 to 1.78 (1.14), 720 to 760 0.87 to 1.35 (1.07; 11 x 864, block 32, 40.8 / 54, but 4 x 2464 43.6 / 40.0), 760 to 800 with shorter rows 0.90 to
        // 1.35 (1.11), with longer ones 0.86 to 1.03 (0.94: 4 x 2624, block 32, 44.5 / 39.1); 800 to 900 0.86 to 1.26 (0.99), beyond that 0.89 to 1.13
        // (0.95).  With few block rows there is no long chain to shorten: 18 x 384, block 64, 20.4 -> 21.7, 8 x 512 15.4 -> 17.2.
        if constexpr (BS > 16)
            if (s.nb >= 16 && (long long)s.BH * (ws.w_max + s.nb) * (BS / 32) <= (nnzb > 6ll * s.nb ? 760 : 800)) launch = launch_bwd<T, BS, Split<T, BS, 1, 4, 1>>;
        if (many_short_rows_bwd(s, nnzb))
            launch = single_block_rows(s, nnzb) ? launch_bwd<T, BS, typename SplitMany<T, BS>::bwd_single>
                                                               : launch_bwd<T, BS, typename SplitMany<T, BS>::bwd>;
        return launch(s, Q, K, V, O, dO, LSE, dQ, dK, dV, row_ptr, col_idx, col_ptr, row_idx, ws, workspace, st);
    }
}

#define SPION_DISPATCH(FN, ...)                                                   \
    do {                                                                          \
        if (s.is_bf16) {                                                          \
            if (s.bs == 16) return FN<bf16_t, 16>(__VA_ARGS__);                   \
            if (s.bs == 32) return FN<bf16_t, 32>(__VA_ARGS__);                   \
            return FN<bf16_t, 64>(__VA_ARGS__);                                   \
        }                                                                         \
        if (s.bs == 16) return FN<float, 16>(__VA_ARGS__);                        \
        if (s.bs == 32) return FN<float, 32>(__VA_ARGS__);                        \
        return FN<float, 64>(__VA_ARGS__);                                        \
    } while (0)

hipError_t launch_attn_fwd(const AttnShape& s, const void* Q, const void* K, const void* V, void* O,
                           float* LSE, const int* row_ptr, const int* col_idx, int nnzb, hipStream_t st) {
    SPION_DISPATCH(fwd_t, s, Q, K, V, O, LSE, row_ptr, col_idx, nnzb, st);
}

hipError_t launch_attn_bwd(const AttnShape& s, const void* Q, const void* K, const void* V,
                           const void* O, const void* dO, const float* LSE, void* dQ, void* dK,
                           void* dV, const int* row_ptr, const int* col_idx, const int* col_ptr,
                           const int* row_idx, int nnzb, void* workspace, hipStream_t st) {
    SPION_DISPATCH(bwd_t, s, Q, K, V, O, dO, LSE, dQ, dK, dV, row_ptr, col_idx, col_ptr, row_idx, nnzb,
                   workspace, st);
}

}  // namespace spion
