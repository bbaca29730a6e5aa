// bf16 block-sparse attention forward (Eq. 5 / Algorithm 5 lines 5-7, softmax as in Algorithm 6) tuned
// for gfx950, block size 32 or 64.
//
// Same mathematics and wave tiling as the generic kernels (16 owned rows per wave on the N index of
// every MFMA tile), plus:
//   - K / V tiles travel HBM -> LDS through the memory pipeline, one block ahead of the block being
//     multiplied, one barrier per kept block;
//   - the kernel starts loading the diagonal block before it has read the index;
//   - workgroup ids are remapped so that each of the 8 XCDs (one L2 each) works on few heads at a time.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "attn_bf16_tiles.h"
#include "attn_common.h"
#include "spion_internal.h"

namespace spion {

// ------------------------------------------------------------------------------------------------
// K / V tiles in two LDS stages, the next block loading while the
// current one is multiplied.  Two stages of {K, V} are 32 KB at block 64; four workgroups share a CU
// with up to 40 KB each.  (A third stage is 48 KB, i.e. three workgroups per CU, and measured 5-10 %
// slower; three K stages + two V stages with a second barrier per block measured 4 % slower.)
// ------------------------------------------------------------------------------------------------
template <int BS>
struct KvSmem {
    bf16_t k[BS * kD];
    bf16_t v[BS * kD];
};

// Wait until this wave's loads of the current block have landed, then meet the other waves: their
// parts have landed too and nobody reads the other stage any more.  younger_in_flight: the block
// after this one was already requested (only at step 0, from the prologue) and may stay in flight.
// A bare barrier: __syncthreads adds fences the kernel has no use for.
__device__ __forceinline__ void stage_ready(bool younger_in_flight) {
    if (younger_in_flight) __builtin_amdgcn_s_waitcnt(kWaitVm4);
    else __builtin_amdgcn_s_waitcnt(kWaitVm0);
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Block row I of head bh.  CUT: its first piece alone if it is a long one; HELPER: the given piece, one of cuts.count.
template <int BS, bool BESIDE, bool CUT, bool HELPER>
__device__ __forceinline__ void attend(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
    bf16_t* __restrict__ O, float* __restrict__ LSE, const int* __restrict__ row_ptr,
    const int* __restrict__ col_idx, const HeadRows<BESIDE>& at, const CutOf<CUT>& cut, int L, int nb, float scale_log2,
    int paper_denom, KvSmem<BS>& sm0, KvSmem<BS>& sm1, int bh, int I, int piece, RowPieces cuts, int lane, int wave) {
    constexpr int NKT = BS / 16;
    const int r = lane & 15, g = lane >> 4;
    const size_t head = at.in_head(bh, L);
    const int row_len = at.in_row();
    const int qrow = I * BS + wave * 16 + r;
    const SwzLane sl(r, g);
    const TileLoadLane tl(wave, lane, row_len);

    auto issue = [&](KvSmem<BS>& st, int J) {
        tile_load_async(K + head + (size_t)J * BS * row_len, st.k, wave, tl);
        tile_load_async(V + head + (size_t)J * BS * row_len, st.v, wave, tl);
    };
    if (!HELPER) issue(sm0, I);   // the diagonal block, before any index is known
    bf16x8 qf[2];
#pragma unroll
    for (int c = 0; c < 2; ++c)
        qf[c] = *reinterpret_cast<const bf16x8*>(Q + head + (size_t)qrow * row_len + c * 32 + g * 8);
    int jb = row_ptr[I];
    const int n_row = row_ptr[I + 1] - jb;
    int n = n_row;   // blocks of this workgroup
    if constexpr (CUT) if (n_row > cut.longest) {
        if (!HELPER) cuts = row_pieces<true>(row_ptr, nb, cut, I, lane);
        const int from = piece * n_row / cuts.count;
        n = (piece + 1) * n_row / cuts.count - from;
        jb += from;
    }
    const int last = n > 0 ? n - 1 : 0;
    const int* cols = col_idx + jb;
    int first[8];
    int pd = n > 0 ? find_in_row(cols, n, I, first) : -1;
    if (HELPER) pd = -1;   // in index order, the diagonal block where it comes
    // block visited at step t (clamped reads stay inside this row's entries; an empty row reads nothing)
    auto col_at = [&](int t) {
        const int j = walk_index(t < last ? t : last, pd);
        return j < 8 ? pick8(first, j) : cols[j];
    };
    // the same for t >= 2: the first 64 blocks of the walk sit one per lane (one readlane instead of thirty
    // scalar instructions a step); older than block 1's tiles, so the wait of step 0 covers the load
    int walk_v = 0;
    if (n > 2) walk_v = cols[walk_index(lane < last ? lane : last, pd)];
    auto later_col = [&](int t) {
        const int u = t < last ? t : last;
        return u < 64 ? __builtin_amdgcn_readlane(walk_v, u) : cols[walk_index(u, pd)];
    };
    if (pd < 0 && n > 0) {
        // no diagonal block in this row (piece): once everyone's early load has landed, load block 0 over it
        if (!HELPER) {
            __builtin_amdgcn_s_waitcnt(kWaitVm0);
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        }
        issue(sm0, first[0]);
    }
    // the second block goes out as soon as its index is known; it is the youngest load from here on
    if (n > 0) issue(sm1, col_at(1));   // (a one-block row loads its block twice: keeps the wait below uniform)

    float m = kLowest;   // what the row's exponentials are taken against, log2 units (score * scale * log2 e)
    f32x4 lacc = f32x4{0.f, 0.f, 0.f, 0.f};   // running row sum, replicated in its 4 elements
    f32x4 oacc[4];
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) oacc[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 ones;
#pragma unroll
    for (int e = 0; e < 8; ++e) ones[e] = (bf16_t)1.0f;

    auto step = [&](const KvSmem<BS>& cur, KvSmem<BS>& tgt, int it) {
        // loads in flight here: block `it`, and at step 0 also block 1, requested by the prologue (the
        // four youngest loads: whatever else the prologue stored or loaded after them only adds waiting)
        stage_ready(it == 0);
        if (it > 0) {
            if (it + 1 < n) issue(tgt, later_col(it + 1));
        }
        // S^T tile kt: [key 16 kt + 4 g + i][query r]; all K fragments are requested up front
        bf16x8 kfr[NKT][2];
#pragma unroll
        for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
            for (int c = 0; c < 2; ++c)
                kfr[kt][c] = *reinterpret_cast<const bf16x8*>(cur.k + kt * 16 * kD + sl.frag[c]);
        f32x4 s[NKT];
#pragma unroll
        for (int kt = 0; kt < NKT; ++kt) {
            s[kt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < 2; ++c) s[kt] = mma_d(s[kt], kfr[kt][c], qf[c]);
        }
        // the transposed V operands of O^T += V^T P^T do not depend on P: requested here, they land
        // while the exponentials below are computed
        constexpr int NM = (BS / 32) * 4;
        bf16x8 vop[NM];
#pragma unroll
        for (int j = 0; j < NM; ++j) {
            const int o = sl.tr(j & 3) + (j >> 2) * 32 * kD;
            vop[j] = join(lds_read_tr(cur.v + o), lds_read_tr(cur.v + 16 * kD + o));
        }
        __builtin_amdgcn_sched_barrier(0);
        bf16x4 pq[NKT];
        f32x4 sums;
        // row sums on the MFMA pipe: a tile of ones times P^T adds up each owned row's probabilities
        // (the bf16 values that also enter P V), every accumulator element holding the same sum
        auto probabilities = [&]() {
#pragma unroll
            for (int kt = 0; kt < NKT; ++kt) {
                f32x4 p;
#pragma unroll
                for (int i = 0; i < 4; ++i) p[i] = fast_exp2(fmaf(s[kt][i], scale_log2, -m));
                pq[kt] = to_quad<bf16_t>(p);
            }
            sums = lacc;
#pragma unroll
            for (int pc = 0; pc < BS / 32; ++pc) sums = mma_d(sums, ones, join(pq[2 * pc], pq[2 * pc + 1]));
        };
        if (it > 0) probabilities();
        // A sum out of bounds tells of a score far above the reference (or NaN): the row takes a higher one and the block's exponentials
        // are taken again.  The step is bound by the issue of vector and matrix instructions (41 of the former and 18 of the latter a
        // wave); the maximum of all scores took another 16 (57: 590 clocks at four waves a SIMD, 485 without its loads).  32 heads x 4096, block 64,
        // 13 blocks a row 42.0 -> 39.8 us, 16 x 16320 80.4 -> 77.4; block 32, 64 x 1024, 25 %, 18.7 -> 17.5.
        if (it == 0 || __any(!(sums[0] <= kSumLimit))) {
            float mx = s[0][0];
#pragma unroll
            for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
                for (int i = 0; i < 4; ++i) mx = fmaxf(mx, s[kt][i]);
            float m_new = fmaxf(m, group_max(mx) * scale_log2);
            if (lacc[0] > 1.f) m_new = fmaxf(m_new, m + log2f(lacc[0]));   // a sum that many blocks have added up to
            const float alpha = fast_exp2(m - m_new);
            m = m_new;
            lacc *= alpha;
#pragma unroll
            for (int dt = 0; dt < 4; ++dt) oacc[dt] *= alpha;
            probabilities();
        }
        lacc = sums;
#pragma unroll
        for (int j = 0; j < NM; ++j) {
            const int pc = j >> 2;
            oacc[j & 3] = mma_d(oacc[j & 3], vop[j], join(pq[2 * pc], pq[2 * pc + 1]));   // O^T[d][query] += V^T P^T
        }
    };

    for (int it = 0; it < n; it += 2) {
        step(sm0, sm1, it);
        if (it + 1 < n) step(sm1, sm0, it + 1);
    }

    // an empty row never waited for its early load: it must land before this workgroup's LDS is freed
    __builtin_amdgcn_s_waitcnt(kWaitVm0);

    if constexpr (CUT) if (cuts.count > 1) {   // a long row in pieces: see attn_bf16_tiles.h
        constexpr int kPart = 64 * 18;   // floats of a wave: nine pairs a lane, its accumulators, then reference and sum
        const size_t slot = (size_t)bh * cut.slots + cuts.slot;
        float* const parts = cut.parts + (slot * (BS / 16) + wave) * kPart + lane * 2;
        float* const mine = parts + (size_t)piece * (BS / 16) * kPart;
#pragma unroll
        for (int i = 0; i < 8; ++i) put_shared(mine + i * 128, oacc[i / 2][i % 2 * 2], oacc[i / 2][i % 2 * 2 + 1]);
        put_shared(mine + 1024, m, lacc[0]);
        // (the flag's place: nobody reads tiles any more behind the barriers, and the patch below is in the K tiles)
        if (!last_to_arrive(cut.counters + slot, cut.tag, cuts.count, reinterpret_cast<int*>(sm0.v))) return;
        m = -INFINITY;
        lacc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) oacc[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int c = 0; c < cuts.count; ++c) {
            const float* const part = parts + (size_t)c * (BS / 16) * kPart;
            float2 v[9];
#pragma unroll
            for (int i = 0; i < 9; ++i) v[i] = get_shared(part + i * 128);
            const float m_new = fmaxf(m, v[8].x), a = fast_exp2(m - m_new), b = fast_exp2(v[8].x - m_new);
            m = m_new;
            lacc = lacc * a + v[8].y * b;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int e = i % 2 * 2;
                oacc[i / 2][e] = oacc[i / 2][e] * a + v[i].x * b;
                oacc[i / 2][e + 1] = oacc[i / 2][e + 1] * a + v[i].y * b;
            }
        }
    }
    float lsum = lacc[0];
    if (paper_denom && n_row > 0 && L > n_row * BS) {
        // Algorithm 6: every masked entry of the row counts as a score of 0 (a row that keeps nothing
        // has no entry to normalise and stays at O = 0, LSE = -inf).  The sums are up to 2^kRescaleSlack times
        // what they would be against the row's maximum.
        const float mp = fmaxf(m, 0.f);
        lsum = scale_down(lacc, m - mp)[0] + (float)(L - n_row * BS) * exp2f(-mp);
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) oacc[dt] = scale_down(oacc[dt], m - mp);
        m = mp;
    }
    const float inv = lsum > 0.f ? 1.f / lsum : 0.f;
    // the stage that the last block did not use is free: every wave is past the barrier that followed
    // its last reader, and the only load that ever targets this wave's 2 KB of it was the wave's own
    bf16_t* patch = ((n & 1) ? sm1.k : sm0.k) + wave * (16 * kD);
    store_rows_coalesced(patch, O + at.out_head(bh, L) + (size_t)(I * BS + wave * 16) * at.out_row(), at.out_row(), oacc, inv, lane);
    if (g == 0) LSE[(size_t)bh * L + qrow] = lsum > 0.f ? (m + log2f(lsum)) * kLn2 : -INFINITY;
}

// In which order block rows start, see fwd_bf16().
enum RowOrder { kAsTheyLie, kDealt, kByLength };

template <int BS, bool BESIDE, bool CUT>
__global__ __launch_bounds__(BS * 4, BS == 64 ? 4 : 5) void attn_fwd_bf16_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
    bf16_t* __restrict__ O, float* __restrict__ LSE, const int* __restrict__ row_ptr,
    const int* __restrict__ col_idx, HeadRows<BESIDE> at, CutOf<CUT> cut, int L, int nb, int heads, RowOrder order,
    float scale_log2, int paper_denom) {
    __shared__ __attribute__((aligned(16))) KvSmem<BS> sm0, sm1;

    const int tid = threadIdx.x;
    int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int id = blockIdx.x;
    if constexpr (CUT) if (id < cut.groups) {   // pieces of long rows
        const int all = heads * cut.helpers;
        if (id >= all) return;
        const int l = xcd_deal(id, 0, all), bh = l / cut.helpers;
        for (int p = l % cut.helpers;; p += cut.helpers) {   // ends behind the head's last piece
            const RowPieces cuts = row_pieces<false>(row_ptr, nb, cut, p, lane);
            if (cuts.row < 0) return;
            attend<BS, BESIDE, true, true>(Q, K, V, O, LSE, row_ptr, col_idx, at, cut, L, nb, scale_log2, paper_denom, sm0, sm1, bh,
                                     cuts.row, p - cuts.first + 1, cuts, lane, wave);
            __syncthreads();   // everyone is done with the tiles' memory
            asm volatile("" : "+v"(lane));   // nothing per lane is kept in registers for the next piece
        }
    }
    if constexpr (CUT) id -= cut.groups;
    ItemOfHead mine;
    if (order == kAsTheyLie) {
        const int vid = xcd_deal(id, 0, heads * nb);
        mine = {vid / nb, vid % nb};
    } else {
        mine = deal_heads(id, heads, false);
        if (mine.item >= nb) return;
        if (order == kByLength) mine.item = row_by_length(row_ptr, nb, mine.item, lane);
    }
    const int I = mine.item;
    attend<BS, BESIDE, CUT, false>(Q, K, V, O, LSE, row_ptr, col_idx, at, cut, L, nb, scale_log2, paper_denom, sm0, sm1, mine.head, I, 0,
                              RowPieces{I, 1, 0, 0}, lane, wave);
}

// Workgroups that run at once: 4 (block 64) and at least 8 (block 32) fit a compute unit.
static int fwd_resident(int bs) { return 256 * (bs == 64 ? 4 : 8); }

// A row is long if it is four times the mean (24 blocks) and, at twice the pace of a workgroup among others, still outlasts the
// launch: twice the steps that each of the workgroups that run at once has to do.  bf16 forward, us, uncut / cut (patterns
// with two long rows): 8 heads x 8192, block 32, rows of 121 blocks, 41.9 / 20.1; 4 x 16384, block 64, 65.5 / 29.2; 4 x 8192, block 64, rows of
// 71, 37.6 / 20.9; 1 x 4096, block 32, 17.1 / 10.8; 16 x 16320, block 64, rows of 112, 83.1 / 78.1.  Rows of 45 and 27 at 64 x 4160 and 128 x 2080,
// block 32, which the rule leaves whole, 38.6 / 40.5 and 38.5 / 41.9.  A pattern without long rows: 76.6 / 76.9, 14.7 / 14.8.
// short_too: rows of twice the mean are cut, where nothing hides the longest (the callers' rules).  33 to 64 block rows that all run at once:
// 8 x 2048, block 32, rows of 24 blocks, 11.2 / 9.5; 32 x 2048 19.3 / 16.6; 4 x 4096, block 64, 16.7 / 13.1; 16 x 4096, 10 %, 26.1 / 19.9; 2 x 4096,
// 15 %, 20.8 / 13.7; without long rows 14.9 / 14.6.
// Pieces of the mean, of rows from half as long again on, where the mean is 10 blocks (`fine`; before 3/2 of it, from twice the mean on): forward, 45 shapes of 34 to
// 255 block rows, 0.83 to 1.04 of the time, 0.93 on average (5 x 3008, block 32, 18.6 blocks a row, 15.7 / 13.2; 9 x 4096, block 64, 12.3, 20.7 / 17.5; 14 x
// 4928, block 64, 35.8 / 37.2).  Left out, over 90 shapes of 33 to 256 block rows: bf16 forward 0.91 to 1.42 of the time, 1.09 on average, backward
// 0.98 to 1.35, 1.02; fp32 forward 0.75 to 1.22, 1.03 (2 x 2240, block 64, 32.4 / 24.3, is worse cut), backward 0.97 to 1.01.  With means of 6 to 9, 0.91 to
// 1.29; block 16, 0.90 to 1.10.
void RowCut::decide(const AttnShape& s, int nnzb, long long steps, bool short_too) {
    // Up to 64 block rows a row is not that long, and what the others pay shows: a kernel of 45 us without a row to cut, 32 heads x
    // 4096, block 64, took 1 us longer.
    if (s.nb <= (short_too ? 32 : 64)) return;
    const int mean = (nnzb + s.nb - 1) / s.nb;
    const bool fine = short_too && s.bs > 16 && mean >= 10;
    piece = fine ? mean : short_too ? (mean < 6 ? 8 : 3 * mean / 2) : (mean < 6 ? 12 : 2 * mean);
    longest = fine ? 3 * mean / 2 : short_too ? (mean < 6 ? 12 : 2 * mean) : (mean < 6 ? 24 : 4 * mean);
    if (s.bs == 16 && longest < 24) longest = 24;
    if (longest < 2 * steps) longest = 2 * steps < s.nb ? (int)(2 * steps) : s.nb;
    if (s.nb <= longest) return;   // no row can be cut
    const int most = nnzb / piece + nnzb / (longest + 1);   // pieces there can be
    slots = most < kSlots ? most : kSlots;
    if (slots < 2) slots = 0;
    tag = s.tag;
}

RowCut::RowCut(const AttnShape& s, int nnzb) {
    if (!s.is_bf16 || s.bs == 16) {
        *this = generic_fwd_cut(s, nnzb);
    } else {
        // Rows of twice the mean are cut too up to 64 block rows if all rows run at once (33 x 2240, block 64, of which 1155 do not, 19.8 / 20.9),
        // above if at most two rounds of them run and the mean is 7 blocks: short rows are no chain to speak of, and helpers
        // that find nothing to do are not free (3 x 5472, block 32, 6.8 blocks a row, 13.9 / 14.5; 9 x 4064, 6.0, 14.6 / 14.9).  The others, 40 of 100 shapes
        // of 65 to 255 block rows, take 0.57 to 1.01 of the time uncut, 0.83 on average: 2 x 10176, block 64, 17.9 blocks a row, 40.2 / 22.9; 4 x 7488,
        // block 32, 43.7, 48.0 / 30.5; of two rounds 9 x 7424, block 64, 20.5, 45.3 / 39.5, 24 x 3424, block 32, 20.4, 31.6 / 27.7, 16 x 6528, block 64, 40.7 / 39.4.
        const long long all = (long long)s.BH * s.nb, at_once = fwd_resident(s.bs);
        const bool short_too = s.nb <= 64 ? all <= at_once : all <= 2 * at_once && nnzb >= 7 * s.nb;
        decide(s, nnzb, (long long)s.BH * nnzb / at_once, short_too);
        // 128 in all, those that find nothing to do are not free: 16 x 4096, block 64, 12.4 -> 12.8 us with 256, 16 x 5248 17.8 -> 19.3, 17 x 2688, block 32, 14.7 ->
        // 16.1.  256 with block 32 where rows go in rounds: many pieces of the mean in place of few of twice the mean are two and more a helper then,
        // 25 x 3424 23.1 -> 17.4 (pieces of twice the mean 18.6), 16 x 7008 32.4 -> 25.9 (28.2).  Up to 256 block rows at most 16 a head, 4 x 4992,
        // block 32, 14.1 / 14.7 with 31; above, long rows are longer: 2 x 23168, block 64, 39.3 / 26.8 (16 / 31).
        const int in_all = s.bs == 32 && all > at_once ? 256 : 128;
        helpers = s.BH < in_all ? in_all / s.BH : 1;
        if (helpers > 16 && s.nb <= 256) helpers = 16;
        if (helpers >= slots) helpers = slots > 0 ? slots - 1 : 0;
        groups = (s.BH * helpers + 7) & ~7;
        if ((long long)s.BH * s.nb + groups > 0x7fffffffll) slots = helpers = groups = 0;   // workgroups of a launch
    }
    if (!s.fwd_room) return;
    counters = static_cast<unsigned long long*>(s.fwd_room);
    parts = reinterpret_cast<float*>(static_cast<char*>(s.fwd_room) + counter_bytes(s.BH));
}

// ------------------------------------------------------------------------------------------------
// launcher (called by the dispatch in attn_kernels.hip)
// ------------------------------------------------------------------------------------------------
template <int BS>
hipError_t fwd_bf16(const AttnShape& s, const void* Q, const void* K, const void* V, void* O, float* LSE,
                    const int* row_ptr, const int* col_idx, int nnzb, hipStream_t st) {
    const int total = s.nb * s.BH;
    RowCut cut;
    if (s.fwd_room) cut = RowCut(s, nnzb);
    // Dealt (deal_heads) where a head's workgroups share tiles and are many; finding its row costs a workgroup a quarter of a
    // microsecond.  As they lie / dealt: 16 heads x 4096, 8 %, 14.3 / 13.2 us, 28 x 1600 12.4 / 10.7, 9 x 6784 13.4 / 12.2; fewer, 24 x 1088, block 64,
    // 5.7 / 6.0, 6 x 5376 7.4 / 7.7, 28 x 768, block 32, 5.1 / 5.6; the diagonal alone, 21 x 1984 5.0 / 5.6.  Longest first where more rows follow than run at once, or a row is six blocks on
    // average: long ones then spread over the compute units.  Dealt / so: 6 x 7680, block 64, 30.3 / 26.0, 5 x 9472 26.3 / 22.7, 28 x 1984, block 32, 14.6 / 13.3; shorter
    // rows, 16 x 4096 13.2 / 13.7, 64 x 1024, block 32, 10.2 / 10.5; up to 256 rows, one or none a compute unit, they are no faster.
    // As they lie, head by head, also where short rows are so many that the order within a head hardly matters and the heads of an XCD do not fit its
    // L2 (by length / so): block 32, 88 x 2880, 3 blocks a row, 28.3 / 24.4, 56 x 4544, 4.4, 30.7 / 25.3; 96 x 2624, 6.9, 35.3 / 38.9; 56 x 1184 (2072 rows) 10.8 / 11.1;
    // block 64, 72 x 3520, 1.8, 24.9 / 22.1, 32 x 4544, 3.0, 18.9 / 17.6; 40 x 3712, 4.5, 21.1 / 22.1; 32 x 2880 (1440 rows) 12.8 / 13.5.
    const bool short_rows = BS == 32 ? nnzb < 6 * s.nb && 4 * total >= 5 * fwd_resident(BS) : nnzb < 4 * s.nb && total >= 2 * fwd_resident(BS);
    const RowOrder order = !short_rows && (total > fwd_resident(BS) || (total > 256 && nnzb >= 6 * s.nb)) ? kByLength
                           : !short_rows && total > (BS == 64 ? 512 : 768) && 2 * nnzb >= 3 * s.nb        ? kDealt
                                                                                                             : kAsTheyLie;
    const long long grid = cut.groups + (order == kAsTheyLie ? total : dealt(s.BH, s.nb, false));
    if (grid > 0x7fffffffll) return hipErrorInvalidValue;
    auto launch = [&](auto kernel, auto at, auto cut_arg) {
        kernel<<<dim3((unsigned)grid), dim3(BS * 4), 0, st>>>(
            static_cast<const bf16_t*>(Q), static_cast<const bf16_t*>(K), static_cast<const bf16_t*>(V),
            static_cast<bf16_t*>(O), LSE, row_ptr, col_idx, at, cut_arg, s.L, s.nb, s.BH, order, s.scale * kLog2e,
            s.paper_denom);
    };
    if (s.heads_beside) {
        if (cut.slots) launch(attn_fwd_bf16_kernel<BS, true, true>, HeadRows<true>{s.heads_beside}, cut);
        else launch(attn_fwd_bf16_kernel<BS, true, false>, HeadRows<true>{s.heads_beside}, NoCut{});
    } else {
        if (cut.slots) launch(attn_fwd_bf16_kernel<BS, false, true>, HeadRows<false>{0}, cut);
        else launch(attn_fwd_bf16_kernel<BS, false, false>, HeadRows<false>{0}, NoCut{});
    }
    return hipGetLastError();
}

template hipError_t fwd_bf16<32>(const AttnShape&, const void*, const void*, const void*, void*, float*,
                                 const int*, const int*, int, hipStream_t);
template hipError_t fwd_bf16<64>(const AttnShape&, const void*, const void*, const void*, void*, float*,
                                 const int*, const int*, int, hipStream_t);

}  // namespace spion
