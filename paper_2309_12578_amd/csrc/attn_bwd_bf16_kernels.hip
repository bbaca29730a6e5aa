// bf16 block-sparse attention backward (the gradient of Eq. 5) tuned for gfx950, block size 32 or 64.
//
// One launch computes dQ, dK and dV.  Its grid holds two kinds of workgroups:
//   - query side: one workgroup per (head, block row I) walks the kept blocks of the row (BSR),
//     delta = rowsum(dO .* O), S^T and dP^T per block, dQ_I accumulated in registers;
//   - key side: one workgroup per (head, work item), a work item being a chunk of the kept rows of
//     one block column (BSC); S and dP per block, dK_J and dV_J accumulated in registers.
// The two sides share no data: the key side computes delta for the query rows of every block it
// visits from the O and dO tiles it loads (an MFMA whose diagonal is the row-wise dot product), so
// neither waits for the other, and workgroups of both kinds fill the machine together.  Block
// columns with more kept rows than one work item takes are cut into chunks that write fp32 partial
// tiles; the last of a column's chunks to arrive adds them up in chunk order: gradients are bit-reproducible.
//
// Every workgroup finds its own work from the index: there is no work list to build, so nothing in
// the grid depends on another workgroup.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "attn_bf16_tiles.h"
#include "attn_common.h"
#include "attn_key_items.h"
#include "spion_internal.h"

namespace spion {

// Own loads landed (up to `younger` younger ones may stay in flight: 0 or 4), previous LDS reads done,
// then meet the other waves.  A bare barrier: the fences of __syncthreads would wait for every load
// in flight, the prefetched blocks included.
__device__ __forceinline__ void tiles_ready(bool four_younger_in_flight) {
    if (four_younger_in_flight) __builtin_amdgcn_s_waitcnt(kWaitVm4);
    else __builtin_amdgcn_s_waitcnt(kWaitVm0);
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// ------------------------------------------------------------------------------------------------
// Grid layout.  Per head: pieces of long rows (CUT), key items [0, w_first), then the nb block rows, then key items
// [w_first, w_max); the long chunks of split columns come early so that they start first, the rows and
// the short columns fill in behind them.  The heads as deal_heads() has them, items of an XCD's heads interleaved; only block rows
// that do not go by length follow head by head where XCDs have whole heads.
// n_key_a / n_rows / n_key_c are the per-head counts of the three groups present in this launch
// (a group is absent when only one side is requested).  w_first leaves room for a quarter of the columns
// besides the chunks, the longest of them: unsplit columns of more than 8 rows that came last ran on alone (64 heads x 1024,
// block 32, 4.8 blocks a row: 31.6 -> 26.5 us; a sixth or a third of the columns measure like a quarter).  With sort_rows
// the rows go by length.
// ------------------------------------------------------------------------------------------------
template <int BS, bool BESIDE, bool CUT>
__global__ __launch_bounds__(BS * 4) void attn_bwd_bf16_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
    const bf16_t* __restrict__ O, const bf16_t* __restrict__ dO, const float* __restrict__ LSE,
    bf16_t* __restrict__ dQ, bf16_t* __restrict__ dK, bf16_t* __restrict__ dV,
    const int* __restrict__ row_ptr, const int* __restrict__ col_idx, const int* __restrict__ col_ptr,
    const int* __restrict__ row_idx, float* __restrict__ partial, unsigned long long* __restrict__ counters,
    unsigned long long tag, HeadRows<BESIDE> at, CutOf<CUT> cut, int n_slots, int BH, int L, int nb, int n_key_a,
    int n_rows, int n_key_c, int w_first, int chunk, int sort_rows, int finest, int few, float scale, float scale_log2) {
    constexpr int NT = BS / 16;   // 16-row tiles per block = waves per workgroup
    // Separate objects, so that the compiler can tell a read of one tile from a load in flight into
    // another and does not wait for it.  Query side: {ta, tb} hold {K, V} of a block, three stages
    // (0, 1, and {tc0, tc1}).  Key side: {ta, tb, tc} hold {Q, dO, O} of a block row, two stages.
    __shared__ __attribute__((aligned(16))) bf16_t ta0[BS * kD], tb0[BS * kD], tc0[BS * kD];
    __shared__ __attribute__((aligned(16))) bf16_t ta1[BS * kD], tb1[BS * kD], tc1[BS * kD];
    __shared__ __attribute__((aligned(16))) float lse0[BS], del0[BS], lse1[BS], del1[BS];

    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const SwzLane sl(r, g);
    const int in_row = at.in_row(), out_row = at.out_row();   // elements between rows of Q, K, V and of O, dO
    const TileLoadLane tl(wave, lane, in_row);

    // which workgroup am I
    const ItemOfHead dealt_to = deal_heads(blockIdx.x, BH, few != 0);
    int bh = dealt_to.head;
    bool key_side = false;
    int idx = dealt_to.item;   // work item (key side) or block row (query side)
    [[maybe_unused]] RowPieces cuts = {0, 1, 0, 0};
    [[maybe_unused]] int piece = 0;
    bool helper = false;
    if constexpr (CUT) {
        helper = idx < cut.helpers;
        if (!helper) idx -= cut.helpers;
    }
    if (helper) {
        if constexpr (CUT) {
            cuts = row_pieces<false>(row_ptr, nb, cut, idx, lane);
            if (cuts.row < 0) return;
            piece = idx - cuts.first + 1;
            idx = cuts.row;
        }
    } else if (idx < n_key_a) {
        key_side = true;
    } else if (idx < n_key_a + n_rows) {
        idx -= n_key_a;
        if (sort_rows) {
            idx = row_by_length(row_ptr, nb, idx, lane);
        } else if ((BH & 7) == 0) {   // whole heads: one after the other
            const int hpx = BH >> 3, first = (blockIdx.x & 7) * hpx, l = idx * hpx + bh - first;
            bh = first + l / nb;
            idx = l % nb;
        }
    } else {
        idx -= n_key_a + n_rows;
        if (idx >= n_key_c) return;
        key_side = true;
        idx += w_first;
    }
    const size_t head = at.in_head(bh, L), out_head = at.out_head(bh, L);
    const size_t vec = (size_t)bh * L;

    if (!key_side) {
        // ========================================================================================
        // query side: block row I, K / V tiles three stages deep (block it + 2 loads while block it
        // is multiplied)
        // ========================================================================================
        const int I = idx;
        const int qrow = I * BS + wave * 16 + r;
        auto issue = [&](bf16_t* kt, bf16_t* vt, int J) {
            tile_load_async(K + head + (size_t)J * BS * in_row, kt, wave, tl);
            tile_load_async(V + head + (size_t)J * BS * in_row, vt, wave, tl);
        };
        if (!helper) issue(ta0, tb0, I);   // the diagonal block, before any index is known
        bf16x8 qf[2], dof[2], of[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const size_t out = out_head + (size_t)qrow * out_row + c * 32 + g * 8;
            qf[c] = *reinterpret_cast<const bf16x8*>(Q + head + (size_t)qrow * in_row + c * 32 + g * 8);
            dof[c] = *reinterpret_cast<const bf16x8*>(dO + out);
            of[c] = *reinterpret_cast<const bf16x8*>(O + out);
        }
        const float lse2 = LSE[vec + qrow] * kLog2e;
        int jb = row_ptr[I], n = row_ptr[I + 1] - jb;
        if constexpr (CUT) if (n > cut.longest) {
            if (!helper) cuts = row_pieces<true>(row_ptr, nb, cut, I, lane);
            const int from = piece * n / cuts.count;
            n = (piece + 1) * n / cuts.count - from;
            jb += from;
        }
        const int last = n > 0 ? n - 1 : 0;
        const int* cols = col_idx + jb;
        int first[8];
        int pd = n > 0 ? find_in_row(cols, n, I, first) : -1;
        if (helper) pd = -1;   // in index order, the diagonal block where it comes
        // block visited at step t (clamped reads stay inside this row's entries; an empty row reads nothing)
        auto col_at = [&](int t) {
            const int j = walk_index(t < last ? t : last, pd);
            return j < 8 ? pick8(first, j) : cols[j];
        };
        if (pd < 0 && n > 0) {
            // no diagonal block in this row (piece): once everyone's early load has landed, load block 0 over it
            if (!helper) {
                __builtin_amdgcn_s_waitcnt(kWaitVm0);
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            }
            issue(ta0, tb0, first[0]);
        }
        // the second block goes out as soon as its index is known (a one-block row loads its block
        // twice: keeps the wait of step 0 uniform); it is the youngest load at step 0
        if (n > 0) issue(ta1, tb1, col_at(1));
        int Jnext = n > 0 ? col_at(2) : 0;   // block of step it + 2

        float delta = 0.f;
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int e = 0; e < 8; ++e) delta = fmaf((float)dof[c][e], (float)of[c][e], delta);
        delta = group_sum(delta);

        f32x4 dq[4];
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) dq[dt] = f32x4{0.f, 0.f, 0.f, 0.f};

        auto step = [&](const bf16_t* kt, const bf16_t* vt, bf16_t* tk, bf16_t* tv, int it) {
            // in flight here: block `it` and block it + 1 (the four youngest loads; at step 0 whatever the
            // prologue loaded before them is waited for as well)
            tiles_ready(it + 1 < n || it == 0);
            if (it + 2 < n) issue(tk, tv, Jnext);
            Jnext = col_at(it + 3);
            // all K and V fragments are requested up front; the transposed K operands of the dQ product do
            // not depend on dS and are requested before the exponentials, so that they land under them
            bf16x8 kfr[NT][2], vfr[NT][2];
#pragma unroll
            for (int kt16 = 0; kt16 < NT; ++kt16)
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    kfr[kt16][c] = *reinterpret_cast<const bf16x8*>(kt + kt16 * 16 * kD + sl.frag[c]);
                    vfr[kt16][c] = *reinterpret_cast<const bf16x8*>(vt + kt16 * 16 * kD + sl.frag[c]);
                }
            f32x4 s[NT], dp[NT];
#pragma unroll
            for (int kt16 = 0; kt16 < NT; ++kt16) {
                // dP - delta comes out of the MFMA: the accumulator starts at -delta instead of 0
                s[kt16] = f32x4{0.f, 0.f, 0.f, 0.f};
                dp[kt16] = f32x4{-delta, -delta, -delta, -delta};
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    s[kt16] = mma_d(s[kt16], kfr[kt16][c], qf[c]);      // S^T = K Q^T
                    dp[kt16] = mma_d(dp[kt16], vfr[kt16][c], dof[c]);   // dP^T = V dO^T
                }
            }
            constexpr int NM = (BS / 32) * 4;
            bf16x8 kop[NM];
#pragma unroll
            for (int j = 0; j < NM; ++j) {
                const int o = sl.tr(j & 3) + (j >> 2) * 32 * kD;
                kop[j] = join(lds_read_tr(kt + o), lds_read_tr(kt + 16 * kD + o));
            }
            __builtin_amdgcn_sched_barrier(0);
            bf16x4 dsq[NT];
#pragma unroll
            for (int kt16 = 0; kt16 < NT; ++kt16) {
                f32x4 ds;
#pragma unroll
                for (int i = 0; i < 4; ++i) ds[i] = fast_exp2(fmaf(s[kt16][i], scale_log2, -lse2)) * dp[kt16][i];
                dsq[kt16] = to_quad<bf16_t>(ds);
            }
#pragma unroll
            for (int j = 0; j < NM; ++j) {
                const int pc = j >> 2;
                dq[j & 3] = mma_d(dq[j & 3], kop[j], join(dsq[2 * pc], dsq[2 * pc + 1]));   // dQ^T[d][query] += K^T dS^T
            }
        };

        for (int it = 0; it < n; it += 3) {
            step(ta0, tb0, tc0, tc1, it);
            if (it + 1 < n) step(ta1, tb1, ta0, tb0, it + 1);
            if (it + 2 < n) step(tc0, tc1, ta1, tb1, it + 2);
        }
        // an empty row never waited for its early load: it must land before this workgroup's LDS is freed
        __builtin_amdgcn_s_waitcnt(kWaitVm0);
        if constexpr (CUT) if (cuts.count > 1) {   // a long row in pieces: see attn_bf16_tiles.h
            constexpr int kPart = 8 * 128;   // eight pairs a lane
            const size_t first_slot = (size_t)bh * cut.slots + cuts.slot;
            float* const parts = cut.parts + (first_slot * NT + wave) * kPart + lane * 2;
            float* const mine = parts + (size_t)piece * NT * kPart;
#pragma unroll
            for (int i = 0; i < 8; ++i) put_shared(mine + i * 128, dq[i / 2][i % 2 * 2], dq[i / 2][i % 2 * 2 + 1]);
            if (!last_to_arrive(cut.counters + first_slot, cut.tag, cuts.count, reinterpret_cast<int*>(lse0))) return;
#pragma unroll
            for (int dt = 0; dt < 4; ++dt) dq[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
            for (int c = 0; c < cuts.count; ++c) {
                float2 v[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) v[i] = get_shared(parts + (size_t)c * NT * kPart + i * 128);
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    dq[i / 2][i % 2 * 2] += v[i].x;
                    dq[i / 2][i % 2 * 2 + 1] += v[i].y;
                }
            }
        }
        // Through a tile nobody reads any more: every wave is past the barrier of the last step, so only
        // the last block's stage can still be read; the wave's own 2 KB of any other tile were only ever
        // written by the wave's own loads, which have all landed.
        bf16_t* patch = (n % 3 == 1 ? ta1 : ta0) + wave * (16 * kD);   // last stage: (n - 1) % 3
        store_rows_coalesced(patch, dQ + head + (size_t)(I * BS + wave * 16) * in_row, in_row, dq, scale, lane);
        return;
    }

    // ============================================================================================
    // key side: work item idx of head bh.  {Q, dO, O} tiles and LSE of a block row in two stages.
    // ============================================================================================
    const KeyItem item = key_item_lookup(col_ptr, nb, chunk, finest, idx, lane);
    if (item.J < 0) return;
    const int J = item.J, n = item.ke - item.kb, slot = item.slot;
    const int krow = J * BS + wave * 16 + r;
    const int last = n > 0 ? n - 1 : 0;
    // the item's block rows, one per lane (an item has at most 64 of them): read once, so that
    // no scalar load is in flight inside the steps (scalar loads return out of order, and while one is
    // outstanding every wait for an LDS read has to wait for all of them)
    static_assert(kChunkMax <= 64, "a key-side work item must fit one wave's lanes");
    const int rows_v = n > 0 ? row_idx[item.kb + (lane < last ? lane : last)] : 0;
    auto row_at = [&](int t) { return __builtin_amdgcn_readlane(rows_v, t < last ? t : last); };

    const TileLoadLane tlo(wave, lane, out_row);
    // six tile loads per wave, plus one 4-byte-per-lane load of LSE in wave 0
    auto load_q = [&](bf16_t* qt, int I) { tile_load_async(Q + head + (size_t)I * BS * in_row, qt, wave, tl); };
    auto load_do = [&](bf16_t* dt_, int I) { tile_load_async(dO + out_head + (size_t)I * BS * out_row, dt_, wave, tlo); };
    auto load_o = [&](bf16_t* ot, float* lse_s, int I) {
        tile_load_async(O + out_head + (size_t)I * BS * out_row, ot, wave, tlo);
        if (wave == 0 && lane < BS)
            __builtin_amdgcn_global_load_lds(LSE + vec + (size_t)I * BS + lane, (lds_void_ptr)lse_s, 4, 0, 0);
    };
    int Inext = 0;   // block row of step it + 1
    if (n > 0) {
        load_q(ta0, row_at(0));
        load_do(tb0, row_at(0));
        load_o(tc0, lse0, row_at(0));
        Inext = row_at(1);
    }
    // owned K / V fragments (step 0 waits for everything issued up to here)
    bf16x8 kf[2], vf[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const size_t off = head + (size_t)krow * in_row + c * 32 + g * 8;
        kf[c] = *reinterpret_cast<const bf16x8*>(K + off);
        vf[c] = *reinterpret_cast<const bf16x8*>(V + off);
    }
    f32x4 dk[4], dv[4];
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) {
        dk[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
        dv[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    auto step = [&](const bf16_t* qt, const bf16_t* dt_, const bf16_t* ot, float* lse_s, float* del_s,
                    bf16_t* nq, bf16_t* nd, bf16_t* no, float* nlse, int it) {
        // everyone's part of block `it` has landed and the other stage is no longer read
        tiles_ready(false);
        // Block 64: the next tiles are requested in three places.  All at once they hold every wave of the workgroup up until the
        // memory pipeline has taken 24 KB: key side of 32 heads x 4096, 13 and 38 blocks a row, 83.2 -> 80.4 and 213.7 -> 205.9 us; with
        // block 32, half of that, the steps are too short for it (62.7 -> 63.5), and for finding the next block row as late (3 heads x 992 14.9 -> 14.6).
        constexpr bool kSpread = BS == 64;
        const bool more = it + 1 < n;
        if (more) {
            load_q(nq, Inext);
            if (!kSpread) {
                load_do(nd, Inext);
                load_o(no, nlse, Inext);
            }
        }
        if (!kSpread) Inext = row_at(it + 2);
        // delta of the 16 query rows 16 wave .. + 15: the diagonal of dO O^T; stored negated, it seeds
        // the dP accumulators below.  Wave 0 also turns LSE into log2 units.
        {
            f32x4 dd = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int off = wave * 16 * kD + sl.frag[c];
                dd = mma_d(dd, *reinterpret_cast<const bf16x8*>(dt_ + off), *reinterpret_cast<const bf16x8*>(ot + off));
            }
            // lane (r, g) holds (dO O^T)[4 g + i][r]: the diagonal entry of row r sits in lane group r / 4
            const float a = (r & 1) ? dd[1] : dd[0], b = (r & 1) ? dd[3] : dd[2];
            if (g == (r >> 2)) del_s[wave * 16 + r] = -((r & 2) ? b : a);
            if (wave == 0 && lane < BS) lse_s[lane] *= kLog2e;
        }
        lds_barrier();
        if (kSpread && more) load_do(nd, Inext);
        // 32 query rows at a time: S and dP of two 16-row tiles, then their share of dV and dK, so that
        // only two tiles' worth of P and dS are live; LDS operands are requested one MFMA group ahead
        bf16x8 fq[2], fd[2];
        auto frags = [&](int qt16) {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                fq[c] = *reinterpret_cast<const bf16x8*>(qt + qt16 * 16 * kD + sl.frag[c]);
                fd[c] = *reinterpret_cast<const bf16x8*>(dt_ + qt16 * 16 * kD + sl.frag[c]);
            }
        };
        auto opnd = [&](int pc, int j) {   // transposed operand of MFMA j of this 32-row group
            const bf16_t* tile = (j & 1) ? qt : dt_;
            const int o = sl.tr(j >> 1) + pc * 32 * kD;
            return join(lds_read_tr(tile + o), lds_read_tr(tile + 16 * kD + o));
        };
        frags(0);
#pragma unroll
        for (int pc = 0; pc < NT / 2; ++pc) {
            bf16x4 pq[2], dsq[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int qt16 = 2 * pc + h;
                f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f};
                f32x4 dp = *reinterpret_cast<const f32x4*>(&del_s[qt16 * 16 + 4 * g]);   // -delta: the MFMA returns dP - delta
                const f32x4 lse4 = *reinterpret_cast<const f32x4*>(&lse_s[qt16 * 16 + 4 * g]);   // log2 units
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    s = mma_d(s, fq[c], kf[c]);     // S = Q K^T
                    dp = mma_d(dp, fd[c], vf[c]);   // dP = dO V^T
                }
                __builtin_amdgcn_sched_barrier(0);
                if (qt16 + 1 < NT) frags(qt16 + 1);   // lands while the exponentials below run
                __builtin_amdgcn_sched_barrier(0);
                f32x4 p, ds;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    p[i] = fast_exp2(fmaf(s[i], scale_log2, -lse4[i]));
                    ds[i] = p[i] * dp[i];
                }
                pq[h] = to_quad<bf16_t>(p);
                dsq[h] = to_quad<bf16_t>(ds);
            }
            if (kSpread && pc == 0 && more) load_o(no, nlse, Inext);
            // dV^T[d][key] += dO^T P and dK^T[d][key] += Q^T dS for these 32 rows, interleaved
            const bf16x8 pf = join(pq[0], pq[1]), dsf = join(dsq[0], dsq[1]);
            bf16x8 ring[2];
            ring[0] = opnd(pc, 0);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if (j + 1 < 8) ring[(j + 1) & 1] = opnd(pc, j + 1);
                __builtin_amdgcn_sched_barrier(0);
                if (j & 1) dk[j >> 1] = mma_d(dk[j >> 1], ring[j & 1], dsf);
                else dv[j >> 1] = mma_d(dv[j >> 1], ring[j & 1], pf);
            }
        }
        if (kSpread) Inext = row_at(it + 2);
    };

    for (int it = 0; it < n; it += 2) {
        step(ta0, tb0, tc0, lse0, del0, ta1, tb1, tc1, lse1, it);
        if (it + 1 < n) step(ta1, tb1, tc1, lse1, del1, ta0, tb0, tc0, lse0, it + 1);
    }
    __builtin_amdgcn_s_waitcnt(kWaitVm0);   // the owned fragments of a column without kept rows

    if (slot >= 0) {
        // A chunk of a column: its accumulators as pairs per lane, [head][slot][wave][dK | dV]; the last of the column's
        // chunks to arrive adds all of them up, in their order.  A launch of its own for the sums cost its 4.5 us and a gap
        // before it: 4 x 4 heads x 4096, block 64, 8 %, forward and backward 52.3 -> 49.6 us; 64 x 1024, block 32, 15 %, 39.1 -> 36.4.
        constexpr int kPart = 16 * 128;
        float* const parts = partial + (((size_t)bh * n_slots + item.first) * NT + wave) * kPart + lane * 2;
        float* const mine = parts + (size_t)(slot - item.first) * NT * kPart;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            put_shared(mine + i * 128, dk[i / 2][i % 2 * 2], dk[i / 2][i % 2 * 2 + 1]);
            put_shared(mine + (8 + i) * 128, dv[i / 2][i % 2 * 2], dv[i / 2][i % 2 * 2 + 1]);
        }
        if (!last_to_arrive(counters + (size_t)bh * n_slots + item.first, tag, item.count, reinterpret_cast<int*>(lse0)))
            return;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) {
            dk[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
            dv[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        for (int c = 0; c < item.count; ++c) {
            float2 v[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) v[i] = get_shared(parts + (size_t)c * NT * kPart + i * 128);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                dk[i / 2][i % 2 * 2] += v[i].x;
                dk[i / 2][i % 2 * 2 + 1] += v[i].y;
                dv[i / 2][i % 2 * 2] += v[8 + i].x;
                dv[i / 2][i % 2 * 2 + 1] += v[8 + i].y;
            }
        }
    }
    // Through the stage the last block did not use: every wave is past the first barrier of the last
    // step, i.e. done reading that stage, no load targets it any more, and the only loads that ever
    // touched this wave's 2 KB of its tiles were the wave's own.
    const bool odd = (n & 1) != 0;   // last block in stage 0 -> stage 1 is free
    bf16_t* pa = (odd ? ta1 : ta0) + wave * (16 * kD);
    bf16_t* pb = (odd ? tb1 : tb0) + wave * (16 * kD);
    const size_t row0 = head + (size_t)(J * BS + wave * 16) * in_row;
    store_rows_coalesced(pa, dK + row0, in_row, dk, scale, lane);
    store_rows_coalesced(pb, dV + row0, in_row, dv, 1.f, lane);
}

// The query side's rows that are cut: the forward's rule, with the steps of both sides (so few heads, and a helper for each
// piece).  Backward, us, uncut / cut / a pattern without long rows: 8 heads x 8192, block 32, rows of 121 blocks, 73.5 / 46.7 / 47.5;
// 4 x 16384, block 64, 112 / 70.5 / 70.3; 4 x 8192, block 64, rows of 71, 65.3 / 39.5 / 40.2; 1 x 4096, block 32, 21.1 / 17.8 / 17.9.
// From a mean of 8 blocks on, rows of twice the mean: 1 x 10176, block 64, 21.3 blocks a row, 67.3 / 32.9; 3 x 8128, block 32, 33.8, 74.2 / 50.0; 2 x 4800, block
// 64, 10.5, 28.6 / 25.0; of 37 such shapes none takes longer than 1.015 of the time.  Below, 0.99 to 1.03 (16 x 3648, block 64, 5.3 blocks, 31.1 / 32.0).
static void decide_row_cut(RowCut& cut, const AttnShape& s, int nnzb) {
    cut.decide(s, nnzb, bwd_steps_per_slot(s.BH, s.bs, s.nb, nnzb), nnzb >= 8 * s.nb);
}
int bwd_bf16_row_slots(const AttnShape& s, int nnzb) {
    RowCut cut;
    decide_row_cut(cut, s, nnzb);
    return cut.slots;
}
static RowCut row_cut(const AttnShape& s, const BwdWorkspace& ws, void* workspace) {
    RowCut cut;
    if (!s.bwd_room) return cut;
    decide_row_cut(cut, s, ws.nnzb);
    if (cut.slots == 0) return cut;
    cut.helpers = cut.slots - 1;
    if ((long long)s.BH * (cut.helpers + s.nb + ws.w_max) > 0x7fffffffll) return RowCut{};   // workgroups of a launch
    cut.counters = reinterpret_cast<unsigned long long*>(static_cast<char*>(workspace) + ws.total);
    cut.parts = reinterpret_cast<float*>(static_cast<char*>(workspace) + ws.row_parts);
    return cut;
}

// ------------------------------------------------------------------------------------------------
// launcher (called by the dispatch in attn_kernels.hip).  phases: bit 0 query side, bit 1 key side.
// ------------------------------------------------------------------------------------------------
template <int BS>
hipError_t bwd_bf16(const AttnShape& s, const void* Q, const void* K, const void* V, const void* O,
                    const void* dO, const float* LSE, void* dQ, void* dK, void* dV, const int* row_ptr,
                    const int* col_idx, const int* col_ptr, const int* row_idx, const BwdWorkspace& ws,
                    void* workspace, hipStream_t st) {
    const bool rows = (s.bwd_phases & 1) != 0, keys = (s.bwd_phases & 2) != 0;
    const int n_key_a = keys ? ws.w_first : 0, n_rows = rows ? s.nb : 0, n_key_c = keys ? ws.w_max - ws.w_first : 0;
    const RowCut cut = rows ? row_cut(s, ws, workspace) : RowCut{};
    const long long items = cut.helpers + n_key_a + n_rows + n_key_c, total = s.BH * items;
    const int few = total <= 512;   // deal_heads()
    const long long grid = dealt(s.BH, items, few != 0);
    if (grid > 0x7fffffffll) return hipErrorInvalidValue;
    if (total > 0) {
        // A row of more than twice the mean that starts late runs alone at the end; finding the rows by length
        // costs each about half a step.  Worth it where such rows are long, by themselves (a mean of 6
        // blocks) or can be against the steps a slot has to do: 16 heads x 8192, block 32, 12.8 blocks a row 130 -> 98 us,
        // 64 heads x 1024, 4.8 blocks a row 26.9 -> 28.3 us.
        const int sort_rows = total > bwd_resident(BS) && (ws.nnzb >= 6 * s.nb || s.nb >= 8 * bwd_steps_per_slot(s.BH, BS, s.nb, ws.nnzb));
        // Order of the unsplit columns.  As they lie while at most one in three places is taken: finding them by length costs 0.2 to 0.4 us (2 x 512,
        // block 32, 8.6 / 9.0, 5 x 896 5.6 / 5.9); with more, long ones should not meet on a compute unit (block 64, 7 x 1472, of 340 workgroups, 8.3 / 7.6,
        // 2 x 9472 10.5 / 9.6).  The more rounds, the less their exact order counts and the more that columns beside each other, which share tiles, follow each
        // other: lengths in units of a quarter of the mean, of 2 and of 4 blocks: 57 x 1472, block 64, of 3.5 rounds, 32.6 / 30.8 / 32.0, 27 x 1728 (1.9)
        // 17.0 / 16.9 / 18.2; 64 x 2880 (7.6) 49.3 / 48.9 / 45.3, 39 x 3456 (5.6) 43.6 / 42.4 / 41.6; block 32, 88 x 2880 (11) 76.8 / 74.0 / 72.5, 95 x 1664 (6.5)
        // 52.8 / 50.7 / 49.7.  As they lie 64 x 2048, block 64, takes 55.0 us (44), 32 x 1280, block 32, 20.9 (16.0).
        const long long at_once = bwd_resident(BS);
        const int finest = 3 * total <= at_once ? 0 : total <= at_once ? 1 : total <= 4 * at_once ? 2 : 4;
        auto launch = [&](auto kernel, auto at, auto cut_arg) {
            kernel<<<dim3((unsigned)grid), dim3(BS * 4), 0, st>>>(
                static_cast<const bf16_t*>(Q), static_cast<const bf16_t*>(K), static_cast<const bf16_t*>(V),
                static_cast<const bf16_t*>(O), static_cast<const bf16_t*>(dO), LSE, static_cast<bf16_t*>(dQ),
                static_cast<bf16_t*>(dK), static_cast<bf16_t*>(dV), row_ptr, col_idx, col_ptr, row_idx,
                reinterpret_cast<float*>(static_cast<char*>(workspace) + ws.counter_bytes),
                static_cast<unsigned long long*>(workspace), s.tag, at, cut_arg,
                ws.n_slots, s.BH, s.L, s.nb, n_key_a, n_rows, n_key_c, ws.w_first, ws.chunk, sort_rows, finest, few, s.scale, s.scale * kLog2e);
        };
        if (s.heads_beside) {
            if (cut.slots) launch(attn_bwd_bf16_kernel<BS, true, true>, HeadRows<true>{s.heads_beside}, cut);
            else launch(attn_bwd_bf16_kernel<BS, true, false>, HeadRows<true>{s.heads_beside}, NoCut{});
        } else {
            if (cut.slots) launch(attn_bwd_bf16_kernel<BS, false, true>, HeadRows<false>{0}, cut);
            else launch(attn_bwd_bf16_kernel<BS, false, false>, HeadRows<false>{0}, NoCut{});
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template hipError_t bwd_bf16<32>(const AttnShape&, const void*, const void*, const void*, const void*,
                                 const void*, const float*, void*, void*, void*, const int*, const int*,
                                 const int*, const int*, const BwdWorkspace&, void*, hipStream_t);
template hipError_t bwd_bf16<64>(const AttnShape&, const void*, const void*, const void*, const void*,
                                 const void*, const float*, void*, void*, void*, const int*, const int*,
                                 const int*, const int*, const BwdWorkspace&, void*, hipStream_t);

}  // namespace spion
