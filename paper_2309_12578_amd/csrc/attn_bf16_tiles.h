// Tile movement and fragment helpers shared by the tuned bf16 attention kernels (block size 32 or 64).
//   - tiles travel HBM -> LDS through the memory pipeline (buffer loads into LDS): no staging registers,
//     no LDS stores;
//   - tiles stay row-major in LDS, 16-byte slots permuted per row so that no read conflicts;
//     operands that must be read along the row index come out of the same tile through the LDS
//     transpose read (ds_read_b64_tr_b16: 16 lanes fetch a 4 x 16 patch, each receives a column).
#ifndef SPION_ATTN_BF16_TILES_H_
#define SPION_ATTN_BF16_TILES_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/spion.h"
#include "attn_common.h"
#include "spion_internal.h"

namespace spion {

__device__ __forceinline__ bf16x4 lds_read_tr(const bf16_t* p) {
    typedef bf16x4 __attribute__((address_space(3))) * lds_ptr;
    return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_ptr)p);
}

// ------------------------------------------------------------------------------------------------
// Tiles loaded by the memory pipeline straight into LDS (16 B per lane; a wave
// instruction fills 1 KB of consecutive LDS, lane l at byte 16 l).  Rows are 128 B apart with no
// padding, so the 16-byte slots of a row are permuted instead: slot s of row `row` holds the row's
// chunk s ^ swz(row), swz = 2 * ((row >> 1) & 3).  Measured with SQ_LDS_BANK_CONFLICT: neither the
// 16-byte fragment reads (lane = row) nor the transpose reads (8 rows x 32 B per half wave) conflict
// in this layout.  (A 16-byte read is served 16 lanes at a time, lanes 0-7 together with lanes of the
// upper half of a neighbouring group of 16: a permutation that also used bit 3 of the row conflicted.)
// ------------------------------------------------------------------------------------------------
typedef __attribute__((address_space(3))) void* lds_void_ptr;

// Where the 64 elements of a row of head bh = b H + h are.  Separate tensors: Q, K, V, O and their gradients are
// [B, H, L, 64].  BESIDE: as the projections of a sub-layer make and take them, Q | K | V (and their gradients) in the
// rows of one [B, L, 3, H, 64] tensor, O and dO in those of [B, L, H, 64].  A row is one 128-byte line either way,
// and the kernels take as long: what a head split and a merge around them cost, 26 us of copies in a sub-layer step of 8 x 2048
// tokens, 4 heads, is saved (forward and backward of the sub-layer 280 -> 250 us, four launches less).
template <bool BESIDE>
struct HeadRows {
    int H;
    __device__ __forceinline__ int in_row() const { return BESIDE ? 3 * H * kD : kD; }    // Q, K, V, dQ, dK, dV
    __device__ __forceinline__ int out_row() const { return BESIDE ? H * kD : kD; }       // O, dO
    __device__ __forceinline__ size_t in_head(int bh, int L) const {
        return BESIDE ? ((size_t)(bh / H) * L * 3 * H + bh % H) * kD : (size_t)bh * L * kD;
    }
    __device__ __forceinline__ size_t out_head(int bh, int L) const {
        return BESIDE ? ((size_t)(bh / H) * L * H + bh % H) * kD : (size_t)bh * L * kD;
    }
};

// s_waitcnt immediates (gfx9 encoding: vmcnt [3:0] and [15:14], expcnt [6:4], lgkmcnt [11:8]); the
// counters not named are left at their maximum, i.e. not waited for
constexpr int kWaitVm0 = 0x0F70, kWaitVm4 = 0x0F74, kWaitVm5 = 0x0F75, kWaitLgkm0 = 0xC07F;

__device__ __forceinline__ int swz(int row) { return ((row >> 1) & 3) << 1; }

// A workgroup of BS / 16 waves loads a BS x 64 tile with two instructions per wave.  `src` and
// `wave` are wave-uniform (the wave index comes from readfirstlane), so each load is a scalar base
// plus the lane's fixed 32-bit offset TileLoadLane::off[k].
struct TileLoadLane {
    unsigned off[2];   // byte offset of this lane's 16 bytes from the tile's first row, for piece 2 wave + k
    __device__ __forceinline__ TileLoadLane(int wave, int lane, int row_stride) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int chunk = (lane & 7) ^ (((lane >> 4) & 3) << 1);   // swz(8 piece + lane / 8)
            off[k] = (unsigned)(((2 * wave + k) * 8 + (lane >> 3)) * row_stride + chunk * 8) * (unsigned)sizeof(bf16_t);
        }
    }
};
// Buffer loads: a scalar base and the lane's offset, where a global load into LDS takes a 64-bit vector addition each.  The descriptor's
// range is all that the offset can say (rows of many heads beside each other are far apart).
__device__ __forceinline__ void tile_load_async(const bf16_t* __restrict__ src, bf16_t* tile, int wave,
                                                const TileLoadLane& tl) {
    const __amdgpu_buffer_rsrc_t from = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(src), (short)0, (int)0xffffffffu, 0x00027000);
#pragma unroll
    for (int k = 0; k < 2; ++k)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(from, (lds_void_ptr)(tile + (2 * wave + k) * 512), 16, tl.off[k], 0, 0, 0);
}

// Per-lane read offsets into such a tile (in elements), fixed for the whole kernel.
struct SwzLane {
    int frag[2];   // 16-byte fragment of row r, chunk 4 c + g; add 1024 per 16-row tile
    int tr_row;    // transpose read: row 4 g + r / 4, element offset 4 (r & 1) within the slot
    int tr_sw;     // swz of that row
    int tr_b;      // (r >> 1) & 1: which slot of the 32-byte pair
    __device__ __forceinline__ SwzLane(int r, int g) {
        const int sw = swz(r);
        frag[0] = r * kD + ((g ^ sw) << 3);
        frag[1] = r * kD + (((4 + g) ^ sw) << 3);
        const int trow = 4 * g + (r >> 2);
        tr_row = trow * kD + 4 * (r & 1);
        tr_sw = swz(trow);
        tr_b = (r >> 1) & 1;
    }
    __device__ __forceinline__ int tr(int dt) const { return tr_row + ((((dt << 1) | tr_b) ^ tr_sw) << 3); }
};

// Write this wave's 16 owned rows x 64 columns (accumulators in the transposed layout: lane (r, g)
// holds columns 16 dt + 4 g .. + 3 of row r) as whole 128-byte rows, 16 bytes per lane, instead of
// 8-byte pieces: through a 2 KB LDS patch private to the wave, 16-byte chunks permuted by the row.
// LDS instructions of one wave execute in order, so no barrier is needed between the two halves.
__device__ __forceinline__ void store_rows_coalesced(bf16_t* patch, bf16_t* __restrict__ grow0, int row_stride,
                                                     const f32x4 (&acc)[4], float mul, int lane) {
    const int r = lane & 15, g = lane >> 4;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) {
        const int chunk = (dt * 2 + (g >> 1)) ^ (r & 7);
        *reinterpret_cast<bf16x4*>(patch + r * kD + chunk * 8 + (g & 1) * 4) = to_quad<bf16_t>(acc[dt] * mul);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int row = (lane >> 3) + 8 * j, c = lane & 7;
        const bf16x8 v = *reinterpret_cast<const bf16x8*>(patch + row * kD + ((c ^ (row & 7)) << 3));
        *reinterpret_cast<bf16x8*>(grow0 + (size_t)row * row_stride + c * 8) = v;
    }
}

// Walk order of a block row.  The diagonal block (I, I) is kept by every pattern the generator makes,
// and its address needs no index lookup, so the row-walking kernels start loading it before they
// have read row_ptr / col_idx and visit it first; the other kept blocks follow in index order.  (The
// order of the blocks changes the rounding of the sums only.)  pd = position of I among the row's
// entries, or -1 if the row has no diagonal block: then the walk is in index order and the early
// load is thrown away.
// Scalar loads on purpose: they do not count against the vector-memory counter, so waiting for
// them does not wait for the tile loads already in flight.  The entries of a row ascend, so the scan
// stops at the first entry >= I.  first[] receives entries 0..7 (clamped to the row), from which
// the first blocks of the walk are taken without another dependent load.
__device__ __forceinline__ int find_in_row(const int* __restrict__ cols, int n, int I, int (&first)[8]) {
    const int last = n - 1;
    int pd = -2;   // -2: not decided yet
#pragma unroll
    for (int e = 0; e < 8; ++e) first[e] = cols[e < last ? e : last];
#pragma unroll
    for (int e = 0; e < 8; ++e)
        if (pd == -2 && first[e] >= I) pd = (first[e] == I && e < n) ? e : -1;
    for (int base = 8; base < n && pd == -2; base += 8) {
        int c[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) c[e] = cols[base + e < last ? base + e : last];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (pd == -2 && c[e] >= I) pd = (c[e] == I && base + e < n) ? base + e : -1;
    }
    return pd == -2 ? -1 : pd;
}
__device__ __forceinline__ int pick8(const int (&v)[8], int i) {
    const int a = (i & 1) ? v[1] : v[0], b = (i & 1) ? v[3] : v[2], c = (i & 1) ? v[5] : v[4],
              d = (i & 1) ? v[7] : v[6];
    const int ab = (i & 2) ? b : a, cd = (i & 2) ? d : c;
    return (i & 4) ? cd : ab;
}
__device__ __forceinline__ int walk_index(int t, int pd) {
    return pd < 0 ? t : (t == 0 ? pd : (t - 1 < pd ? t - 1 : t));
}

// Workgroups go round the 8 XCDs in id order.  Workgroup ids lo .. hi - 1 as numbers 0 .. hi - lo - 1 such that each XCD (id % 8) has a contiguous run of
// them, whatever the two bounds are.
__device__ __forceinline__ int xcd_deal(int id, int lo, int hi) {
    const int x = id & 7;
    auto lower_xcds = [x](int n) { return x * (n >> 3) + min(x, n & 7); };   // ids below n of the XCDs before x
    return lower_xcds(hi) - lower_xcds(lo) + (id >> 3) - ((lo + 7 - x) >> 3);
}

// Heads on XCDs, whose number they need not divide: each XCD takes an eighth of the heads, some of which it shares with its neighbour, and
// of its heads the items number 0, 1, .. in this order.  Of eight items running, head h has the points 8 h .. 8 h + 7 of 8 `heads`,
// and XCD x the points from x heads on: `heads` of them.  id: of a workgroup (or of several beside each other), on XCD id % 8; the ids run to
// dealt(heads, items), some of them beyond the last item.  Item by item round all XCDs, each L2 read the tensors of all heads: bf16,
// backward, 42 heads x 5632, block 32, 226 -> 177 us, 75 x 2688 241 -> 175, 78 x 2176, block 64, 117 -> 102; forward, 14 x 2528, block 32, 14.0 -> 11.7, 18 x 6400, block
// 64, 31.0 -> 27.2.  Up to 512 workgroups (`few`) finding the point costs more, 0.1 to
// 0.3 us: backward, round all XCDs over dealt so, 49 shapes up to there 0.95 to 1.05 (0.98 on average), of 512 to 1000 workgroups 0.96 to 1.17 (1.04), above 0.97 to 1.36.
struct ItemOfHead {
    int head, item;
};
__device__ __forceinline__ ItemOfHead deal_heads(int id, int heads, bool few) {
    const int x = id & 7, l = id >> 3;
    if ((heads & 7) == 0) return {x * (heads >> 3) + l % (heads >> 3), l / (heads >> 3)};
    if (few) return {id % heads, id / heads};
    const int round = l / heads;
    int t = l - round * heads, first = 0;   // the XCD's points of item k of the round: x heads + first + 8 t
#pragma unroll 1
    for (int k = 0;; ++k) {   // ends at k = 7 at the latest: there are `heads` points
        first = (k - x * heads) & 7;
        const int n = (heads - first + 7) >> 3;
        if (t < n || k == 7) break;
        t -= n;
    }
    const int at = x * heads + first + 8 * t;
    return {at >> 3, round * 8 + (at & 7)};
}
inline long long dealt(long long heads, long long items, bool few) { return few || heads % 8 == 0 ? items * heads : (items + 7) / 8 * 8 * heads; }

// Rows (columns) in the order of their lengths: longest first, equal ones by index; lengths count in quarters of the mean, four
// times the mean and more alike.  Lane l holds the entry 64 k + l of group k: its length in those units and, as bits
// of a group, which entries take part.  The entry whose place is `want`, found a bit of the length at a time (not at all where no lengths
// count): some 40 instructions a group, no memory access.  Half the mean as unit, a bit less, saves nothing and orders worse (fp32, 64 x 1024, block 32,
// backward 110.8 -> 113 us).  All lanes active, the result uniform; -1: there are not so many entries.
constexpr int kLengthBits = 4;
__device__ __forceinline__ float quarters_of_mean(int nb, int nnzb) { return 4.f * (float)nb * __builtin_amdgcn_rcpf((float)max(nnzb, 1)); }
__device__ __forceinline__ int length_key(int cnt, float quarters) { return min((int)((float)cnt * quarters), (1 << kLengthBits) - 1); }
template <int NG>
__device__ __forceinline__ int entry_by_length(const int (&key)[NG], unsigned long long (&mask)[NG], int want, int lane, bool by_length) {
#pragma unroll 1
    for (int bit = by_length ? 1 << (kLengthBits - 1) : 0; bit; bit >>= 1) {
        unsigned long long upper[NG];
        int n = 0;
#pragma unroll
        for (int k = 0; k < NG; ++k) {
            upper[k] = mask[k] & __ballot((key[k] & bit) != 0);
            n += __popcll(upper[k]);
        }
        const bool in = want < n;
        if (!in) want -= n;
#pragma unroll
        for (int k = 0; k < NG; ++k) mask[k] = in ? upper[k] : mask[k] & ~upper[k];
    }
#pragma unroll
    for (int k = 0; k < NG; ++k) {
        const int members = __popcll(mask[k]);
        if (want < members) {
            const unsigned long long hit = __ballot(((mask[k] >> lane) & 1ull) && lanes_below(mask[k]) == want);
            return 64 * k + __ffsll((long long)hit) - 1;
        }
        want -= members;
    }
    return -1;
}

template <int NG>
__device__ __forceinline__ int row_of_rank(const int* __restrict__ row_ptr, int nb, int rank, int lane) {
    const float quarters = quarters_of_mean(nb, row_ptr[nb]);
    int key[NG];
    unsigned long long mask[NG];
#pragma unroll
    for (int k = 0; k < NG; ++k) {
        const int r = 64 * k + lane;
        key[k] = r < nb ? row_ptr[r + 1] - row_ptr[r] : 0;
        mask[k] = __ballot(r < nb);
    }
#pragma unroll
    for (int k = 0; k < NG; ++k) key[k] = length_key(key[k], quarters);
    return entry_by_length<NG>(key, mask, rank, lane, true);
}
// The same for any number of entries.  What takes part and the four bits of the lengths are kept by lane, a bit for each group of 64,
// and the loops over groups are loops.  As many groups unrolled as SPION_MAX_NB has take 32 masks, more scalar registers than a
// kernel has besides (1 to 32 spilled), and code that whoever calls the kernel pays for at the start of its workgroups: the backward
// kernels had 41 to 53 KB, so 25 to 37; fp32 backward, 6 heads x 640, block 64, 27.4 -> 23.6 us, 15 x 992, block 32, 37.0 -> 34.1.
struct EntriesByLength {
    unsigned in = 0, key[kLengthBits] = {};
    static_assert(SPION_MAX_NB <= 64 * 32, "a bit of a word for each group");
    __device__ __forceinline__ void add(int group, bool takes_part, int length) {
        in |= (unsigned)takes_part << group;
#pragma unroll
        for (int b = 0; b < kLengthBits; ++b) key[b] |= (unsigned)(length >> b & 1) << group;
    }
    __device__ __forceinline__ int entry(int groups, int want, int lane) const {
        unsigned left = in;
#pragma unroll
        for (int b = kLengthBits - 1; b >= 0; --b) {
            const unsigned upper = left & key[b];
            const int n = __builtin_amdgcn_readlane(wave_incl_scan(__popc(upper), lane), 63);
            left = want < n ? upper : left & ~upper;
            if (want >= n) want -= n;
        }
#pragma unroll 1
        for (int k = 0; k < groups; ++k) {
            const unsigned long long mask = __ballot((left >> k & 1u) != 0);
            const int members = __popcll(mask);
            if (want < members) {
                const unsigned long long hit = __ballot(((mask >> lane) & 1ull) && lanes_below(mask) == want);
                return 64 * k + __ffsll((long long)hit) - 1;
            }
            want -= members;
        }
        return -1;
    }
};
__device__ __forceinline__ int row_of_rank_any(const int* __restrict__ row_ptr, int nb, int rank, int lane) {
    const float quarters = quarters_of_mean(nb, row_ptr[nb]);
    EntriesByLength rows;
#pragma unroll 1
    for (int base = 0; base < nb; base += 512) {   // eight groups whose loads are in flight together
        int cnt[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int r = base + 64 * k + lane;
            cnt[k] = r < nb ? row_ptr[r + 1] - row_ptr[r] : -1;
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) rows.add(base / 64 + k, cnt[k] >= 0, length_key(max(cnt[k], 0), quarters));
    }
    return rows.entry((nb + 63) / 64, rank, lane);
}
__device__ __forceinline__ int row_by_length(const int* __restrict__ row_ptr, int nb, int rank, int lane) {
    if (nb <= 64) return row_of_rank<1>(row_ptr, nb, rank, lane);
    if (nb <= 128) return row_of_rank<2>(row_ptr, nb, rank, lane);
    if (nb <= 256) return row_of_rank<4>(row_ptr, nb, rank, lane);
    return row_of_rank_any(row_ptr, nb, rank, lane);
}

// ------------------------------------------------------------------------------------------------
// Long rows in pieces.  A block row is one chain of steps; patterns have a row or two of several times the mean, up to
// half the columns, and where there are few heads such a chain outlasts everything else: 8 heads x 8192, block 32, 13
// blocks a row and two rows of 120: forward 44 us, 14 without those rows.  A row of more than `longest` blocks is cut into pieces
// of about `piece`.  The row's own workgroup takes the first piece; `helpers` workgroups of each head, which come first in the grid,
// take the others (the forward's in turn; the backward's query side has one for each).  Where a pattern has more pieces than there are
// `slots` for, pieces are half as long again, and rows are cut that are 3/2 of them, until it has not: so the longest rows are
// cut, whatever the shorter ones need.  (Cut in their order as long as there was room, they used it up before the longest came, or had themselves
// more pieces than there was room for: 4 heads x 16384, block 32, 10 blocks a row, two rows of 200, forward 85 -> 27.5 us, backward
// 115 -> 50.)  Every workgroup finds the same cuts from row_ptr.
// Each piece leaves its accumulators, reference and sum in memory; the workgroup that is the last of its row to do so adds
// up the pieces in their order (the same bits whoever that is) and writes the row.  Nobody waits for anybody.
// ------------------------------------------------------------------------------------------------
struct RowPieces {
    int row;      // -1: none
    int count;    // pieces of the row, 1: not cut
    int first;    // number of its second piece among the head's pieces that are not the first of their row
    int slot;     // of its first piece
};
// Kernels that cut nothing carry no plan.
struct NoCut {};
template <bool CUT>
using CutOf = std::conditional_t<CUT, RowCut, NoCut>;

// The row that piece number `want`, not the first of its row, belongs to, or (BY_ROW) row number `want`.  All lanes
// active, the result uniform.
template <bool BY_ROW>
__device__ __forceinline__ RowPieces row_pieces(const int* __restrict__ row_ptr, int nb, const RowCut& cut, int want, int lane) {
    for (int piece = cut.piece; piece < 2 * SPION_MAX_NB; piece += piece / 2) {   // a piece is 8 blocks or more; ends with no row to cut at the latest
        const int longest = piece == cut.piece ? cut.longest : max(cut.longest, 3 * piece / 2);
        const float per_piece = __builtin_amdgcn_rcpf((float)piece);
        int others = 0, cut_rows = 0;   // pieces (not the first of a row) and long rows before this group of 64 rows
        RowPieces found = {BY_ROW ? want : -1, 1, 0, 0};
        auto kept = [&](int r) { return r < nb ? row_ptr[r + 1] - row_ptr[r] : 0; };
        int next = kept(lane);
#pragma unroll 1
        for (int base = 0; base < nb; base += 64) {
            const int r = base + lane, cnt = next;
            next = kept(r + 64);   // in flight over this group
            if (!__any(cnt > longest)) continue;
            const int count = cnt > longest ? (int)(((float)(cnt + piece) - 0.5f) * per_piece) : 1;   // rounded up
            const int incl = others + wave_incl_scan(count - 1, lane), first = incl - (count - 1);
            const unsigned long long longs = __ballot(count > 1);
            const unsigned long long hit = __ballot(count > 1 && (BY_ROW ? r == want : want >= first && want < incl));
            if (hit) {
                const int src = __ffsll((long long)hit) - 1;
                const int f = __builtin_amdgcn_readlane(first, src);
                found = {base + src, __builtin_amdgcn_readlane(count, src), f, f + cut_rows + (int)__popcll(longs & ((1ull << src) - 1ull))};
            }
            others = __builtin_amdgcn_readlane(incl, 63);
            cut_rows += (int)__popcll(longs);
        }
        if (others + cut_rows <= cut.slots) return found;
    }
    return {BY_ROW ? want : -1, 1, 0, 0};
}

// Partial results go between workgroups, which may be on different XCDs, by accesses of device scope: past the L2 to where
// all XCDs meet.  (Plain accesses with a release and an acquire around the counter write a whole L2 back and drop what it
// holds, tiles of everyone's K and V, for every piece: 64 heads x 4160, block 32, 384 pieces: 36 us uncut, 55 so.)
__device__ __forceinline__ void put_shared(float* p, float a, float b) {
    const unsigned long long v = (unsigned long long)__builtin_bit_cast(unsigned, b) << 32 | __builtin_bit_cast(unsigned, a);
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 get_shared(const float* p) {
    const unsigned long long v = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return make_float2(__builtin_bit_cast(float, (unsigned)v), __builtin_bit_cast(float, (unsigned)(v >> 32)));
}

// Counts the calling workgroup's piece at *counter; whether it is the last of `count`.  What the others' waves have
// put_shared before their calls, every wave can get_shared after it then.  The counter holds the launch's tag and the pieces
// that have arrived, or whatever else is in the memory when the first one comes; the last one clears it, for a launch
// with the same tag (a graph that is replayed).  All threads; `flag` is in LDS.
__device__ __forceinline__ bool last_to_arrive(unsigned long long* counter, unsigned long long tag, int count, int* flag) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's stores are done, at device scope
    __syncthreads();                                   // and those of the others
    if (threadIdx.x == 0) {
        unsigned long long seen = __hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), next;
        do {
            next = seen >> kArriveBits == tag ? seen + 1 : tag << kArriveBits | 1;
        } while (!__hip_atomic_compare_exchange_strong(counter, &seen, next, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        const bool last = (int)(next & ((1ull << kArriveBits) - 1ull)) == count;
        if (last) __hip_atomic_store(counter, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *flag = last;
    }
    __syncthreads();
    asm volatile("" ::: "memory");   // nothing of the others' is read before
    return *flag != 0;
}

}  // namespace spion
#endif
