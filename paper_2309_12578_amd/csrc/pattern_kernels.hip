// Pattern generation kernels for gfx950 (Algorithm 3 and Algorithm 4 of the SPION paper).
//
//   conv_pool_kernel      Eq. 3 + Eq. 4 fused: one streaming pass over A^s that splits every input
//                         block's (fixed-point) scores over the <= 7 pooled blocks its diagonal filter
//                         window touches and writes the seven sums.  HBM bound: A^s is read exactly
//                         once, nothing L x L is written, no atomics.
//   pattern_finish_kernel L / block <= 64, one workgroup: adds the sums up into pool_sum, then
//                         threshold (exact order statistic / mean + k std), flood fill, forced
//                         diagonal, BSR + BSC compaction.  Latency bound (at most 4096 cells).
//   grid_*_kernel         the same steps for larger grids (up to 1024 x 1024 cells), spread over the
//                         machine: four grid-wide kernels and one of two workgroups for the serial
//                         parts.
//
// Arithmetic: a_q = rint(a * 2^40) as an exact integer; all sums are integer, so any summation
// order (tiling, partial sums) gives the same bits.  This file is compiled with -ffp-contract=off: the
// fp64 mean / std threshold must round exactly as its sequential definition.
//
// The fill works on rows of bits.  With D, R, G the sets of cells of row r whose down / right / diagonal
// neighbour equals the maximum of the three, and E the expanded cells (reached, or a seed: row 0 and
// column 0), row r gets its entries from the row above,
//     entry = (E[r-1] & D[r-1]) | ((E[r-1] & G[r-1]) << 1),
// and spreads them to the right along R.  Spreading a set x along runs of ones in R is a carry chain:
// (x & R) + R carries from the lowest member of x in a run to the first position behind the run, so
//     E = x | (((x & R) + R) ^ R),   x = entry | seeds.
// A row is one addition, so the fill takes one short chain per row instead of one dependent step per
// anti-diagonal.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "grid_bins.h"
#include "spion_internal.h"

namespace spion {

// ------------------------------------------------------------------------------------------------
// conv + pool
// ------------------------------------------------------------------------------------------------
// Input block (I, J) of A^s (bs x bs scores).  conv_out(i, j) = sum_{g=-p..p} a(i+g, j+g), so the
// score at local position (u, v) of this block is added to the outputs (u-g, v-g), g in [-p, p].
// Those outputs fall into blocks (I+di, J+dj) with di, dj in {-1, 0, +1} (p < bs) and never into
// (-1,+1) or (+1,-1) because g shifts both coordinates alike.  With (x)+ = max(x, 0), u' = bs-1-u and
// v' = bs-1-v, of the F = 2p+1 positions of the filter
//     (p-u)+  leave the block upwards, (p-v)+ to the left, and min of the two do both,
//     (p-u')+ leave it downwards, (p-v')+ to the right, and min of the two do both,
// so the seven sums of a block follow from row-weighted sums, column-weighted sums (which are weighted
// column sums), and two corner sums that only scores near the corners enter:
//     (-1,-1) = C1 = sum min((p-u)+, (p-v)+) a_q       (-1,0) = sum (p-u)+ a_q - C1,  (0,-1) likewise
//     (+1,+1) = C2 = sum min((p-u')+, (p-v')+) a_q     (+1,0) = sum (p-u')+ a_q - C2, (0,+1) likewise
//     (0,0)   = F sum a_q - the six others.
//
// Fixed point: a * 2^40 is exact in fp32 (a power of two), so rint of it is a_q = rint(a * 2^40), ties to
// even, an integer of at most 41 bits.  Per lane the sums stay in fp64: |a_q| <= 2^40, a lane owns at
// most 64 scores of a block and the weights add up to F <= 127, so every partial sum is an integer below
// 2^53 and exact.  (fp64 adds and fused multiply-adds issue at the rate of fp32 ones here.)

// Slot s of the sums of input block (I, J) belongs to pooled block (I + di(s), J + dj(s)):
// 0 (0,0)  1 (-1,0)  2 (+1,0)  3 (0,-1)  4 (0,+1)  5 (-1,-1)  6 (+1,+1)
constexpr int kSlots = 7;

// Sum of the slots 2a and 2b (64-bit) over lane pairs that differ in bit 5 (SWAP32) or bit 4 of the lane
// number: lanes with the bit clear end up with a's sum, the others with b's.  The swap exchanges half of
// one register with the other half of the other in the VALU, without the LDS crossbar.
template <bool SWAP32>
__device__ __forceinline__ long long pair_sum(long long a, long long b) {
    const unsigned al = (unsigned)a, ah = (unsigned)(a >> 32), bl = (unsigned)b, bh = (unsigned)(b >> 32);
    unsigned x0, x1, y0, y1;
    if constexpr (SWAP32) {
        const auto l = __builtin_amdgcn_permlane32_swap(al, bl, false, false);
        const auto h = __builtin_amdgcn_permlane32_swap(ah, bh, false, false);
        x0 = l[0], y0 = l[1], x1 = h[0], y1 = h[1];
    } else {
        const auto l = __builtin_amdgcn_permlane16_swap(al, bl, false, false);
        const auto h = __builtin_amdgcn_permlane16_swap(ah, bh, false, false);
        x0 = l[0], y0 = l[1], x1 = h[0], y1 = h[1];
    }
    return (long long)((unsigned long long)x1 << 32 | x0) + (long long)((unsigned long long)y1 << 32 | y0);
}

__device__ __forceinline__ long long shfl_xor_i64(long long v, int mask) { return __shfl_xor(v, mask); }

// One wave per tile of BS rows x 64 columns (one block of 64, two of 32 or four of 16): every load
// instruction covers 4 rows of 256 bytes, all of a tile's loads are requested before the first is used,
// and 16 waves per compute unit are resident.  Lane (k, j) owns rows 4 i + k and columns 4 j .. 4 j + 3.
// Slot sums go to part[slot][I * nb + J] (index of the SOURCE block), so that the waves of a workgroup
// write neighbouring words and the readers read whole rows of them.
// Measured: 64 MiB map, block 64: 13.5 us = 5.0 TB/s (17.7 with one wave per block, general weights per score
// and 210 registers); 256 MiB map, block 16: 48.9 us = 5.5 TB/s (172: a whole wave per block of 1 KB).
// The map is read once: non-temporal loads take 2 us off a call at 256 MiB, block 64 (89.8 -> 87.8).
template <int BS>
__global__ __launch_bounds__(256, 4) void conv_pool_kernel(const float* __restrict__ A, int L, int p,
                                                           long long* __restrict__ part, unsigned* __restrict__ zero,
                                                           int n_zero) {
    constexpr int NL = BS / 4;     // loads (row groups) per lane
    constexpr int BPT = 64 / BS;   // blocks side by side in a tile
    const int gid = blockIdx.x * 256 + threadIdx.x;
    if (gid < n_zero) zero[gid] = 0u;   // counters that the kernels after this one add to
    const int nb = L / BS, tiles_x = (nb + BPT - 1) / BPT;
    const int lane = threadIdx.x & 63;
    const int tile = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
    if (tile >= nb * tiles_x) return;
    const int I = tile / tiles_x, tx = tile % tiles_x;
    const int k = lane >> 4, j = lane & 15;
    const int J = tx * BPT + (4 * j) / BS;
    const bool live = J < nb;      // the last tile of a row may reach past the matrix
    const float* src = A + (size_t)I * BS * L + tx * 64;   // wave-uniform, the lane's part is a 32-bit offset
    const unsigned off = (unsigned)(k * L + 4 * j);
    typedef float f32x4_t __attribute__((ext_vector_type(4)));
    f32x4_t a[NL];
    if (BPT == 1 || live) {
#pragma unroll
        for (int i = 0; i < NL; ++i) a[i] = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(src + (size_t)(4 * i) * L + off));
    } else {
#pragma unroll
        for (int i = 0; i < NL; ++i) a[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }

    int pl[4], pr[4];              // (p - v)+ and (p - v')+ of the lane's columns
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int v = (4 * j) % BS + e;
        pl[e] = max(p - v, 0);
        pr[e] = max(p - (BS - 1 - v), 0);
    }
    double cs[4] = {0.0, 0.0, 0.0, 0.0}, rt = 0.0, rb = 0.0, c1 = 0.0, c2 = 0.0;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        // The weights depend only on the lane and the filter; left to itself the compiler makes those of
        // all row groups while it waits for the loads, and spills them.  Hiding the filter's half-width
        // and the lane's row makes them per-group work.
        int ph = p, kh = k;
        asm volatile("" : "+s"(ph), "+v"(kh));
        __builtin_amdgcn_sched_barrier(0);
        const float av[4] = {a[i].x, a[i].y, a[i].z, a[i].w};
        double q[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            q[e] = (double)__builtin_rintf(av[e] * 1099511627776.0f);
            cs[e] += q[e];
            asm volatile("" : "+v"(cs[e]));   // added now: the compiler would keep the terms for the end
        }
        if (4 * i < ph) {                         // some of these rows lie within p of the top edge
            const int pu = max(ph - 4 * i - kh, 0);
            rt = __builtin_fma((double)pu, (q[0] + q[1]) + (q[2] + q[3]), rt);
#pragma unroll
            for (int e = 0; e < 4; ++e) c1 = __builtin_fma((double)min(pu, pl[e]), q[e], c1);
        }
        if (4 * i + 3 > BS - 1 - ph) {            // ... of the bottom edge
            const int pd = max(ph - (BS - 1 - 4 * i - kh), 0);
            rb = __builtin_fma((double)pd, (q[0] + q[1]) + (q[2] + q[3]), rb);
#pragma unroll
            for (int e = 0; e < 4; ++e) c2 = __builtin_fma((double)min(pd, pr[e]), q[e], c2);
        }
    }
    double cl = 0.0, cr = 0.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        cl = __builtin_fma((double)pl[e], cs[e], cl);
        cr = __builtin_fma((double)pr[e], cs[e], cr);
    }
    const double all = (double)(2 * p + 1) * ((cs[0] + cs[1]) + (cs[2] + cs[3]));
    // from here on in 64-bit integers: the sums over a block's lanes can exceed 2^53
    long long t[8];
    t[1] = (long long)(rt - c1);
    t[2] = (long long)(rb - c2);
    t[3] = (long long)(cl - c1);
    t[4] = (long long)(cr - c2);
    t[5] = (long long)c1;
    t[6] = (long long)c2;
    t[0] = (long long)(all - ((rt + cl - c1) + (rb + cr - c2)));
    t[7] = 0;
    // reduce-scatter over the lanes of a block (lane bits 5 and 4 are its rows; of bits 0..3 the lowest
    // log2(BS / 4) are its columns): 8 slots -> 4 -> 2 -> 1, then plain steps over the bits left
    constexpr int kThird = BS == 64 ? 8 : (BS == 32 ? 4 : 2);
#pragma unroll
    for (int s = 0; s < 4; ++s) t[s] = pair_sum<true>(t[s], t[s + 4]);
#pragma unroll
    for (int s = 0; s < 2; ++s) t[s] = pair_sum<false>(t[s], t[s + 2]);
    const bool up = (lane & kThird) != 0;
    const long long send = up ? t[0] : t[1], keep = up ? t[1] : t[0];
    long long sum = keep + shfl_xor_i64(send, kThird);
#pragma unroll
    for (int m = kThird >> 1; m > 0; m >>= 1) sum += shfl_xor_i64(sum, m);
    if ((lane & (kThird - 1)) == 0 && live) {
        const int slot = ((lane >> 5) & 1) * 4 + ((lane >> 4) & 1) * 2 + (up ? 1 : 0);
        if (slot < kSlots) part[(size_t)slot * ((size_t)nb * nb) + (size_t)I * nb + J] = sum;
    }
}

// pool_sum of cell (ti, tj): slot s of its source block (ti - di(s), tj - dj(s)), for the source blocks that
// exist.  The loads of the others are redirected to the cell itself and dropped, so that all seven are
// requested at once.
struct PoolParts {
    long long v[kSlots];
};
__device__ __forceinline__ PoolParts load_parts(const long long* __restrict__ part, int nb, int ti, int tj) {
    const int n = nb * nb, i = ti * nb + tj;
    const bool up = ti >= 1, down = ti + 1 < nb, left = tj >= 1, right = tj + 1 < nb;
    PoolParts r;
    r.v[0] = part[i];
    r.v[1] = part[(size_t)n + (down ? i + nb : i)];
    r.v[2] = part[(size_t)2 * n + (up ? i - nb : i)];
    r.v[3] = part[(size_t)3 * n + (right ? i + 1 : i)];
    r.v[4] = part[(size_t)4 * n + (left ? i - 1 : i)];
    r.v[5] = part[(size_t)5 * n + (down && right ? i + nb + 1 : i)];
    r.v[6] = part[(size_t)6 * n + (up && left ? i - nb - 1 : i)];
    return r;
}
__device__ __forceinline__ long long sum_parts(const PoolParts& r, int nb, int ti, int tj) {
    const bool up = ti >= 1, down = ti + 1 < nb, left = tj >= 1, right = tj + 1 < nb;
    return r.v[0] + (down ? r.v[1] : 0) + (up ? r.v[2] : 0) + (right ? r.v[3] : 0) + (left ? r.v[4] : 0) +
           (down && right ? r.v[5] : 0) + (up && left ? r.v[6] : 0);
}

// pool_sum alone (the convolution + pooling stage run on its own)
__global__ __launch_bounds__(256) void pool_gather_kernel(const long long* __restrict__ part, int nb,
                                                          long long* __restrict__ pool) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < nb * nb) pool[i] = sum_parts(load_parts(part, nb, i / nb, i % nb), nb, i / nb, i % nb);
}

// ------------------------------------------------------------------------------------------------
// helpers of the threshold, fill and compaction steps
// ------------------------------------------------------------------------------------------------
constexpr int kFinishThreads = 1024;
constexpr int kFinishWaves = kFinishThreads / 64;

struct Thresh {
    int is_int;
    long long ti;
    double td;
};
__device__ __forceinline__ bool above(long long x, const Thresh& t) {
    return t.is_int ? x > t.ti : (double)x > t.td;
}

// Inclusive prefix sum over the wave with DPP moves (VALU speed, no LDS crossbar): shifts of 1, 2, 4, 8
// inside each row of 16 lanes, then lane 15 of rows 0 and 2 added to rows 1 and 3, then lane 31 added to
// rows 2 and 3.  A lane whose source is outside its row, or whose row is masked off, adds the 0 given as
// old value.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_fetch(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROW_MASK, 0xf, false);
}
__device__ __forceinline__ int wave_inclusive_scan_dpp(int v) {
    v += dpp_fetch<0x111, 0xf>(v);   // row_shr:1
    v += dpp_fetch<0x112, 0xf>(v);   // row_shr:2
    v += dpp_fetch<0x114, 0xf>(v);   // row_shr:4
    v += dpp_fetch<0x118, 0xf>(v);   // row_shr:8
    v += dpp_fetch<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
    v += dpp_fetch<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
    return v;
}

// Sum over the wave, same data movement; the result is in lane 63.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ long long dpp_fetch_i64(long long v) {
    const unsigned lo = (unsigned)dpp_fetch<CTRL, ROW_MASK>((int)(unsigned)v), hi = (unsigned)dpp_fetch<CTRL, ROW_MASK>((int)(v >> 32));
    return (long long)((unsigned long long)hi << 32 | lo);
}
__device__ __forceinline__ long long wave_sum_i64(long long v) {
    v += dpp_fetch_i64<0x111, 0xf>(v);
    v += dpp_fetch_i64<0x112, 0xf>(v);
    v += dpp_fetch_i64<0x114, 0xf>(v);
    v += dpp_fetch_i64<0x118, 0xf>(v);
    v += dpp_fetch_i64<0x142, 0xa>(v);
    v += dpp_fetch_i64<0x143, 0xc>(v);
    return v;
}

// Minimum over the wave, same data movement; the result is in lane 63.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_fetch_or_self(int v) {
    return __builtin_amdgcn_update_dpp(v, v, CTRL, ROW_MASK, 0xf, false);
}
__device__ __forceinline__ int wave_min_dpp(int v) {
    v = min(v, dpp_fetch_or_self<0x111, 0xf>(v));
    v = min(v, dpp_fetch_or_self<0x112, 0xf>(v));
    v = min(v, dpp_fetch_or_self<0x114, 0xf>(v));
    v = min(v, dpp_fetch_or_self<0x118, 0xf>(v));
    v = min(v, dpp_fetch_or_self<0x142, 0xa>(v));
    v = min(v, dpp_fetch_or_self<0x143, 0xc>(v));
    return v;
}

// Successor bits of a cell: which of down / right / diagonal equal the maximum of the three (none in the
// last row and column, where walks stop).
struct Succ {
    bool down, right, diag;
};
__device__ __forceinline__ Succ successors(long long dn, long long rt, long long dg, bool inner) {
    long long mx = dn > rt ? dn : rt;
    mx = mx > dg ? mx : dg;
    return {inner && dn == mx, inner && rt == mx, inner && dg == mx};
}

// Sum of n doubles in index order, s = ((x[0] + x[1]) + x[2]) + ...: the order is the definition of the
// mean / std threshold, so the additions are one dependent chain.  x is in LDS, 16-byte aligned; 16 values
// are requested ahead of the 16 being added, so that the chain never waits for a load.  Every lane of the
// calling wave computes the same value.
__device__ __forceinline__ double ordered_sum(const double* x, int n) {
    double s = 0.0;
    double2 even[8], odd[8];
    const double2* v = reinterpret_cast<const double2*>(x);
    const int groups = n >> 4, last = groups > 0 ? groups - 1 : 0;
    auto request = [&](double2 (&dst)[8], int g) {
#pragma unroll
        for (int e = 0; e < 8; ++e) dst[e] = v[(g < last ? g : last) * 8 + e];
        __builtin_amdgcn_sched_barrier(0);   // before the additions of the other group
    };
    auto add = [&](const double2 (&src)[8]) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            s = s + src[e].x;
            s = s + src[e].y;
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    if (groups > 0) request(even, 0);
    for (int g = 0; g < groups; g += 2) {
        request(odd, g + 1);
        add(even);
        request(even, g + 2);
        if (g + 1 < groups) add(odd);
    }
    for (int i = groups << 4; i < n; ++i) s = s + x[i];
    return s;
}

__device__ __forceinline__ unsigned long long read_lane_u64(unsigned long long w, int l) {
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)w, l);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(w >> 32), l);
    return (unsigned long long)hi << 32 | lo;
}

// Radix selection: digits of kDigitBits bits, most significant first; 64-bit keys need kSelPasses.
constexpr int kDigitBits = 11, kBins = 1 << kDigitBits, kSelPasses = 6;
static_assert(kDigitBits * (kSelPasses - 1) < 64 && kDigitBits * kSelPasses >= 64, "passes must cover 64 bits");
static_assert(kBins == 32 * 64, "one wave scans a histogram with 32 bins per lane");
// Where the counter of digit D lives in a histogram: lane D / 32 of a scanning wave owns the 32
// consecutive digits 32 (D / 32) .. + 31 as eight 16-byte groups, and group j of all lanes is
// contiguous, so that the wave reads it without bank conflicts.
__device__ __forceinline__ int bin_slot(unsigned D) { return (int)(((D >> 2) & 7u) * 256u + (D >> 5) * 4u + (D & 3u)); }

struct SelectShared {
    int digit, below, count, cand_n, common_lz;
    int n_below, shift;                       // sampled selection (nb <= 64)
    unsigned long long cand[64], key, lo, hi;
};

// One wave: the digit whose bin holds rank k, how many keys lie below it and in it (nothing is written if the
// histogram holds no more than k keys).  Lane owns digits 32 lane .. 32 lane + 31 as 8 groups of 4.
__device__ __forceinline__ void scan_histogram(const unsigned* h, int k, SelectShared* sh) {
    const int lane = threadIdx.x & 63;
    const uint4* const h4 = reinterpret_cast<const uint4*>(h);
    int s4[8], s32 = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const uint4 v = h4[j * 64 + lane];
        s4[j] = (int)(v.x + v.y + v.z + v.w);
        s32 += s4[j];
    }
    const int incl = wave_inclusive_scan_dpp(s32);
    int e = incl - s32, qj = 0;
    const bool hit = k >= e && k < incl;   // at most one lane
#pragma unroll
    for (int j = 0; j < 7; ++j) {
        const bool adv = qj == j && k >= e + s4[j];
        e = adv ? e + s4[j] : e;
        qj = adv ? j + 1 : qj;
    }
    const uint4 v = h4[qj * 64 + lane];
    const int c3[3] = {(int)v.x, (int)v.y, (int)v.z};
    int qt = 0;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const bool adv = qt == j && k >= e + c3[j];
        e = adv ? e + c3[j] : e;
        qt = adv ? j + 1 : qt;
    }
    if (hit) {
        sh->digit = 32 * lane + 4 * qj + qt;
        sh->below = e;
        sh->count = (int)(qt == 0 ? v.x : (qt == 1 ? v.y : (qt == 2 ? v.z : v.w)));
    }
}

// All waves: the k-th smallest of the sh->cand_n <= 64 collected keys, into sh->key.  A wave ranks every 16th
// of them: one ballot counts the smaller ones.
__device__ __forceinline__ void rank_candidates(int k, SelectShared* sh) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), cn = sh->cand_n;
    const unsigned long long mine = lane < cn ? sh->cand[lane] : ~0ull;
    for (int t = wave; t < cn; t += kFinishWaves) {
        const unsigned long long other = read_lane_u64(mine, t);
        const int less = __popcll(__ballot(mine < other)), same = __popcll(__ballot(lane < cn && mine == other));
        if (lane == 0 && k >= less && k < less + same) sh->key = other;   // equal keys write the same value
    }
}

// Exact k-th smallest (0-based) of a set of 64-bit keys held by a workgroup of kFinishThreads threads, by
// radix selection.  each(f) calls f(key, active) for every key of the calling thread, all lanes of a wave
// together; `ref` is any one of the keys (the same in all threads).  hist: 3 * kBins counters, cleared here.
// A pass: every wave counts its keys' digits into a histogram; one wave scans it (32 bins per lane, a DPP
// prefix sum) and publishes the digit that holds rank k; three histograms rotate, the other waves clear
// the one of the pass before meanwhile.  Leading bits that all keys share need no pass, and as soon as at
// most 64 keys share the selected prefix they are collected and one wave ranks them against each other.
template <class Each>
__device__ __forceinline__ unsigned long long select_kth(Each&& each, unsigned long long ref, int k, unsigned* hist,
                                                         SelectShared* sh) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int i = tid; i < 3 * kBins; i += kFinishThreads) hist[i] = 0u;
    if (tid == 0) {
        sh->common_lz = 64;
        sh->cand_n = 0;
    }
    __syncthreads();
    unsigned long long differ = 0ull;
    each([&](unsigned long long u, bool active) { differ |= active ? u ^ ref : 0ull; });
    const int lz = wave_min_dpp(differ ? __clzll((long long)differ) : 64);
    if (lane == 63) atomicMin(&sh->common_lz, lz);
    __syncthreads();
    const int n_passes = (64 - sh->common_lz + kDigitBits - 1) / kDigitBits;   // 0: all keys are equal
    unsigned long long prefix = 0ull;
    if (kDigitBits * n_passes < 64) prefix = ref & ~((1ull << (kDigitBits * n_passes)) - 1ull);
#pragma unroll 1
    for (int pass = 0; pass < n_passes; ++pass) {
        const int shift = kDigitBits * (n_passes - 1 - pass);   // without shared bits: 55, 44, ..., 0
        const int top = shift + kDigitBits;                     // bits >= top are already decided
        unsigned* const h = hist + (pass % 3) * kBins;
        each([&](unsigned long long u, bool active) {
            const bool match = active && (top >= 64 || (u >> top) == (prefix >> top));
            const unsigned digit = (unsigned)(u >> shift) & (unsigned)(kBins - 1);
            // the leading digits are usually equal for the whole wave: one atomic instead of 64
            const unsigned long long m = __ballot(match);
            if (m == 0ull) return;
            const unsigned first = (unsigned)__builtin_amdgcn_readlane((int)digit, __ffsll((long long)m) - 1);
            if (__ballot(match && digit == first) == m) {
                if (lane == 0) atomicAdd(&h[bin_slot(first)], (unsigned)__popcll(m));
            } else if (match) {
                atomicAdd(&h[bin_slot(digit)], 1u);
            }
        });
        __syncthreads();
        if (wave != 0) {
            // the histogram of the pass before (last read before the barrier above) is cleared for the
            // pass after the next, off the path of the wave that scans
            unsigned* const hz = hist + ((pass + 2) % 3) * kBins;
            for (int i = tid - 64; i < kBins; i += kFinishThreads - 64) hz[i] = 0u;
        } else {
            scan_histogram(h, k, sh);
        }
        __syncthreads();
        k -= sh->below;
        prefix |= (unsigned long long)(unsigned)sh->digit << shift;
        if (pass + 1 < n_passes && sh->count <= 64) {
            // few keys are left (typically after the second pass); k is the rank among them
            each([&](unsigned long long u, bool active) {
                if (active && (u >> shift) == (prefix >> shift)) sh->cand[atomicAdd(&sh->cand_n, 1)] = u;
            });
            __syncthreads();
            rank_candidates(k, sh);
            __syncthreads();
            prefix = sh->key;
            break;
        }
    }
    return prefix;
}

constexpr unsigned long long kSign = 0x8000000000000000ull;   // int64 order as unsigned order: flip the sign bit

// ------------------------------------------------------------------------------------------------
// threshold + fill + compaction, nb <= 64 (one workgroup)
// ------------------------------------------------------------------------------------------------
// Thread (wave, lane) owns the cells (4 wave + j, lane), j < 4, and keeps their values in registers: a wave
// owns whole rows, so a ballot is a row of bits.  Which cells a walk reaches does not depend on the
// threshold, so wave 1 fills (scalar 64-bit words, one short chain per row) while the others select; its own
// four rows are selected from by the waves 2 to 5.
// Order statistic: 64 sampled cells are ranked against each other and bracket the wanted rank; one
// histogram of 2048 bins over the bracket, and the few keys of one bin are ranked.  A bracket of a fifth of
// the cells spreads them over the bins, where a radix digit piles most of them into a few counters, whose
// LDS atomics then queue up.  Where the bracket misses (or a bin holds more than 64 keys: ties) the radix
// selection above decides.
// Bound by latency: of 14 us at nb = 64, the loads of the slot sums (just written by other XCDs) are 4.3,
// the selection with the fill beside it 6, the rest short steps between barriers.  (22.4 us with three radix
// passes and an anti-diagonal fill of 127 steps behind them; with mean + k std at nb = 16, 51 -> 11.4 us,
// the additions being taken from LDS instead of from memory one by one.)
// mode: 0 = threshold given in t_abs, 1 = quantile rank k_rank, 2 = mean + kval * std.
// part: sums of conv_pool_kernel, from which pool[] is first computed; nullptr: pool[] is given.
// nnzb_host: nullptr, or a word of host memory that receives nnzb after everything else is written.
__global__ __launch_bounds__(kFinishThreads) void pattern_finish_kernel(
    const long long* __restrict__ part, long long* pool, int nb, int mode, int k_rank, double kval,
    double t_abs, int no_fill, uint8_t* __restrict__ fl, int* __restrict__ row_ptr, int* __restrict__ col_idx,
    int* __restrict__ col_ptr, int* __restrict__ row_idx, int* __restrict__ bsr_pos,
    int* __restrict__ nnzb_out, int* nnzb_host) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = nb * nb;
    __shared__ __attribute__((aligned(16))) long long pool_s[64 * 64];   // every 4th row of pool_sum; later doubles
    __shared__ __attribute__((aligned(16))) unsigned hist[3 * kBins];
    __shared__ unsigned long long down[64], right[64], diag[64], reached[64], rowmask[64], colmask[64];
    __shared__ int line_start[64], col_start[64];
    __shared__ Thresh th;
    __shared__ SelectShared sel;

    constexpr int kCached = 4;
    static_assert(kCached * kFinishWaves == 64, "the owned cells of a thread cover 64 rows");
    const int row0 = kCached * wave;   // this wave's rows: row0 .. row0 + 3
    auto own_cell = [&](int j, int& i) {
        i = (row0 + j) * nb + lane;
        return row0 + j < nb && lane < nb;
    };

    // ---- 0. pool_sum: all of a thread's loads are requested before the first is used --------------------
    long long val[kCached] = {0, 0, 0, 0};
    if (part) {
        PoolParts rec[kCached];
#pragma unroll
        for (int j = 0; j < kCached; ++j) {
            int i;
            const bool ok = own_cell(j, i);
            rec[j] = load_parts(part, nb, ok ? row0 + j : 0, ok ? lane : 0);
        }
        for (int i = tid; i < kBins; i += kFinishThreads) hist[i] = 0u;
#pragma unroll
        for (int j = 0; j < kCached; ++j) {
            int i;
            if (own_cell(j, i)) {
                val[j] = sum_parts(rec[j], nb, row0 + j, lane);
                pool[i] = val[j];
            }
        }
    } else {
        for (int i = tid; i < kBins; i += kFinishThreads) hist[i] = 0u;
#pragma unroll
        for (int j = 0; j < kCached; ++j) {
            int i;
            if (own_cell(j, i)) val[j] = pool[i];
        }
    }
    if (tid == 0) {
        sel.n_below = 0;
        sel.cand_n = 0;
        sel.count = -1;
    }
    pool_s[wave * 64 + lane] = val[0];   // the row below the last of wave - 1
    if (wave == 1) {
#pragma unroll
        for (int j = 0; j < kCached; ++j) pool_s[(kFinishWaves + j) * 64 + lane] = val[j];
    }
    __syncthreads();

    // ---- 1. successor bits, one 64-bit word per row and direction; row r + 1 is this wave's next row, or
    //         the first of the next wave; right neighbours come from the next lane -----------------------------
    if (!no_fill) {
        auto from_right = [&](long long v) {
            const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)v, 0x130 /* wave_shl:1 */, 0xf, 0xf, false);
            const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(v >> 32), 0x130, 0xf, 0xf, false);
            return (long long)((unsigned long long)hi << 32 | lo);
        };
        const long long next_first = pool_s[(wave + 1 < kFinishWaves ? wave + 1 : wave) * 64 + lane];
        long long dg_of[kCached + 1];
#pragma unroll
        for (int j = 0; j < kCached; ++j) dg_of[j] = from_right(val[j]);
        dg_of[kCached] = from_right(next_first);
#pragma unroll
        for (int j = 0; j < kCached; ++j) {
            const int r = row0 + j;
            if (r >= nb) continue;   // wave-uniform
            const bool inner = r + 1 < nb && lane + 1 < nb;
            const Succ s = successors(j + 1 < kCached ? val[j + 1 < kCached ? j + 1 : j] : next_first, dg_of[j],
                                      dg_of[j + 1], inner);
            const unsigned long long bd = __ballot(s.down), br = __ballot(s.right), bg = __ballot(s.diag);
            if (lane == 0) {
                down[r] = bd;
                right[r] = br;
                diag[r] = bg;
            }
        }
    }
    __syncthreads();

    // ---- 2. fill: one wave; the words of row r sit in lane r and move through scalar registers, eight rows at
    //         a time (rows past the last have no bits and lead nowhere).  Every cell of row 0 and the first of
    //         every row is a seed: with the down bit of column 0 set throughout, the latter needs no step of
    //         its own, and whether a walk REACHED column 0 is the down bit as it was. ------------------------------
    unsigned long long E = nb == 64 ? ~0ull : (1ull << nb) - 1ull, D = ~0ull, G = 0ull;   // "row -1": seeds row 0
    unsigned long long dw = 0ull, rw = 0ull, gw = 0ull;
    if (wave == 1 && !no_fill && lane < nb) {
        dw = down[lane];
        rw = right[lane];
        gw = diag[lane];
    }
    auto fill_rows = [&](int first, int end) {   // multiples of 8
        if (no_fill) return;
        for (int base = first; base < end && base < nb; base += 8) {
            unsigned long long d8[8], r8[8], g8[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                d8[u] = read_lane_u64(dw | 1ull, base + u);
                r8[u] = read_lane_u64(rw, base + u);
                g8[u] = read_lane_u64(gw, base + u);
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const unsigned long long x = (E & D) | ((E & G) << 1);
                E = x | (((x & r8[u]) + r8[u]) ^ r8[u]);
                reached[base + u] = E;   // the expanded cells, for fill_done (all lanes the same word)
                D = d8[u];
                G = g8[u];
            }
        }
    };
    auto fill_done = [&]() {   // lane r: the reached word of row r
        if (no_fill) {
            reached[lane] = ~0ull;
            return;
        }
        const unsigned long long e = reached[lane];   // written by this wave
        const unsigned down0 = (unsigned)__builtin_amdgcn_update_dpp(0, (int)((unsigned)dw & 1u), 0x138 /* wave_shr:1 */,
                                                                     0xf, 0xf, false);
        reached[lane] = lane == 0 ? rw << 1 : ((e & ~1ull) | down0);
    };

    // ---- 3. threshold ----------------------------------------------------------------------------------------
    if (mode == 1) {
        unsigned long long key = 0ull;
        auto each = [&](auto&& f) {
#pragma unroll
            for (int j = 0; j < kCached; ++j) {
                int i;
                const bool ok = own_cell(j, i);
                f((unsigned long long)val[j] ^ kSign, ok);
            }
        };
        // the same keys, those of wave 1 handed to four other waves
        const int extra_row = kCached + (wave - 2);   // wave 1 owns rows 4 .. 7
        const bool extra = wave >= 2 && wave < 2 + kCached && extra_row < nb && lane < nb;
        const unsigned long long extra_key =
            extra ? (unsigned long long)pool_s[(kFinishWaves + wave - 2) * 64 + lane] ^ kSign : 0ull;
        auto each_shared = [&](auto&& f) {
            each(f);
            if (wave >= 2 && wave < 2 + kCached) f(extra_key, extra);
        };
        {
            // four cells of each of the rows 0, 4, 8, ..., spread over the columns; wave w ranks samples w, w + 16, ..
            const int rows4 = (nb + 3) >> 2, r = ((lane >> 2) * rows4) >> 4, c = ((lane & 3) * nb + (((lane >> 2) * nb) >> 4)) >> 2;
            const unsigned long long mine = (unsigned long long)pool_s[r * 64 + c] ^ kSign;
            // the wanted rank falls on sample `mid`; seven samples to either side are 2.7 standard deviations
            // of a sample's rank or more
            const int mid = (int)((unsigned)k_rank * 64u / (unsigned)n), from = mid - 7, to = mid + 7;
            if (wave != 1) {
                for (int t = wave == 0 ? 0 : wave - 1; t < 64; t += kFinishWaves - 1) {
                    const unsigned long long other = read_lane_u64(mine, t);
                    const int rank = __popcll(__ballot(mine < other || (mine == other && lane < t)));
                    if (lane == 0 && rank == from) sel.lo = other;
                    if (lane == 0 && rank == to) sel.hi = other;
                }
                if (tid == 0 && from < 0) sel.lo = 0ull;
                if (tid == 0 && to > 63) sel.hi = ~0ull;
            } else {
                fill_rows(0, 8);
            }
        }
        __syncthreads();
        const unsigned long long lo = sel.lo, width = sel.hi - lo;
        const int shift = width >> kDigitBits ? 64 - kDigitBits - __clzll((long long)width) : 0;
        if (wave != 1) {
            int n_below = 0;
            each_shared([&](unsigned long long u, bool active) {
                n_below += __popcll(__ballot(active && u < lo));
                if (active && u - lo <= width) atomicAdd(&hist[bin_slot((unsigned)((u - lo) >> shift))], 1u);
            });
            if (lane == 0 && n_below) atomicAdd(&sel.n_below, n_below);
        } else {
            fill_rows(8, 24);
        }
        __syncthreads();
        const int k = k_rank - sel.n_below;
        if (wave == 0) {
            if (k >= 0) scan_histogram(hist, k, &sel);
        } else if (wave == 1) {
            fill_rows(24, 40);
        }
        __syncthreads();
        if (sel.count > 0 && sel.count <= 64) {   // the bracket holds the rank, in a bin of few keys
            const unsigned digit = (unsigned)sel.digit;
            if (wave != 1) {
                each_shared([&](unsigned long long u, bool active) {
                    if (active && u - lo <= width && (unsigned)((u - lo) >> shift) == digit)
                        sel.cand[atomicAdd(&sel.cand_n, 1)] = u;
                });
            } else {
                fill_rows(40, 56);
            }
            __syncthreads();
            if (wave == 1) {
                fill_rows(56, 64);
                fill_done();
            }
            rank_candidates(k - sel.below, &sel);
            __syncthreads();
            key = sel.key;
        } else {
            if (wave == 1) {
                fill_rows(40, 64);
                fill_done();
            }
            key = select_kth(each, (unsigned long long)pool_s[0] ^ kSign, k_rank, hist, &sel);
        }
        if (tid == 0) {
            th.is_int = 1;
            th.ti = (long long)(key ^ kSign);
            th.td = (double)th.ti;
        }
    } else if (mode == 2) {
        // both sums in row-major order: the order is the definition.  pool_s is free from here on (its
        // rows have been compared): it holds the doubles to be added.
        // While the magnitudes add up to less than 2^53 every partial sum is an integer that a double holds, and the order of
        // the first sum does not matter: it is taken from all threads' integers.  (One dependent chain of additions of 13 clocks: 1.4 us
        // at nb = 16, 22 us at nb = 64, for each of the two sums.)
        double* const xs = reinterpret_cast<double*>(pool_s);
        if (wave == 1) {
            fill_rows(0, 64);
            fill_done();
        }
        if (row0 < nb) {   // wave-uniform
            constexpr long long kExact = 1ll << 53;
            long long sum = 0, size = 0;   // size: at most 64 x 4 times 2^53
#pragma unroll
            for (int j = 0; j < kCached; ++j) {   // cells that are not there are 0
                sum += val[j];
                const unsigned long long m = val[j] < 0 ? 0ull - (unsigned long long)val[j] : (unsigned long long)val[j];
                size += m < (unsigned long long)kExact ? (long long)m : kExact;
            }
            sum = wave_sum_i64(sum);
            size = wave_sum_i64(size);
            if (lane == 63) {
                sel.cand[wave] = (unsigned long long)sum;
                sel.cand[kFinishWaves + wave] = (unsigned long long)(size < kExact ? size : kExact);
            }
        }
#pragma unroll
        for (int j = 0; j < kCached; ++j) {
            int i;
            if (own_cell(j, i)) xs[i] = (double)val[j];
        }
        __syncthreads();
        if (wave == 0) {
            const bool there = lane < kFinishWaves && kCached * lane < nb;
            const long long sum = (long long)read_lane_u64((unsigned long long)wave_sum_i64(there ? (long long)sel.cand[lane] : 0), 63);
            const long long size = (long long)read_lane_u64((unsigned long long)wave_sum_i64(there ? (long long)sel.cand[kFinishWaves + lane] : 0), 63);
            const double mean = (size < (1ll << 53) ? (double)sum : ordered_sum(xs, n)) / (double)n;
            if (lane == 0) th.td = mean;
        }
        __syncthreads();
        const double mean = th.td;
#pragma unroll
        for (int j = 0; j < kCached; ++j) {
            int i;
            if (own_cell(j, i)) {
                const double dlt = (double)val[j] - mean;
                xs[i] = dlt * dlt;
            }
        }
        __syncthreads();
        if (wave == 0) {
            const double var = ordered_sum(xs, n) / (double)n;
            const double sd = sqrt(var);
            const double ks = kval * sd;
            if (lane == 0) {
                th.is_int = 0;
                th.ti = 0;
                th.td = mean + ks;
            }
        }
    } else {
        if (wave == 1) {
            fill_rows(0, 64);
            fill_done();
        }
        if (tid == 0) {
            th.is_int = 0;
            th.ti = 0;
            th.td = t_abs;
        }
    }
    __syncthreads();
    const Thresh t = th;
    const bool want_bsc = col_ptr != nullptr;

    // ---- 4. fl_out = reached and above the threshold, or on the diagonal: a word per row and per column -------
#pragma unroll
    for (int j = 0; j < kCached; ++j) {
        const int r = row0 + j;
        if (r >= nb) continue;   // wave-uniform
        const unsigned long long ab = __ballot(lane < nb && above(val[j], t));
        const unsigned long long f = (ab & reached[r]) | (1ull << r);
        if (lane < nb) fl[r * nb + lane] = (uint8_t)((f >> lane) & 1ull);
        if (lane == 0) rowmask[r] = f;
    }
    __syncthreads();
    {
        // the column words: lane r holds row r's word, a ballot over bit c is column c; wave w makes the
        // columns w, w + 16, ...
        const unsigned long long rm = lane < nb ? rowmask[lane] : 0ull;
        for (int c = wave; c < nb; c += kFinishWaves) {
            const unsigned long long cm = __ballot(((rm >> c) & 1ull) != 0ull);
            if (lane == 0) colmask[c] = cm;
        }
    }
    __syncthreads();

    // ---- 5. compaction: every kept cell finds its place in BSR and BSC from population counts ------------------
    int total = 0;
    if (wave == 0) {
        const int v = lane < nb ? __popcll(rowmask[lane]) : 0;
        const int incl = wave_inclusive_scan_dpp(v);
        total = __builtin_amdgcn_readlane(incl, 63);
        if (lane < nb) {
            line_start[lane] = incl - v;
            row_ptr[lane] = incl - v;
        }
        if (lane == 63) {
            row_ptr[nb] = incl;
            *nnzb_out = incl;
        }
    } else if (wave == 1 && want_bsc) {
        const int v = lane < nb ? __popcll(colmask[lane]) : 0;
        const int incl = wave_inclusive_scan_dpp(v);
        if (lane < nb) {
            col_start[lane] = incl - v;
            col_ptr[lane] = incl - v;
        }
        if (lane == 63) col_ptr[nb] = incl;
    }
    __syncthreads();
    for (int r = wave; r < nb; r += kFinishWaves) {
        const int c = lane;
        const unsigned long long rm = rowmask[r];
        if (c < nb && ((rm >> c) & 1ull)) {
            const int k = line_start[r] + __popcll(rm & ((1ull << c) - 1ull));
            col_idx[k] = c;
            if (want_bsc) {
                const int k2 = col_start[c] + __popcll(colmask[c] & ((1ull << r) - 1ull));
                row_idx[k2] = r;
                bsr_pos[k2] = k;
            }
        }
    }
    if (nnzb_host) {
        // A host that has seen the word may go on with the pattern on any stream, so the stores have to have left
        // this XCD's L2 by then: every wave's have reached it, then one release writes them back.
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) __hip_atomic_store(nnzb_host, total, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// ------------------------------------------------------------------------------------------------
// threshold + fill + compaction, 64 < nb <= 1024 (several kernels)
// ------------------------------------------------------------------------------------------------
// Words of 64 columns: W = ceil(nb / 64) per row.  Scratch of the stages, all in the workspace:
//   cells      grid_pool_kernel: pool_sum; for a quantile also a histogram over bins that grow with the value (grid_bins.h)
//   candidates grid_bits_kernel: successor bits of every row; the cells of the bin that holds the wanted
//              rank, in any order
//   serial     grid_serial_kernel: workgroup 0 the threshold (order statistic of the candidates), workgroup
//              1 the fill (the expanded cells of every row): neither needs the other
//   words      grid_words_kernel: kept bits per row and, transposed, per column, and their counts
//   index      grid_index_kernel: BSR and BSC
// Measured at nb = 512: the five kernels take 7 + 5 + 19 + 5 + 4 us (one workgroup with a barrier per
// anti-diagonal took 2454); the longest part is the serial one, its threshold and its fill about alike.
constexpr int kGridMax = 1024;   // same bound as SPION_MAX_NB of the public header

struct GridScratch {
    unsigned* hist;              // kGridBins + 4 (counter of the candidates, rank inside the bin), zeroed
    Thresh* th;
    unsigned long long* cand;    // nb * nb keys (over the slot sums, which are used up by then), behind them
    uint4 *row_cnt, *col_cnt;    // nb lines: kept cells of each word, a byte a word
    unsigned long long *down, *right, *diag, *reached, *kept, *kept_t;   // nb * W words each
};
constexpr int kGridZeroWords = kGridBins + 4;
static_assert(kGridMax / 64 <= (int)sizeof(uint4), "a byte for every word of a line");

static size_t grid_aux_bytes(size_t nb) {
    const size_t words = nb * ((nb + 63) / 64);
    return (kGridZeroWords * 4 + 255) / 256 * 256 + 256 + 6 * words * 8;
}
static GridScratch grid_carve(char* aux, void* part, size_t nb) {
    const size_t words = nb * ((nb + 63) / 64);
    GridScratch s;
    s.hist = reinterpret_cast<unsigned*>(aux);
    char* p = aux + (kGridZeroWords * 4 + 255) / 256 * 256;
    s.th = reinterpret_cast<Thresh*>(p);
    s.down = reinterpret_cast<unsigned long long*>(p + 256);
    s.right = s.down + words;
    s.diag = s.right + words;
    s.reached = s.diag + words;
    s.kept = s.reached + words;
    s.kept_t = s.kept + words;
    s.cand = static_cast<unsigned long long*>(part);
    s.row_cnt = reinterpret_cast<uint4*>(s.cand + (nb * nb + 1) / 2 * 2);   // 32 nb bytes, of 48 nb^2 that are left
    s.col_cnt = s.row_cnt + nb;
    return s;
}

__global__ __launch_bounds__(256) void grid_zero_kernel(unsigned* __restrict__ zero) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < kGridZeroWords) zero[i] = 0u;
}

// A thread takes CELLS cells, all their loads in flight together.  Bound by the latency of the short steps, and by the
// additions to the histogram, whose lines pass between the XCDs' L2s: 256 threads of 4 cells took 9.5 us at nb = 512 and
// 5.2 at 128, 1024 threads of 1 / 2 / 4 cells 8.7 / 7.0 / 8.1 and 4.0 / 4.9 / 6.6 (at 256: 4.0 / 4.8 / 6.6).
constexpr int kPoolThreads = 1024;
template <int CELLS>
__global__ __launch_bounds__(kPoolThreads) void grid_pool_kernel(const long long* __restrict__ part, long long* pool, int nb,
                                                        int want_hist, unsigned* __restrict__ hist) {
    __shared__ unsigned h[kGridBins];
    const int tid = threadIdx.x, n = nb * nb;
    if (want_hist) {
        for (int i = tid; i < kGridBins; i += kPoolThreads) h[i] = 0u;
        __syncthreads();
    }
    long long v[CELLS];
    if (part) {
        PoolParts rec[CELLS];
#pragma unroll
        for (int j = 0; j < CELLS; ++j) {
            const int i = blockIdx.x * (CELLS * kPoolThreads) + j * kPoolThreads + tid, c = i < n ? i : n - 1;
            rec[j] = load_parts(part, nb, c / nb, c % nb);
        }
#pragma unroll
        for (int j = 0; j < CELLS; ++j) {
            const int i = blockIdx.x * (CELLS * kPoolThreads) + j * kPoolThreads + tid, c = i < n ? i : n - 1;
            v[j] = sum_parts(rec[j], nb, c / nb, c % nb);
            if (i < n) pool[i] = v[j];
        }
    } else {
#pragma unroll
        for (int j = 0; j < CELLS; ++j) {
            const int i = blockIdx.x * (CELLS * kPoolThreads) + j * kPoolThreads + tid;
            v[j] = pool[i < n ? i : n - 1];
        }
    }
    if (!want_hist) return;
#pragma unroll
    for (int j = 0; j < CELLS; ++j) {
        const bool ok = blockIdx.x * (CELLS * kPoolThreads) + j * kPoolThreads + tid < n;
        const int b = grid_bin(v[j]);
        const unsigned long long m = __ballot(ok);
        if (m == 0ull) continue;
        const int first = __builtin_amdgcn_readlane(b, __ffsll((long long)m) - 1);
        if (__ballot(ok && b == first) == m) {   // one bin for the whole wave: one atomic
            if ((tid & 63) == 0) atomicAdd(&h[first], (unsigned)__popcll(m));
        } else if (ok) {
            atomicAdd(&h[b], 1u);
        }
    }
    __syncthreads();
    for (int i = tid; i < kGridBins; i += kPoolThreads)
        if (h[i]) atomicAdd(&hist[i], h[i]);
}

// A wave takes a word (64 cells of a row).  Every workgroup finds the bin of the wanted rank itself, 8
// bins per thread and two scans (4096 bins: 16 a thread and four words a wave, in 256 threads, 6.5 us at nb = 512, 4 a thread 5.1),
// and takes room for its candidates with one addition: with one per wave and
// word, all on one counter, a map of 512 x 512 nearly equal cells (one bin) took 50 us,
// now 8.8.
constexpr int kBitsThreads = 1024, kBitsWords = kBitsThreads / 64;   // words of a workgroup
__global__ __launch_bounds__(kBitsThreads) void grid_bits_kernel(const long long* __restrict__ pool, int nb, int mode,
                                                        int k_rank, int no_fill, GridScratch s) {
    __shared__ int wave_sum[kBitsWords], sel_bin;
    __shared__ unsigned wave_cand[kBitsWords], cand_base;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int W = (nb + 63) >> 6, words = nb * W, word = blockIdx.x * kBitsWords + wave;
    const bool there = word < words;   // uniform
    const int r = there ? word / W : 0, c = (there ? word % W * 64 : 0) + lane;
    const bool inner = c + 1 < nb && r + 1 < nb;
    const int i = r * nb + (c < nb ? c : 0);
    const long long v = pool[i];
    const long long dn = inner && !no_fill ? pool[i + nb] : 0, rt = inner && !no_fill ? pool[i + 1] : 0,
                    dg = inner && !no_fill ? pool[i + nb + 1] : 0;
    int bin = -1;
    if (mode == 1) {
        static_assert(kGridBins == 8 * kBitsThreads, "eight bins a thread");
        const uint4 q0 = reinterpret_cast<const uint4*>(s.hist)[2 * tid], q1 = reinterpret_cast<const uint4*>(s.hist)[2 * tid + 1];
        const unsigned q[8] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w};
        int cnt = 0;
#pragma unroll
        for (int b = 0; b < 8; ++b) cnt += (int)q[b];
        const int scan = wave_inclusive_scan_dpp(cnt);
        if (lane == 63) wave_sum[wave] = scan;
        __syncthreads();
        const int sums = wave_inclusive_scan_dpp(lane < kBitsWords ? wave_sum[lane] : 0);
        const int incl = scan + (wave > 0 ? __builtin_amdgcn_readlane(sums, wave - 1) : 0);
        int e0 = incl - cnt;
        if (k_rank >= e0 && k_rank < incl) {   // exactly one thread
            int b = 0;
#pragma unroll
            for (int i = 0; i < 7; ++i) {
                if (k_rank < e0 + (int)q[i]) break;
                e0 += (int)q[i];
                ++b;
            }
            sel_bin = tid * 8 + b;
            if (blockIdx.x == 0) s.hist[kGridBins + 1] = (unsigned)(k_rank - e0);   // rank among the candidates
        }
        __syncthreads();
        bin = sel_bin;
    }
    if (!no_fill && there) {
        const Succ sc = successors(dn, rt, dg, inner);
        const unsigned long long bd = __ballot(sc.down), br = __ballot(sc.right), bg = __ballot(sc.diag);
        if (lane == 0) {
            s.down[word] = bd;
            s.right[word] = br;
            s.diag[word] = bg;
        }
    }
    if (mode != 1) return;
    const bool mine = there && c < nb && grid_bin(v) == bin;
    const unsigned long long m = __ballot(mine);
    if (lane == 0) wave_cand[wave] = (unsigned)__popcll(m);
    __syncthreads();
    const int found = wave_inclusive_scan_dpp(lane < kBitsWords ? (int)wave_cand[lane] : 0);
    if (tid == 0) {
        const unsigned all = (unsigned)__builtin_amdgcn_readlane(found, kBitsWords - 1);
        cand_base = all ? atomicAdd(&s.hist[kGridBins], all) : 0u;
    }
    __syncthreads();
    if (mine)
        s.cand[cand_base + (unsigned)(wave > 0 ? __builtin_amdgcn_readlane(found, wave - 1) : 0) + (unsigned)__popcll(m & ((1ull << lane) - 1ull))] =
            (unsigned long long)v ^ kSign;
}

// The fill on rows of up to 1024 bits: lane l of wave 0 holds columns 32 l .. 32 l + 31 and is l rows behind lane 0.
// In step t it works on row t - l, for which its left neighbour found the carry out of the row's addition one step before
// and the last column of the row above two steps before: the one reaches it as a bit set in scalar registers, shifted
// by one lane, the other as a lane shift, both away from the chain of the step.
// (All lanes on one row, the carries resolved by a second addition on the bit set of lanes that generate one, took
// 225 cycles a row: the kernel 49 us at nb = 512.)  Bound by the wave's own issue, an instruction every 6 to 7 cycles
// whether or not it depends on the one before: so the other waves bring the words as the step takes them, the diagonal
// bits in their target's place, the seeds in, and four steps' words of a lane side by side in LDS.  A step is eight
// vector instructions, a scalar one and one access to LDS instead of 14 (115 -> 62 cycles, the kernel 29 -> 19 us at
// nb = 512).  They also store what was found in the steps before, which takes the place of the words of `right`: a
// trip to memory takes longer than many steps.
constexpr int kFillSteps = 64;
constexpr int kFillLd = kGridMax / 32;                  // words of a step in LDS, used or not
constexpr int kFillPlane = kFillSteps * kFillLd;        // one array's words of a piece
constexpr int kFillWords = 2 * 3 * kFillPlane;          // two pieces of down, diagonal, right

__device__ void grid_fill(const GridScratch& s, int nb, unsigned* buf /* kFillWords, LDS, 16-byte aligned */) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int W2 = 2 * ((nb + 63) >> 6);   // 32-bit words per row
    const int pieces = (nb + W2 - 1 + kFillSteps - 1) / kFillSteps;
    constexpr int kOwn = (kFillPlane + kFinishThreads - 65) / (kFinishThreads - 64);   // words of a thread
    const unsigned *const down = reinterpret_cast<const unsigned*>(s.down), *const right = reinterpret_cast<const unsigned*>(s.right),
                   *const diag = reinterpret_cast<const unsigned*>(s.diag);
    // One piece further for the threads from `first` on: store the words found in piece - 2, bring those of `piece`: what
    // lets a cell of the row above down and diagonally into the lane's word of row r, and what lets one of r on to the right.
    // Rows above the first pass on what they are given; rows behind the last take nothing.
    auto exchange = [&](int piece, int first, int threads) {
        unsigned* const at = buf + (piece & 1) * 3 * kFillPlane;
        unsigned w[kOwn][4];
        if (piece < pieces) {
#pragma unroll
            for (int e = 0; e < kOwn; ++e) {
                const int i = tid - first + e * threads, l = i % kFillLd, row = piece * kFillSteps + i / kFillLd - l;
                const bool there = i < kFillPlane && l < W2 && row >= 0 && row < nb, above = there && row > 0;
                const size_t here = (size_t)row * W2 + l;
                w[e][0] = above ? down[here - W2] : (row <= 0 ? ~0u : 0u);
                w[e][1] = above ? diag[here - W2] : 0u;
                w[e][2] = above && l > 0 ? diag[here - W2 - 1] : 0u;
                w[e][3] = there ? right[here] : 0u;
            }
        }
#pragma unroll
        for (int e = 0; e < kOwn; ++e) {
            const int i = tid - first + e * threads, l = i % kFillLd, t = i / kFillLd, row = (piece - 2) * kFillSteps + t - l;
            if (i >= kFillPlane || l >= W2) continue;
            unsigned* const slot = at + (t >> 2) * (4 * kFillLd) + 4 * l + (t & 3);
            if (piece >= 2 && row >= 0 && row < nb) reinterpret_cast<unsigned*>(s.reached)[(size_t)row * W2 + l] = slot[2 * kFillPlane];
            if (piece < pieces) {
                slot[0] = w[e][0] | (l == 0 ? 1u : 0u);   // the first cell of every row is a seed
                slot[kFillPlane] = w[e][1] << 1 | w[e][2] >> 31;
                slot[2 * kFillPlane] = w[e][3];
            }
        }
    };
    auto meet = [&]() {   // LDS only: the stores of the words already found need not be waited for
        __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    if (wave != 0) exchange(0, 64, kFinishThreads - 64);
    meet();
    const int first_col = 32 * lane;
    // "row -1": every cell of row 0 is a seed
    unsigned E = first_col >= nb ? 0u : (nb - first_col >= 32 ? ~0u : (1u << (nb - first_col)) - 1u);
    unsigned E_before = 0u;                 // E of the step before
    unsigned carry_lanes = 0u;              // lanes that have a carry to give
    for (int piece = 0; piece < pieces; ++piece) {
        if (wave != 0) {
            exchange(piece + 1, 64, kFinishThreads - 64);
        } else if (lane < kFillLd) {
            typedef unsigned Word4 __attribute__((ext_vector_type(4)));
            Word4* const src = reinterpret_cast<Word4*>(buf + (piece & 1) * 3 * kFillPlane) + lane;
            // (behind the branch a value per lane to the compiler: a scalar again before the instruction that needs one)
            unsigned long long carry = (unsigned)__builtin_amdgcn_readfirstlane((int)carry_lanes);
            constexpr int U = 4;   // steps whose words are requested together, one group ahead
            Word4 d[2], g[2], q[2];
            auto request = [&](int h, int group) {
                d[h] = src[group * kFillLd];
                g[h] = src[group * kFillLd + kFillPlane / 4];
                q[h] = src[group * kFillLd + kFillPlane / 2];
                __builtin_amdgcn_sched_barrier(0);
            };
            auto work = [&](int h, int group) {
                Word4 found;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const unsigned prev = (unsigned)__builtin_amdgcn_update_dpp(0, (int)E_before, 0x138 /* wave_shr:1 */, 0xf, 0xf, true);
                    const unsigned shifted = __builtin_amdgcn_alignbit(E, prev, 31);
                    // to the neighbours; not next to the addition, whose result it would wait for
                    asm("s_lshl_b64 %0, %0, 1" : "+s"(carry) : "v"(shifted) : "scc");
                    const unsigned x = (E & d[h][u]) | (shifted & g[h][u]);
                    const unsigned R = q[h][u];
                    unsigned sum;
                    asm("v_addc_co_u32 %0, %1, %2, %3, %1" : "=v"(sum), "+s"(carry) : "v"(x & R), "v"(R));
                    E_before = E;
                    E = __builtin_amdgcn_bitop3_b32(x, sum, R, 0xF6);   // x | (sum ^ R): the compiler splits it up over two steps
                    found[u] = E;
                }
                src[group * kFillLd + kFillPlane / 2] = found;
                __builtin_amdgcn_sched_barrier(0);
            };
            constexpr int kGroups = kFillSteps / U;
            request(0, 0);
#pragma unroll 1
            for (int group = 0; group < kGroups; group += 2) {
                request(1, group + 1);
                work(0, group);
                request(0, (group + 2) & (kGroups - 1));   // behind the last group: the first again, unused
                work(1, group + 1);
            }
            carry_lanes = (unsigned)carry;   // of 32 lanes
        }
        meet();
    }
    if (wave != 0) exchange(pieces + 1, 64, kFinishThreads - 64);   // piece - 1 is stored, nothing is brought
}

__global__ __launch_bounds__(kFinishThreads) void grid_serial_kernel(const long long* __restrict__ pool, int nb, int mode,
                                                                     double kval, double t_abs, int no_fill,
                                                                     GridScratch s) {
    __shared__ __attribute__((aligned(16))) unsigned hist[kFillWords > 3 * kBins ? kFillWords : 3 * kBins];   // or the fill's words
    __shared__ SelectShared sel;
    __shared__ double part_s;
    const int tid = threadIdx.x, n = nb * nb;
    if (blockIdx.x == 1) {
        const int words = nb * ((nb + 63) >> 6);
        if (no_fill) {
            for (int i = tid; i < words; i += kFinishThreads) s.reached[i] = ~0ull;
        } else {
            grid_fill(s, nb, hist);
        }
        return;
    }
    Thresh t = {0, 0, t_abs};
    if (mode == 1) {
        const int m = (int)s.hist[kGridBins];
        const unsigned long long key = select_kth(
            [&](auto&& f) {
                constexpr int kFlight = 16;   // keys requested before the first is used
                for (int base = 0; base < m; base += kFlight * kFinishThreads) {
                    unsigned long long u[kFlight];
#pragma unroll
                    for (int e = 0; e < kFlight; ++e) {
                        const int i = base + e * kFinishThreads + tid;
                        u[e] = s.cand[i < m ? i : 0];
                    }
#pragma unroll
                    for (int e = 0; e < kFlight; ++e) {
                        const int i = base + e * kFinishThreads + tid;
                        if (base + e * kFinishThreads < m) f(u[e], i < m);   // uniform
                    }
                }
            },
            s.cand[0], (int)s.hist[kGridBins + 1], hist, &sel);
        t.is_int = 1;
        t.ti = (long long)(key ^ kSign);
        t.td = (double)t.ti;
    } else if (mode == 2) {
        // sequential sums in row-major order (the order is the definition), staged through LDS in pieces
        double* const xs = reinterpret_cast<double*>(hist);
        constexpr int kPiece = 3072;
        static_assert(kPiece * 8 <= 3 * kBins * 4 && kPiece % 16 == 0, "the piece must fit");
        double mean = 0.0, acc = 0.0;
        for (int round = 0; round < 2; ++round) {
            acc = 0.0;
            for (int base = 0; base < n; base += kPiece) {
                const int len = n - base < kPiece ? n - base : kPiece;
                __syncthreads();
                for (int i = tid; i < len; i += kFinishThreads) {
                    const double x = (double)pool[base + i], dlt = x - mean;
                    xs[i] = round == 0 ? x : dlt * dlt;
                }
                __syncthreads();
                if (tid < 64) {
                    for (int i = 0; i < len; i += 16) {
                        double v[16];
                        const int left = len - i;
#pragma unroll
                        for (int e = 0; e < 16; ++e) v[e] = xs[i + (e < left ? e : 0)];
                        if (left >= 16) {
#pragma unroll
                            for (int e = 0; e < 16; ++e) acc = acc + v[e];
                        } else {
                            for (int e = 0; e < left; ++e) acc = acc + xs[i + e];
                        }
                    }
                }
            }
            if (tid == 0) part_s = acc;
            __syncthreads();
            acc = part_s / (double)n;
            if (round == 0) mean = acc;
        }
        const double sd = sqrt(acc);
        const double ks = kval * sd;
        t.td = mean + ks;
    }
    if (tid == 0) *s.th = t;
}

// One workgroup per 64 x 64 tile of cells: wave w its rows 4 w .. 4 w + 3, one ballot each; the 64 words,
// transposed by 64 more ballots, are 64 column words.  How many cells a word keeps is stored as a byte beside those of
// the line's other words: counters per line that the workgroups add to are lines of memory that pass from one XCD's L2
// to the next with every addition (12.5 us at any size; 8.2 with a byte a word, 4.8 with
// four rows a wave instead of sixteen: a wave alone issues an instruction every 6 cycles).
__global__ __launch_bounds__(1024) void grid_words_kernel(const long long* __restrict__ pool, int nb, int no_fill,
                                                          GridScratch s, uint8_t* __restrict__ fl) {
    __shared__ unsigned long long tile[64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int W = (nb + 63) >> 6, rs = blockIdx.x / W, cs = blockIdx.x % W;
    const int c = cs * 64 + lane;
    const Thresh t = *s.th;
    constexpr int kRows = 4;
    long long v[kRows];
    unsigned long long reached_w = 0ull;   // lane j: the word of this wave's row j
    const int r_first = rs * 64 + wave * kRows;
    if (lane < kRows && r_first + lane < nb) {
        // a seed is not reached by being one: row 0 is from its left neighbours, column 0 from above
        const int r = r_first + lane;
        reached_w = s.reached[r * W + cs];
        if (!no_fill && r == 0)
            reached_w = s.right[cs] << 1 | (cs > 0 ? s.right[cs - 1] >> 63 : 0ull);
        else if (!no_fill && cs == 0)
            reached_w = (reached_w & ~1ull) | (s.down[(r - 1) * W] & 1ull);
    }
#pragma unroll
    for (int j = 0; j < kRows; ++j) {
        const int r = r_first + j;
        v[j] = pool[r < nb && c < nb ? r * nb + c : 0];
    }
#pragma unroll
    for (int j = 0; j < kRows; ++j) {
        const int r = rs * 64 + wave * kRows + j;
        unsigned long long f = 0ull;
        if (r < nb) {   // wave-uniform
            const bool ab = c < nb && above(v[j], t);
            f = __ballot(ab) & read_lane_u64(reached_w, j);
            if (r >> 6 == cs) f |= 1ull << (r & 63);
            if (c < nb) fl[(size_t)r * nb + c] = (uint8_t)((f >> lane) & 1ull);
            if (lane == 0) {
                s.kept[r * W + cs] = f;
                reinterpret_cast<uint8_t*>(s.row_cnt + r)[cs] = (uint8_t)__popcll(f);
            }
        }
        if (lane == 0) tile[wave * kRows + j] = f;
    }
    __syncthreads();
    const unsigned long long rw = tile[lane];
#pragma unroll
    for (int j = 0; j < kRows; ++j) {
        const int cc = cs * 64 + wave * kRows + j;
        const unsigned long long m = __ballot(((rw >> (wave * kRows + j)) & 1ull) != 0ull);
        if (lane == 0 && cc < nb) {
            s.kept_t[cc * W + rs] = m;
            reinterpret_cast<uint8_t*>(s.col_cnt + cc)[rs] = (uint8_t)__popcll(m);
        }
    }
}

// Sum of the first n bytes (n uniform).
__device__ __forceinline__ int sum_bytes(uint4 v, int n) {
    auto first = [n](unsigned w, int k) { return n >= 4 * k + 4 ? w : n <= 4 * k ? 0u : w & ((1u << (8 * (n - 4 * k))) - 1u); };
    const unsigned lo = __builtin_amdgcn_sad_u8(first(v.y, 1), 0u, __builtin_amdgcn_sad_u8(first(v.x, 0), 0u, 0u));
    return (int)__builtin_amdgcn_sad_u8(first(v.w, 3), 0u, __builtin_amdgcn_sad_u8(first(v.z, 2), 0u, lo));
}

// One wave per row (BSR) and, behind them, one per column (BSC).  A wave adds up the counts of the lines before its own;
// where the row-wise index holds a cell of a column follows from its row's start, the counts of the words before the
// cell's and that word.  Bound by latency: everything a wave needs is requested at once (at nb = 512, the words before a
// cell's one after the other: 9.5 us, 4.4 so).
template <int GROUPS>   // groups of 64 lines, at least W
__global__ __launch_bounds__(256) void grid_index_kernel(int nb, GridScratch s, int* __restrict__ row_ptr,
                                                         int* __restrict__ col_idx, int* __restrict__ col_ptr,
                                                         int* __restrict__ row_idx, int* __restrict__ bsr_pos,
                                                         int* __restrict__ nnzb_out, int* nnzb_host) {
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
    const int W = (nb + 63) >> 6;
    if (w >= (col_ptr ? 2 * nb : nb)) return;
    const bool cols = w >= nb;
    const int line = cols ? w - nb : w, word = line >> 6;
    const uint4* const cnt = cols ? s.col_cnt : s.row_cnt;
    uint4 before[GROUPS], rows[GROUPS];
    unsigned long long cell[GROUPS];   // columns: the word of row 64 q + lane that holds the cell
#pragma unroll
    for (int q = 0; q < GROUPS; ++q) {
        const int i = q * 64 + lane;
        before[q] = i < line ? cnt[i] : make_uint4(0u, 0u, 0u, 0u);
        rows[q] = cols && i < nb ? s.row_cnt[i] : make_uint4(0u, 0u, 0u, 0u);
        cell[q] = cols && i < nb ? s.kept[(size_t)i * W + word] : 0ull;
    }
    const unsigned long long words = lane < W ? (cols ? s.kept_t : s.kept)[line * W + lane] : 0ull;
    const int own = sum_bytes(cnt[line], W);
    int sum = 0;
#pragma unroll
    for (int q = 0; q < GROUPS; ++q) sum += sum_bytes(before[q], W);
    int k = __builtin_amdgcn_readlane(wave_inclusive_scan_dpp(sum), 63);
    int* const ptr = cols ? col_ptr : row_ptr;
    if (lane == 0) {
        ptr[line] = k;
        if (line == nb - 1) {
            const int total = k + own;
            ptr[nb] = total;
            if (!cols) {
                *nnzb_out = total;
                if (nnzb_host) __hip_atomic_store(nnzb_host, total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            }
        }
    }
    int run = 0;   // kept cells of the rows before this group of 64 (columns only)
#pragma unroll
    for (int seg = 0; seg < GROUPS; ++seg) {
        if (seg < W) {   // uniform
            const unsigned long long m = read_lane_u64(words, seg);
            const bool bit = ((m >> lane) & 1ull) != 0ull;
            const int pos = k + __popcll(m & ((1ull << lane) - 1ull));
            const int other = seg * 64 + lane;
            if (!cols) {
                if (bit) col_idx[pos] = other;
            } else {
                const int rc = sum_bytes(rows[seg], W);
                const int incl = wave_inclusive_scan_dpp(rc);
                if (bit) {
                    row_idx[pos] = other;
                    bsr_pos[pos] = run + incl - rc + sum_bytes(rows[seg], word) +
                                   __popcll(cell[seg] & ((1ull << (line & 63)) - 1ull));
                }
                run += __builtin_amdgcn_readlane(incl, 63);
            }
            k += __popcll(m);
        }
    }
}

// ------------------------------------------------------------------------------------------------
// index check (one workgroup)
// ------------------------------------------------------------------------------------------------
// The attention kernels trust their index: an entry out of range there is an access out of bounds.
// An index that did not come from pattern_finish_kernel can be checked here first.  Three stages,
// each reading only what the stage before has shown to be in range: (1) the pointer arrays run
// from 0 to nnzb without decreasing; (2) the entries of every row (column) lie in [0, nb) and
// ascend strictly; (3) every entry of the transposed index names a position of the row-wise index
// that lies in the row it claims and holds the column it claims (with equal counts and distinct
// (row, column) pairs, that makes the transposed index the exact transpose).
__global__ __launch_bounds__(1024) void index_check_kernel(
    const int* __restrict__ row_ptr, const int* __restrict__ col_idx, const int* __restrict__ col_ptr,
    const int* __restrict__ row_idx, const int* __restrict__ bsr_pos, int nb, int nnzb, int err_code,
    int* __restrict__ status) {
    __shared__ int bad;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n_waves = blockDim.x >> 6;
    if (tid == 0) bad = 0;
    __syncthreads();
    auto pointers_ok = [&](const int* ptr) {
        bool ok = true;
        for (int i = tid; i < nb; i += blockDim.x) {
            const int a = ptr[i], b = ptr[i + 1];
            ok = ok && a >= 0 && b >= a && b <= nnzb;
        }
        if (tid == 0) ok = ok && ptr[0] == 0 && ptr[nb] == nnzb;
        return ok;
    };
    if (!pointers_ok(row_ptr)) bad = 1;
    if (col_ptr && !pointers_ok(col_ptr)) bad = 1;
    __syncthreads();
    if (bad) {
        if (tid == 0) *status = err_code;
        return;
    }
    auto entries_ok = [&](const int* ptr, const int* idx) {
        bool ok = true;
        for (int i = wave; i < nb; i += n_waves) {
            const int a = ptr[i], b = ptr[i + 1];
            for (int k = a + lane; k < b; k += 64) {
                const int c = idx[k];
                ok = ok && c >= 0 && c < nb && (k == a || idx[k - 1] < c);
            }
        }
        return ok;
    };
    if (!entries_ok(row_ptr, col_idx)) bad = 1;
    if (col_ptr && !entries_ok(col_ptr, row_idx)) bad = 1;
    __syncthreads();
    if (bad) {
        if (tid == 0) *status = err_code;
        return;
    }
    if (col_ptr) {
        bool ok = true;
        for (int j = wave; j < nb; j += n_waves) {
            const int a = col_ptr[j], b = col_ptr[j + 1];
            for (int k = a + lane; k < b; k += 64) {
                const int i = row_idx[k], pos = bsr_pos[k];
                ok = ok && pos >= row_ptr[i] && pos < row_ptr[i + 1] && col_idx[pos] == j;
            }
        }
        if (!ok) bad = 1;
    }
    __syncthreads();
    if (tid == 0) *status = bad ? err_code : 0;
}

// ------------------------------------------------------------------------------------------------
// host launchers
// ------------------------------------------------------------------------------------------------
size_t pattern_part_bytes(size_t nb) { return kSlots * nb * nb * sizeof(long long); }
size_t pattern_aux_bytes(size_t nb) { return nb > 64 ? grid_aux_bytes(nb) : 0; }

hipError_t launch_conv_pool(const float* A, int L, int bs, int p, long long* part, void* aux, hipStream_t st) {
    const int nb = L / bs, per_tile = 64 / bs;
    const unsigned tiles = (unsigned)nb * (unsigned)((nb + per_tile - 1) / per_tile);
    const dim3 grid((tiles + 3) / 4);
    // the counters of the grid kernels are cleared on the way; with more than 64 block rows the grid has
    // more than enough threads for that
    unsigned* const zero = static_cast<unsigned*>(nb > 64 ? aux : nullptr);
    const int n_zero = zero ? kGridZeroWords : 0;
    static_assert(65 * ((65 + 3) / 4) / 4 * 256 >= kGridZeroWords, "one thread per cleared word");
    if (bs == 16)
        conv_pool_kernel<16><<<grid, dim3(256), 0, st>>>(A, L, p, part, zero, n_zero);
    else if (bs == 32)
        conv_pool_kernel<32><<<grid, dim3(256), 0, st>>>(A, L, p, part, zero, n_zero);
    else
        conv_pool_kernel<64><<<grid, dim3(256), 0, st>>>(A, L, p, part, zero, n_zero);
    return hipGetLastError();
}

hipError_t launch_pool_gather(const long long* part, int nb, long long* pool, hipStream_t st) {
    pool_gather_kernel<<<dim3((unsigned)((nb * nb + 255) / 256)), dim3(256), 0, st>>>(part, nb, pool);
    return hipGetLastError();
}

hipError_t launch_pattern_finish(bool from_part, long long* part, long long* pool, int nb, int mode, long long k_rank,
                                 double kval, double t_abs, int no_fill, void* aux, uint8_t* fl, int* row_ptr,
                                 int* col_idx, int* col_ptr, int* row_idx, int* bsr_pos, int* nnzb, int* nnzb_host,
                                 hipStream_t st) {
    const long long* const src = from_part ? part : nullptr;
    if (nb <= 64) {   // one workgroup, a wave instruction per row: 64 columns are its limit
        pattern_finish_kernel<<<dim3(1), dim3(kFinishThreads), 0, st>>>(src, pool, nb, mode, (int)k_rank, kval, t_abs,
                                                                        no_fill, fl, row_ptr, col_idx, col_ptr,
                                                                        row_idx, bsr_pos, nnzb, nnzb_host);
        return hipGetLastError();
    }
    const GridScratch s = grid_carve(static_cast<char*>(aux), part, (size_t)nb);
    const unsigned n = (unsigned)(nb * nb), W = (unsigned)((nb + 63) / 64), words = (unsigned)nb * W;
    if (!from_part) grid_zero_kernel<<<dim3((kGridZeroWords + 255) / 256), dim3(256), 0, st>>>(s.hist);
    if (from_part || mode == 1) {
        if (nb <= 256)
            grid_pool_kernel<1><<<dim3((n + kPoolThreads - 1) / kPoolThreads), dim3(kPoolThreads), 0, st>>>(src, pool, nb, mode == 1, s.hist);
        else
            grid_pool_kernel<2><<<dim3((n + 2 * kPoolThreads - 1) / (2 * kPoolThreads)), dim3(kPoolThreads), 0, st>>>(src, pool, nb, mode == 1, s.hist);
    }
    grid_bits_kernel<<<dim3((words + kBitsWords - 1) / kBitsWords), dim3(kBitsThreads), 0, st>>>(pool, nb, mode, (int)k_rank, no_fill, s);
    grid_serial_kernel<<<dim3(2), dim3(kFinishThreads), 0, st>>>(pool, nb, mode, kval, t_abs, no_fill, s);
    grid_words_kernel<<<dim3(W * W), dim3(1024), 0, st>>>(pool, nb, no_fill, s, fl);
    const unsigned lines = (unsigned)(col_ptr ? 2 * nb : nb);
    auto* const index = W <= 4 ? grid_index_kernel<4> : W <= 8 ? grid_index_kernel<8> : grid_index_kernel<16>;
    index<<<dim3((lines + 3) / 4), dim3(256), 0, st>>>(nb, s, row_ptr, col_idx, col_ptr, row_idx, bsr_pos, nnzb, nnzb_host);
    return hipGetLastError();
}

hipError_t launch_index_check(const int* row_ptr, const int* col_idx, const int* col_ptr, const int* row_idx,
                              const int* bsr_pos, int nb, int nnzb, int err_code, int* status, hipStream_t st) {
    index_check_kernel<<<dim3(1), dim3(1024), 0, st>>>(row_ptr, col_idx, col_ptr, row_idx, bsr_pos, nb, nnzb,
                                                       err_code, status);
    return hipGetLastError();
}

}  // namespace spion
