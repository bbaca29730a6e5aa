// Around the attention of the sub-layer (Algorithm 5): gradient of a projection's weight, head split and merge.
//
// dW[n][m] = sum over rows of dY[row][n] * X[row][m] has few outputs (N, M: the embedding width, or three times
// it) and a long contraction (every token of the batch).  A library product that gives each output tile to one
// workgroup leaves the chip idle: 16384 rows, 768 x 256 and 256 x 256 outputs took 91 us each (48 and 16 workgroups),
// for 34 MB and 17 MB of reads.  Here the rows are cut into slices, each slice and 128 x 128 tile of outputs a
// workgroup that writes fp32 partial sums, and a second launch adds the slices in their order (no atomics, the
// same bits every time): 24 and 20 us with both launches; 4096 rows, 512 x 512 outputs 27 -> 21, 2048 rows, 192 x 64
// 19 -> 7.5, 32768 rows, 1536 x 512 196 -> 91, 48 rows, 192 x 64 19 -> 6.5.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "attn_bf16_tiles.h"
#include "attn_common.h"
#include "spion_internal.h"

namespace spion {

namespace {

// Workgroups to aim at (one or two run on a compute unit) and rows of a slice, at least.  256 and 512 workgroups
// took 27 and 24 us for 16384 rows, 768 x 256 outputs, 19 and 21 for 256 x 256; 256 rows a slice, 8.5 instead of 7.5 us for
// 2048 rows, 192 x 64.
constexpr int kWeightGradGroups = 384;
constexpr int kWeightGradMinRows = 128;
constexpr int kTile = 128;       // outputs of a workgroup in each direction; a wave has 64 x 64 of them
constexpr int kStepRows = 32;    // rows of a step: one bf16 MFMA contracts over 32
constexpr int kLd = kTile + 16;  // elements between rows in LDS: the 16 rows x 32 B of a transpose read fall on
                                 // different banks, 8 rows at a time

// Bound by the latency of the loads (a step is 16 MFMAs a wave and 16 KB): rows are requested two steps ahead into
// registers and one step ahead into LDS, one barrier a step.  Rows behind the last
// are read as the last and count nothing, columns beside the last as the tile's first and are not written.
__global__ __launch_bounds__(256) void weight_grad_kernel(const bf16_t* __restrict__ dY, const bf16_t* __restrict__ X,
                                                          float* __restrict__ partial, int rows, int N, int M,
                                                          int slices, int slice_rows, int tiles_n, int tiles_m) {
    __shared__ __attribute__((aligned(16))) bf16_t ys[2][kStepRows * kLd], xs[2][kStepRows * kLd];
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // the tiles of a slice on one XCD: they read the same rows
    const int tiles = tiles_n * tiles_m, l = blockIdx.x >> 3;
    const int slice = l / tiles * 8 + (blockIdx.x & 7), tile = l % tiles;
    if (slice >= slices) return;
    const int n0 = tile / tiles_m * kTile, m0 = tile % tiles_m * kTile;
    const int first = slice * slice_rows, end = min(rows, first + slice_rows);

    // a thread brings 16 bytes of rows row, row + 16 of both matrices
    const int row = tid >> 4, col = (tid & 15) * 8;
    const bool has_n = n0 + col < N, has_m = m0 + col < M;
    const bf16_t* const py = dY + n0 + (has_n ? col : 0);
    const bf16_t* const px = X + m0 + (has_m ? col : 0);
    struct Rows {
        bf16x8 y[2], x[2];
    };
    auto request = [&](Rows& v, int at) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const size_t i = (size_t)min(at + row + 16 * k, end - 1);   // no branch: the loads stay in flight over it
            v.y[k] = *reinterpret_cast<const bf16x8*>(py + i * N);
            v.x[k] = *reinterpret_cast<const bf16x8*>(px + i * M);
        }
    };
    auto put = [&](Rows& v, int at, int b) {
        if (at + kStepRows > end) {   // uniform; rows behind the last count nothing
#pragma unroll
            for (int k = 0; k < 2; ++k)
                if (at + row + 16 * k >= end) v.y[k] = v.x[k] = bf16x8{};
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            *reinterpret_cast<bf16x8*>(&ys[b][(row + 16 * k) * kLd + col]) = v.y[k];
            *reinterpret_cast<bf16x8*>(&xs[b][(row + 16 * k) * kLd + col]) = v.x[k];
        }
    };
    const int wn = (wave >> 1) * 64, wm = (wave & 1) * 64;
    const int tr = (4 * g + (r >> 2)) * kLd + 4 * (r & 3);   // transpose read: lane r receives column r of rows 4 g ..
    f32x4 acc[4][4];   // [n tile][m tile]
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](int b) {
        bf16x8 fy[4], fx[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const bf16_t* const y = &ys[b][tr + wn + 16 * t];
            const bf16_t* const x = &xs[b][tr + wm + 16 * t];
            fy[t] = join(lds_read_tr(y), lds_read_tr(y + 16 * kLd));
            fx[t] = join(lds_read_tr(x), lds_read_tr(x + 16 * kLd));
        }
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[a][c] = mma_d(acc[a][c], fx[c], fy[a]);   // [m][n]
    };
    // LDS only: __syncthreads would also wait for the rows requested ahead
    auto meet = [&]() {
        __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    const int steps = (end - first + kStepRows - 1) / kStepRows;
    Rows va, vb;
    request(va, first);
    request(vb, first + kStepRows);
    put(va, first, 0);
    request(va, first + 2 * kStepRows);
    meet();
    for (int s = 0, at = first; s < steps; s += 2, at += 2 * kStepRows) {
        put(vb, at + kStepRows, 1);
        request(vb, at + 3 * kStepRows);
        multiply(0);
        meet();
        if (s + 1 >= steps) break;
        put(va, at + 2 * kStepRows, 0);
        request(va, at + 4 * kStepRows);
        multiply(1);
        meet();
    }
    float* const out = partial + (size_t)slice * N * M;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        const int n = n0 + wn + 16 * a + r;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int m = m0 + wm + 16 * c + 4 * g;
            if (n < N && m < M) *reinterpret_cast<f32x4*>(out + (size_t)n * M + m) = acc[a][c];
        }
    }
}

// A workgroup has 64 vectors of 4 outputs, a wave a quarter of their slices; the quarters are added in order.
__global__ __launch_bounds__(256) void weight_grad_sum_kernel(const float* __restrict__ partial, int slices, int n4,
                                                              bf16_t* __restrict__ dW) {
    __shared__ f32x4 part[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i = blockIdx.x * 64 + lane;
    const f32x4* const p = reinterpret_cast<const f32x4*>(partial) + (i < n4 ? i : n4 - 1);
    const int end = (wave + 1) * slices / 4;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int s = wave * slices / 4; s < end; s += 8) {
        f32x4 v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = p[(size_t)min(s + k, end - 1) * n4];
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (s + k < end) acc += v[k];
    }
    part[wave][lane] = acc;
    __syncthreads();
    if (wave == 0 && i < n4) store_quad<bf16_t>(dW + 4 * (size_t)i, ((part[0][lane] + part[1][lane]) + part[2][lane]) + part[3][lane]);
}

// Between the layout of the projections, [B, L, n, H, 64] (n = 3: Q | K | V, n = 1: the heads' outputs side by side),
// and that of the attention's kernels for fp32 and block 16, n tensors [B, H, L, 64] (the others read the projections'
// layout, HeadRows).  Bound by HBM.  A wave moves 4 pieces of 1 KB that are
// contiguous in the attention's layout (8 tokens of a head in bf16, 4 in fp32), rows of 128 or 256 bytes in the other.
// 8 x 2048 tokens, 4 heads, bf16: 8.2 us for three tensors (50 MB, out of the caches in part), 4.7 us for one.  As
// torch operators these were 8 copies of 8 us and, for the gradients of the three slices, as many fills of the whole
// and two additions: 125 us a step.
typedef unsigned Vec16 __attribute__((ext_vector_type(4)));   // (an array of uint4 is not kept in registers here)
template <bool SPLIT>
__global__ __launch_bounds__(256) void heads_kernel(Vec16* merged, Vec16* t0, Vec16* t1, Vec16* t2, int L, int H, int n,
                                                    int log_v /* vectors per 64 elements */, int pieces, unsigned waves) {
    const unsigned w = __builtin_amdgcn_readfirstlane(blockIdx.x * 4u + (threadIdx.x >> 6));
    if (w >= waves) return;
    const int lane = threadIdx.x & 63, v = 1 << log_v, c = lane & (v - 1), tokens = 64 >> log_v;
    const unsigned h = w % (unsigned)H, part = w / (unsigned)H % (unsigned)n, at = w / ((unsigned)H * (unsigned)n);
    const unsigned b = at / (unsigned)pieces;
    const int l = (int)(at % (unsigned)pieces) * 4 * tokens + (lane >> log_v);
    Vec16* const m = merged + (((size_t)b * L * n + part) * H + h) * v + c;
    Vec16* const t = (part == 0 ? t0 : part == 1 ? t1 : t2) + ((size_t)b * H + h) * L * v + c;
    const size_t m_row = (size_t)n * H * v;
    Vec16 x[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int row = min(l + k * tokens, L - 1);
        x[k] = SPLIT ? m[row * m_row] : t[(size_t)row * v];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int row = l + k * tokens;
        if (row < L) (SPLIT ? t[(size_t)row * v] : m[row * m_row]) = x[k];
    }
}

struct WeightGradPlan {
    int tiles_n, tiles_m, slices, slice_rows;
    WeightGradPlan(int rows, int N, int M) {
        tiles_n = (N + kTile - 1) / kTile;
        tiles_m = (M + kTile - 1) / kTile;
        const int most = (rows + kWeightGradMinRows - 1) / kWeightGradMinRows, want = kWeightGradGroups / (tiles_n * tiles_m);
        slices = want < 1 ? 1 : want > most ? most : want;
        slice_rows = ((rows + slices - 1) / slices + kStepRows - 1) / kStepRows * kStepRows;
        slices = (rows + slice_rows - 1) / slice_rows;
    }
};

}  // namespace

size_t weight_grad_workspace_bytes(int rows, int N, int M) {
    return (size_t)WeightGradPlan(rows, N, M).slices * N * M * sizeof(float);
}

hipError_t launch_weight_grad(const void* dY, const void* X, void* dW, int rows, int N, int M, void* workspace,
                              hipStream_t st) {
    const WeightGradPlan p(rows, N, M);
    float* const partial = static_cast<float*>(workspace);
    const unsigned groups = (unsigned)((p.slices + 7) / 8 * 8 * p.tiles_n * p.tiles_m);
    weight_grad_kernel<<<dim3(groups), dim3(256), 0, st>>>(static_cast<const bf16_t*>(dY), static_cast<const bf16_t*>(X),
                                                           partial, rows, N, M, p.slices, p.slice_rows, p.tiles_n, p.tiles_m);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int n4 = N * M / 4;
    weight_grad_sum_kernel<<<dim3((unsigned)((n4 + 63) / 64)), dim3(256), 0, st>>>(partial, p.slices, n4,
                                                                                    static_cast<bf16_t*>(dW));
    return hipGetLastError();
}

hipError_t launch_heads(bool split, void* merged, void* const* t, int B, int L, int H, int n, bool is_bf16, hipStream_t st) {
    const int log_v = is_bf16 ? 3 : 4, pieces = (L + (256 >> log_v) - 1) / (256 >> log_v);
    const unsigned waves = (unsigned)((size_t)B * pieces * n * H), groups = (waves + 3u) / 4u;
    Vec16 *m = static_cast<Vec16*>(merged), *a = static_cast<Vec16*>(t[0]), *b = static_cast<Vec16*>(t[n > 1 ? 1 : 0]),
          *c = static_cast<Vec16*>(t[n > 1 ? 2 : 0]);
    if (split)
        heads_kernel<true><<<dim3(groups), dim3(256), 0, st>>>(m, a, b, c, L, H, n, log_v, pieces, waves);
    else
        heads_kernel<false><<<dim3(groups), dim3(256), 0, st>>>(m, a, b, c, L, H, n, log_v, pieces, waves);
    return hipGetLastError();
}

}  // namespace spion
