// Producers of the pattern input (both HBM-bound streaming reductions):
//   score_mean_kernel   the attention-score maps of a layer's heads (and batch items) are averaged
//                       into one L x L map before pattern generation (Section 3, "Motivation")
//   frobenius kernels   Eq. 2: distance_i = | ||A^s_{i-1}||_F - ||A^s_i||_F |, the test that ends the
//                       dense-attention phase (Section 4.1)
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "spion_internal.h"

namespace spion {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
template <typename T> struct MapVec { typedef f32x4_t type; };
template <> struct MapVec<__bf16> { typedef bf16x8_t type; };

// out[i] = (sum over maps m = 0 .. n_maps-1, in that order, of A[m][i]) / n_maps, fp32 arithmetic.
// Bound by HBM reads.  A thread owns U vectors of 16 bytes, 256 vectors apart; its loads of 8 maps are in flight
// together, also of the last, incomplete 8.  The maps are read once and past the caches' keeping: as ordinary
// loads, one vector a thread, 16 bf16 maps of 4096^2 took 117 us (5.2 TB/s), non-temporal 105, two vectors 99
// (6.1 TB/s); 16 maps or 4 vectors in flight, or a grid of 1024 or 2048 workgroups, measure the same or slower.
template <typename T, int U>
__global__ __launch_bounds__(256) void score_mean_kernel(const T* __restrict__ A, int n_maps, size_t n,
                                                         float* __restrict__ out) {
    typedef typename MapVec<T>::type Vec;
    constexpr int V = 16 / sizeof(T);   // elements per vector
    const size_t nvec = n / V;
    const float inv = 1.0f / (float)n_maps;
    for (size_t v0 = (size_t)blockIdx.x * (256 * U) + threadIdx.x; v0 < nvec; v0 += (size_t)gridDim.x * (256 * U)) {
        float acc[U][V];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < V; ++e) acc[u][e] = 0.f;
        const T* p[U];
#pragma unroll
        for (int u = 0; u < U; ++u) p[u] = A + (v0 + u * 256 < nvec ? v0 + u * 256 : nvec - 1) * V;
        auto add8 = [&](int m, int maps) {   // maps m .. m + maps - 1, uniform; a literal 8 leaves no branches
            Vec x[8][U];
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (j < maps) {
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        x[j][u] = __builtin_nontemporal_load(reinterpret_cast<const Vec*>(p[u] + (size_t)(m + j) * n));
                }
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (j < maps) {
#pragma unroll
                    for (int u = 0; u < U; ++u)
#pragma unroll
                        for (int e = 0; e < V; ++e) acc[u][e] += (float)x[j][u][e];
                }
        };
        int m = 0;
        for (; m + 8 <= n_maps; m += 8) add8(m, 8);
        if (m < n_maps) add8(m, n_maps - m);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (v0 + u * 256 < nvec) {
#pragma unroll
                for (int e = 0; e < V; e += 4)
                    *reinterpret_cast<float4*>(out + (v0 + u * 256) * V + e) =
                        make_float4(acc[u][e] * inv, acc[u][e + 1] * inv, acc[u][e + 2] * inv, acc[u][e + 3] * inv);
            }
    }
}

constexpr int kFrobBlocks = 1024, kFrobThreads = 256;

__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// partial[b] = {sum of squares of a, sum of squares of b} over the float4s block b owns (fp64).  Bound by HBM reads.
// 4 workgroups a compute unit keep them going as well as 16, and the one workgroup that adds up the
// partials then has a quarter of them: with 4096, and ordinary loads, the call took 31.8 us for two maps of
// 4096^2 and 12.0 for two of 512^2, now 25.3 (5.3 TB/s) and 6.1.
__global__ __launch_bounds__(kFrobThreads) void frobenius_partial_kernel(const float* __restrict__ a,
                                                                        const float* __restrict__ b, size_t n,
                                                                        double2* __restrict__ partial) {
    const size_t nvec = n / 4;
    const size_t stride = (size_t)kFrobBlocks * kFrobThreads;
    double sa = 0.0, sb = 0.0;
    auto sq = [](double acc, const f32x4_t x) {
        return acc + ((double)x.x * x.x + (double)x.y * x.y) + ((double)x.z * x.z + (double)x.w * x.w);
    };
    size_t v = (size_t)blockIdx.x * kFrobThreads + threadIdx.x;
    // four float4 of each array in flight per thread
    for (; v + 3 * stride < nvec; v += 4 * stride) {
        f32x4_t x[4], y[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            x[u] = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(a) + v + u * stride);
            y[u] = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(b) + v + u * stride);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            sa = sq(sa, x[u]);
            sb = sq(sb, y[u]);
        }
    }
    for (; v < nvec; v += stride) {
        sa = sq(sa, reinterpret_cast<const f32x4_t*>(a)[v]);
        sb = sq(sb, reinterpret_cast<const f32x4_t*>(b)[v]);
    }
    if (blockIdx.x == 0 && threadIdx.x == 0)   // tail: n not a multiple of 4
        for (size_t i = nvec * 4; i < n; ++i) {
            sa += (double)a[i] * a[i];
            sb += (double)b[i] * b[i];
        }
    __shared__ double2 wsum[kFrobThreads / 64];
    sa = wave_sum_f64(sa);
    sb = wave_sum_f64(sb);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = make_double2(sa, sb);
    __syncthreads();
    if (threadIdx.x == 0) {
        double ta = 0.0, tb = 0.0;
        for (int w = 0; w < kFrobThreads / 64; ++w) {
            ta += wsum[w].x;
            tb += wsum[w].y;
        }
        partial[blockIdx.x] = make_double2(ta, tb);
    }
}

// out[0] = | sqrt(sum a^2) - sqrt(sum b^2) |, out[1] = ||a||_F, out[2] = ||b||_F; fixed summation order
__global__ __launch_bounds__(kFrobThreads) void frobenius_final_kernel(const double2* __restrict__ partial,
                                                                      double* __restrict__ out) {
    double sa = 0.0, sb = 0.0;
    for (int i = threadIdx.x; i < kFrobBlocks; i += kFrobThreads) {
        sa += partial[i].x;
        sb += partial[i].y;
    }
    __shared__ double2 wsum[kFrobThreads / 64];
    sa = wave_sum_f64(sa);
    sb = wave_sum_f64(sb);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = make_double2(sa, sb);
    __syncthreads();
    if (threadIdx.x == 0) {
        double ta = 0.0, tb = 0.0;
        for (int w = 0; w < kFrobThreads / 64; ++w) {
            ta += wsum[w].x;
            tb += wsum[w].y;
        }
        const double na = sqrt(ta), nb = sqrt(tb);
        out[0] = fabs(na - nb);
        out[1] = na;
        out[2] = nb;
    }
}

template <typename T>
static hipError_t mean_t(const T* A, int n_maps, size_t n, float* out, hipStream_t st) {
    const size_t nvec = n * sizeof(T) / 16;
    // two vectors a thread where that still gives every compute unit its eight workgroups
    if (nvec >= 2048 * 512) {
        const size_t blocks = (nvec + 511) / 512, most = (size_t)1 << 22;
        score_mean_kernel<T, 2><<<dim3((unsigned)(blocks < most ? blocks : most)), dim3(256), 0, st>>>(A, n_maps, n, out);
    } else {
        score_mean_kernel<T, 1><<<dim3((unsigned)((nvec + 255) / 256)), dim3(256), 0, st>>>(A, n_maps, n, out);
    }
    return hipGetLastError();
}

hipError_t launch_score_mean(const void* A, int is_bf16, int n_maps, size_t n, float* out, hipStream_t st) {
    return is_bf16 ? mean_t(static_cast<const __bf16*>(A), n_maps, n, out, st)
                   : mean_t(static_cast<const float*>(A), n_maps, n, out, st);
}

size_t frobenius_workspace_bytes() { return (size_t)kFrobBlocks * sizeof(double2); }

hipError_t launch_frobenius_distance(const float* a, const float* b, size_t n, double* out, void* workspace,
                                     hipStream_t st) {
    double2* partial = static_cast<double2*>(workspace);
    frobenius_partial_kernel<<<dim3(kFrobBlocks), dim3(kFrobThreads), 0, st>>>(a, b, n, partial);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    frobenius_final_kernel<<<dim3(1), dim3(kFrobThreads), 0, st>>>(partial, out);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Traffic yardstick: moves n_tiles x 16 KB from src to dst with the access shapes of the attention
// kernels (16 bytes per lane from HBM straight into LDS through the memory pipeline, one wave
// instruction per 1 KB; 16 bytes per lane row stores out).  It reads and writes every byte exactly
// once, so what the hardware traffic counters report for it gives their scale.
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void copy_yardstick_kernel(const char* __restrict__ src, char* __restrict__ dst) {
    typedef __attribute__((address_space(3))) void* lds_ptr;
    __shared__ __attribute__((aligned(16))) char tile[16384];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const size_t base = (size_t)blockIdx.x * 16384;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int piece = wave * 4 + k;   // 1 KB pieces
        __builtin_amdgcn_global_load_lds(src + base + piece * 1024 + lane * 16, (lds_ptr)(tile + piece * 1024), 16, 0,
                                         0);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): this wave's pieces have landed (it reads only those)
    asm volatile("" ::: "memory");
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int off = (wave * 4 + k) * 1024 + lane * 16;
        *reinterpret_cast<float4*>(dst + base + off) = *reinterpret_cast<const float4*>(tile + off);
    }
}

hipError_t launch_copy_yardstick(const void* src, void* dst, size_t n_tiles, hipStream_t st) {
    copy_yardstick_kernel<<<dim3((unsigned)n_tiles), dim3(256), 0, st>>>(static_cast<const char*>(src),
                                                                        static_cast<char*>(dst));
    return hipGetLastError();
}

}  // namespace spion
