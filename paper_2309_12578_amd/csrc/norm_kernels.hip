// LayerNorm of the sub-layer (Algorithm 5) and its gradients, for rows of D = 64 k <= 2048 elements, fp32 or bf16.
//
// Bound by HBM: x in, y out; backward x, dY and the gradient of a residual that leaves from x in, their sum out.  A wave takes whole rows and keeps a row in registers (4
// consecutive elements a lane, every 256), statistics and sums in fp32 as two passes over the registers.  In the
// backward a wave adds its rows' shares of the gradients of weight and bias up in registers, a workgroup writes one
// partial row of each, a second launch adds these in order (no atomics).
// 16384 rows of 256, bf16: 8.0 us forward, 13.2 + 3.9 us backward with a residual's gradient (11.0 without); torch's kernels took
// 22 and 29 + 16 + 5.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "attn_common.h"
#include "spion_internal.h"

namespace spion {

namespace {

constexpr int kNormMaxGroups = 512;   // workgroups of the backward: partial rows that the second launch adds

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}
__device__ __forceinline__ f32x4 load4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
__device__ __forceinline__ f32x4 load4(const bf16_t* p) {
    const bf16x4 v = *reinterpret_cast<const bf16x4*>(p);
    return f32x4{(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
}
__device__ __forceinline__ float sum4(f32x4 v) { return (v[0] + v[1]) + (v[2] + v[3]); }

template <typename T, int K>   // K = groups of 256 columns
__global__ __launch_bounds__(256) void layer_norm_kernel(const T* __restrict__ x, const T* __restrict__ w,
                                                         const T* __restrict__ b, T* __restrict__ y, float* __restrict__ mean,
                                                         float* __restrict__ rstd, int rows, int D, float eps) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const float inv = 1.f / (float)D;
    for (int row = blockIdx.x * 4 + wave; row < rows; row += gridDim.x * 4) {
        f32x4 v[K];
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int c = k * 256 + lane * 4;
            v[k] = c < D ? load4(x + (size_t)row * D + c) : f32x4{0.f, 0.f, 0.f, 0.f};
            s += sum4(v[k]);
        }
        const float mu = wave_sum(s) * inv;
        s = 0.f;
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (k * 256 + lane * 4 < D) {
                v[k] -= mu;
                s += sum4(v[k] * v[k]);
            }
        const float rs = 1.f / sqrtf(wave_sum(s) * inv + eps);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int c = k * 256 + lane * 4;
            if (c < D) store_quad<T>(y + (size_t)row * D + c, v[k] * rs * load4(w + c) + load4(b + c));
        }
        if (lane == 0) {
            mean[row] = mu;
            rstd[row] = rs;
        }
    }
}

// dr: what else arrives at x, or nullptr.  Added here, in fp32, it costs the read of dr; as an addition of its own behind
// the kernel a pass over three tensors and a launch (16384 rows of 256, bf16: 11.0 -> 13.1 us here, 5.8 us saved there).
template <typename T, int K>
__global__ __launch_bounds__(256) void layer_norm_grad_kernel(const T* __restrict__ dy, const T* __restrict__ dr,
                                                              const T* __restrict__ x, const T* __restrict__ w, 
                                                              const float* __restrict__ mean, const float* __restrict__ rstd,
                                                              T* __restrict__ dx,
                                                              float* __restrict__ partial, int rows, int D) {
    __shared__ f32x4 part[4][2][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const float inv = 1.f / (float)D;
    f32x4 dw[K], db[K], wv[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int c = k * 256 + lane * 4;
        dw[k] = db[k] = f32x4{0.f, 0.f, 0.f, 0.f};
        wv[k] = c < D ? load4(w + c) : f32x4{0.f, 0.f, 0.f, 0.f};
    }
    for (int row = blockIdx.x * 4 + wave; row < rows; row += gridDim.x * 4) {
        const float mu = mean[row], rs = rstd[row];
        f32x4 xh[K], g[K], r[K];
        float sg = 0.f, sgx = 0.f;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int c = k * 256 + lane * 4;
            xh[k] = g[k] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (c < D) {
                xh[k] = (load4(x + (size_t)row * D + c) - mu) * rs;
                g[k] = load4(dy + (size_t)row * D + c);
                if (dr) r[k] = load4(dr + (size_t)row * D + c);
            }
            dw[k] += g[k] * xh[k];
            db[k] += g[k];
            g[k] *= wv[k];
            sg += sum4(g[k]);
            sgx += sum4(g[k] * xh[k]);
        }
        sg = wave_sum(sg) * inv;
        sgx = wave_sum(sgx) * inv;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int c = k * 256 + lane * 4;
            if (c < D) {
                f32x4 v = (g[k] - sg - xh[k] * sgx) * rs;
                if (dr) v += r[k];
                store_quad<T>(dx + (size_t)row * D + c, v);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        __syncthreads();   // the group before has been read
        part[wave][0][lane] = dw[k];
        part[wave][1][lane] = db[k];
        __syncthreads();
        const int c = k * 256 + lane * 4;
        if (wave < 2 && c < D)
            *reinterpret_cast<f32x4*>(partial + ((size_t)blockIdx.x * 2 + wave) * D + c) =
                ((part[0][wave][lane] + part[1][wave][lane]) + part[2][wave][lane]) + part[3][wave][lane];
    }
}

// 64 of the 2 D columns a workgroup (weight's, then bias'), a wave every 16th partial row.
template <typename T>
__global__ __launch_bounds__(1024) void layer_norm_sum_kernel(const float* __restrict__ partial, int groups, int D,
                                                              T* __restrict__ dw, T* __restrict__ db) {
    __shared__ float part[16][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = blockIdx.x * 64 + lane;
    float s = 0.f;
#pragma unroll 8
    for (int g = wave; g < groups; g += 16) s += partial[(size_t)g * 2 * D + col];
    part[wave][lane] = s;
    __syncthreads();
    if (wave != 0) return;
#pragma unroll
    for (int k = 1; k < 16; ++k) s += part[k][lane];
    (col < D ? dw + col : db + (col - D))[0] = (T)s;
}

int norm_grad_groups(int rows) {
    const int groups = (rows + 15) / 16;   // 4 rows a wave
    return groups < kNormMaxGroups ? groups : kNormMaxGroups;
}

template <typename T, int K>
hipError_t forward_k(const void* x, const void* w, const void* b, void* y, float* mean, float* rstd, int rows, int D,
                     float eps, hipStream_t st) {
    const unsigned groups = (unsigned)((rows + 3) / 4);
    layer_norm_kernel<T, K><<<dim3(groups < 16384u ? groups : 16384u), dim3(256), 0, st>>>(
        static_cast<const T*>(x), static_cast<const T*>(w), static_cast<const T*>(b), static_cast<T*>(y), mean, rstd, rows, D, eps);
    return hipGetLastError();
}
template <typename T, int K>
hipError_t backward_k(const void* dy, const void* dr, const void* x, const void* w, const float* mean, const float* rstd, void* dx, void* dw,
                      void* db, float* partial, int rows, int D, hipStream_t st) {
    const int groups = norm_grad_groups(rows);
    layer_norm_grad_kernel<T, K><<<dim3((unsigned)groups), dim3(256), 0, st>>>(
        static_cast<const T*>(dy), static_cast<const T*>(dr), static_cast<const T*>(x), static_cast<const T*>(w), mean, rstd,
        static_cast<T*>(dx), partial, rows, D);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    layer_norm_sum_kernel<T><<<dim3((unsigned)(2 * D / 64)), dim3(1024), 0, st>>>(partial, groups, D, static_cast<T*>(dw),
                                                                                   static_cast<T*>(db));
    return hipGetLastError();
}

}  // namespace

size_t layer_norm_workspace_bytes(int rows, int D) { return (size_t)norm_grad_groups(rows) * 2 * D * sizeof(float); }

#define SPION_NORM_DISPATCH(FN, ...)                                                             \
    do {                                                                                         \
        if (is_bf16) {                                                                           \
            if (D <= 256) return FN<bf16_t, 1>(__VA_ARGS__);                                     \
            if (D <= 512) return FN<bf16_t, 2>(__VA_ARGS__);                                     \
            return D <= 1024 ? FN<bf16_t, 4>(__VA_ARGS__) : FN<bf16_t, 8>(__VA_ARGS__);          \
        }                                                                                        \
        if (D <= 256) return FN<float, 1>(__VA_ARGS__);                                          \
        if (D <= 512) return FN<float, 2>(__VA_ARGS__);                                          \
        return D <= 1024 ? FN<float, 4>(__VA_ARGS__) : FN<float, 8>(__VA_ARGS__);                \
    } while (0)

hipError_t launch_layer_norm(const void* x, const void* w, const void* b, void* y, float* mean, float* rstd, int rows,
                             int D, float eps, bool is_bf16, hipStream_t st) {
    SPION_NORM_DISPATCH(forward_k, x, w, b, y, mean, rstd, rows, D, eps, st);
}
hipError_t launch_layer_norm_grad(const void* dy, const void* dr, const void* x, const void* w, const float* mean,
                                  const float* rstd, void* dx, void* dw, void* db, float* partial, int rows, int D, bool is_bf16, hipStream_t st) {
    SPION_NORM_DISPATCH(backward_k, dy, dr, x, w, mean, rstd, dx, dw, db, partial, rows, D, st);
}

}  // namespace spion
