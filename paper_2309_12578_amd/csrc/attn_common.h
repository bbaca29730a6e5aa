// Device helpers shared by the attention kernels: MFMA wrappers, fragment types, wave-level
// reductions and scans.
#ifndef SPION_ATTN_COMMON_H_
#define SPION_ATTN_COMMON_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace spion {

typedef __bf16 bf16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kD = 64;  // head dimension
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// What a row's exponentials are taken against before any score has been seen: finite, so that scores of -infinity alone (a
// masked block, or a whole piece of a row) add 0 and not exp2(inf - inf).
constexpr float kLowest = -3.4028234663852886e38f;

// How far (in log2 units) a score may lie above the value its row's exponentials are taken against before the
// running sums are rescaled.  P = exp2(s - m) above 1 is as exact as below (it keeps its relative
// error, the fp32 sums have range to spare), so what a row's maximum does inside this slack need not be
// known: the generic kernels look at a lane's own scores only, the tuned forward at the running sum, which no score can be out of
// bounds without passing; the reduction over the lanes of a row, the rescaling and the branch are left to the first block
// of a row and to scores that really run away.
// The sums hold up to 2^kRescaleSlack times what they would against the row's maximum: |V| above about 1e29 can
// overflow them.
constexpr float kRescaleSlack = 30.f;
constexpr float kSumLimit = 1073741824.f;   // 2^kRescaleSlack

// Per element type: a 16-byte lane fragment of EPL elements; four lane groups make a chunk of KC
// contraction elements along d.
template <typename T>
struct Elem;
template <>
struct Elem<float> {
    static constexpr int EPL = 4, KC = 16;
    typedef f32x4 Frag;   // d-chunk fragment
    typedef f32x4 Quad;   // 4 consecutive elements (one accumulator tile's worth per lane)
};
template <>
struct Elem<bf16_t> {
    static constexpr int EPL = 8, KC = 32;
    typedef bf16x8 Frag;
    typedef bf16x4 Quad;
};

// v * 2^x, x <= 0, for v far above 1 and x as far below 0: 2^x by itself would be 0 below x = -149.
__device__ __forceinline__ f32x4 scale_down(f32x4 v, float x) {
    const float k = fmaxf(floorf(x), -1024.f), f = exp2f(x - k);
    return f32x4{ldexpf(v[0] * f, (int)k), ldexpf(v[1] * f, (int)k), ldexpf(v[2] * f, (int)k), ldexpf(v[3] * f, (int)k)};
}

// 2^x of the exponent unit alone; a result below the smallest normal number comes out as 0
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// acc[16x16] += A(16 x KC) * B(KC x 16), both fragments indexed [lane % 16][chunk + (lane / 16) * EPL + e]
__device__ __forceinline__ f32x4 mma_d(f32x4 acc, bf16x8 a, bf16x8 b) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mma_d(f32x4 acc, f32x4 a, f32x4 b) {
#pragma unroll
    for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[i], acc, 0, 0, 0);
    return acc;
}
template <typename T>
__device__ __forceinline__ typename Elem<T>::Quad to_quad(f32x4 v);
template <>
__device__ __forceinline__ f32x4 to_quad<float>(f32x4 v) {
    return v;
}
template <>
__device__ __forceinline__ bf16x4 to_quad<bf16_t>(f32x4 v) {
    bf16x4 r;
    r[0] = (bf16_t)v[0];
    r[1] = (bf16_t)v[1];
    r[2] = (bf16_t)v[2];
    r[3] = (bf16_t)v[3];
    return r;
}
__device__ __forceinline__ bf16x8 join(bf16x4 lo, bf16x4 hi) {
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

// Reductions over the four lanes r, r + 16, r + 32, r + 48 that hold values of the same owned row.
// v_permlane16_swap / v_permlane32_swap exchange rows of 16 (halves of 32) lanes between two
// registers in the VALU: with both registers holding v, one comes back as {row 0, row 0, row 2,
// row 2} and the other as {row 1, row 1, row 3, row 3} (resp. low half twice / high half twice).
// No LDS round trip, unlike a shuffle.  The two results pass through an empty asm statement: given
// equal inputs the compiler otherwise treats them as equal and drops the combine.
__device__ __forceinline__ void swap_rows16(float v, float& a, float& b) {
    const unsigned u = __builtin_bit_cast(unsigned, v);
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    unsigned r0 = r[0], r1 = r[1];
    asm volatile("" : "+v"(r0), "+v"(r1));
    a = __builtin_bit_cast(float, r0);
    b = __builtin_bit_cast(float, r1);
}
__device__ __forceinline__ void swap_halves32(float v, float& a, float& b) {
    const unsigned u = __builtin_bit_cast(unsigned, v);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    unsigned r0 = r[0], r1 = r[1];
    asm volatile("" : "+v"(r0), "+v"(r1));
    a = __builtin_bit_cast(float, r0);
    b = __builtin_bit_cast(float, r1);
}
__device__ __forceinline__ float group_max(float v) {
    float a, b;
    swap_rows16(v, a, b);
    swap_halves32(fmaxf(a, b), a, b);
    return fmaxf(a, b);
}
__device__ __forceinline__ float group_sum(float v) {
    float a, b;
    swap_rows16(v, a, b);
    swap_halves32(a + b, a, b);
    return a + b;
}

template <typename T>
__device__ __forceinline__ void store_quad(T* dst, f32x4 v) {
    *reinterpret_cast<typename Elem<T>::Quad*>(dst) = to_quad<T>(v);
}

// Inclusive prefix sum over the wave with DPP moves (VALU speed, no LDS crossbar): shifts of 1, 2, 4, 8
// inside each row of 16 lanes, then lane 15 of rows 0 and 2 added to rows 1 and 3, then lane 31 added
// to rows 2 and 3.  A lane whose source is outside its row, or whose row is masked off, adds the 0
// given as old value.  All lanes must be active.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_fetch0(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROW_MASK, 0xf, false);
}
__device__ __forceinline__ int wave_incl_scan(int v, int /*lane*/) {
    v += dpp_fetch0<0x111, 0xf>(v);   // row_shr:1
    v += dpp_fetch0<0x112, 0xf>(v);   // row_shr:2
    v += dpp_fetch0<0x114, 0xf>(v);   // row_shr:4
    v += dpp_fetch0<0x118, 0xf>(v);   // row_shr:8
    v += dpp_fetch0<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
    v += dpp_fetch0<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
    return v;
}

// How many lanes below the calling one are set in `mask`.
__device__ __forceinline__ int lanes_below(unsigned long long mask) {
    return __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0));
}

}  // namespace spion
#endif
