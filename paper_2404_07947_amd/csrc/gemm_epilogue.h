// What the GEMM kernels share: the MFMA step over 64 bytes of K, and the epilogue (alpha, bias, activation, and the store
// in one of the three output modes).
#pragma once
#include "common.h"

namespace exe {

typedef __attribute__((ext_vector_type(4))) unsigned u32x4;

template <typename T> struct Vec4;                     // four consecutive elements in one access
template <> struct Vec4<float> { typedef f32x4 type; };
template <> struct Vec4<bf16_t> { typedef bf16x4 type; };

// 64 bytes of K of 16 weight rows times 16 activation rows: lane l holds 16 bytes of row l % 16, the k-values of lane group
// l / 16.  Which k a lane group holds does not matter as long as both operands agree.  The weights are the MFMA's A
// operand: the accumulator of lane l is output features 4 * (l / 16) .. +3 of row l % 16.
template <typename T> struct HalfUnit;
template <> struct HalfUnit<bf16_t> {
    static __device__ __forceinline__ f32x4 mma(u32x4 w, u32x4 a, f32x4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, a), c, 0, 0, 0);
    }
};
template <> struct HalfUnit<float> {
    static __device__ __forceinline__ f32x4 mma(u32x4 w, u32x4 a, f32x4 c)
    {
        f32x4 wf = __builtin_bit_cast(f32x4, w), af = __builtin_bit_cast(f32x4, a);
#pragma unroll
        for (int i = 0; i < 4; ++i) c = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[i], af[i], c, 0, 0, 0);
        return c;
    }
};

// Floats as the sum of three bf16 parts, all of their bits: x rounded, what is left rounded, and the rest; bf16 pairs in dwords.  The
// products of two such floats that count (see kernels_gemm_f32.hip) are PARTS of the one and the other, smallest first.
//
// What is parted is x * PART_SCALE: the lowest bit of a float is 2^-149 or more, of that 2^-125, a normal bf16, so no float is too
// small for its parts (without the factor elements below 2^-109 lost bits: operands of 2^-115 gave products with errors of 1e-6,
// of 2^-122 1e-4, where ordinary ones err 1e-7).  Sums of products carry the factor twice; where they, or a part of an element of
// 2^104 and more, are too large for a float, they come out infinite or NaN, and who takes them looks for that.
constexpr int PARTS[6][2] = {{2, 0}, {0, 2}, {1, 1}, {1, 0}, {0, 1}, {0, 0}};
constexpr float PART_SCALE = 0x1p24f, PARTS_UNSCALE = 0x1p-48f;
__device__ __forceinline__ unsigned bf16_pair(float a, float b)
{
    unsigned r;
    asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ void bf16_parts(f32x4 v, uint2 (&w)[3])
{
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        w[p] = uint2{bf16_pair(v[0], v[1]), bf16_pair(v[2], v[3])};
        if (p < 2) v -= f32x4{bf16lo(w[p].x), bf16hi(w[p].x), bf16lo(w[p].y), bf16hi(w[p].y)};
    }
}

// Stores 4 consecutive output features n..n+3 of row m.  v = raw accumulators.
template <typename T>
__device__ __forceinline__ void epilogue_store4(f32x4 v, int m, int n, int N, const T* __restrict__ bias, int act,
                                                float alpha, int out_mode, void* __restrict__ out)
{
    f32x4 r;
#pragma unroll
    for (int j = 0; j < 4; ++j) r[j] = v[j] * alpha + (bias ? to_f32(bias[n + j]) : 0.f);
    int64_t o = (int64_t)m * N + n;
    if (out_mode == OUT_T) {
        T* p = (T*)out + o;
        if constexpr (sizeof(T) == 2) {
            bf16x4 w;
#pragma unroll
            for (int j = 0; j < 4; ++j) w[j] = (bf16_t)act_apply(r[j], act);
            *(bf16x4*)p = w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) r[j] = act_apply(r[j], act);
            *(f32x4*)p = r;
        }
    } else if (out_mode == OUT_RESID) {
        f32x4* p = (f32x4*)((float*)out + o);
        f32x4 h = *p;
        *p = h + r;
    } else {
        *(f32x4*)((float*)out + o) = r;
    }
}

}  // namespace exe
