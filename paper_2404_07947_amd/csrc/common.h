// Shared device/host helpers for the gfx950 kernels (wave64, CDNA4).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace exe {

typedef __bf16 bf16_t;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr int WAVE = 64;

enum Dtype { DT_F32 = 0, DT_BF16 = 1 };
enum OutMode { OUT_T = 0, OUT_RESID = 1, OUT_F32 = 2 };

__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(bf16_t x) { return (float)x; }
template <typename T> __device__ __forceinline__ T from_f32(float x);
template <> __device__ __forceinline__ float from_f32<float>(float x) { return x; }
template <> __device__ __forceinline__ bf16_t from_f32<bf16_t>(float x) { return (bf16_t)x; }  // round to nearest even

// bf16 pair packed in a dword -> two floats (exact)
__device__ __forceinline__ float bf16lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf16hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }

__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, WAVE);
    return v;
}
__device__ __forceinline__ float wave_max(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, WAVE));
    return v;
}

// GELU, erf form: x * Phi(x), with Phi(-t) = 2^-(1 + t * R(t)) for t >= 0.  R is a polynomial of degree 11, fitted to
// (-log2(Phi(-t)) - 1) / t on [0, 9] by weighted least squares (weights iterated towards equal error, relative error of Phi
// within 4e-8 for t < 2.5 and falling with Phi beyond); its leading coefficient is positive, so Phi vanishes beyond.
// What bounds it: the vector ALU of an epilogue.  0.5 * x * (1 + erff(x / sqrt 2)) took about 50 instructions, both of erff's
// branches in most waves, this takes 20: bf16 8192 x 4096, K 1024 83.4 -> 72.9 us (60.6 without an activation), 8192 x 49152, K 12288
// 6528 -> 6394, float 12288 x 1024, K 256 66.8 -> 63.3.
// Error against 64 bits over normally distributed x 3.4e-8 of the result (2-norm; the erff form, with an erf rounded once, 3.8e-8),
// and for negative x, where 1 + erf cancels, smaller throughout (x in [-3, -2]: 7e-7 relative, there 1e-5).
__device__ __forceinline__ float gelu(float x)
{
    float t = fabsf(x);
    float r = 1.1646179e-10f;
    r = fmaf(r, t, -6.0699383e-09f);
    r = fmaf(r, t, 1.4037859e-07f);
    r = fmaf(r, t, -1.8968133e-06f);
    r = fmaf(r, t, 1.6492046e-05f);
    r = fmaf(r, t, -9.3861607e-05f);
    r = fmaf(r, t, 3.1115115e-04f);
    r = fmaf(r, t, -2.8213937e-05f);
    r = fmaf(r, t, -6.9429772e-03f);
    r = fmaf(r, t, 5.2453075e-02f);
    r = fmaf(r, t, 4.5921367e-01f);
    r = fmaf(r, t, 1.1511053e+00f);
    float e = __builtin_amdgcn_exp2f(-fmaf(r, t, 1.f));      // Phi(-t)
    return x * (x < 0.f ? e : 1.f - e);
}

__device__ __forceinline__ float act_apply(float x, int act)
{
    if (act == 0) return x > 0.f ? x : 0.f;
    if (act == 1) return gelu(x);
    return x;
}

}  // namespace exe
