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

// Sum over groups of W lanes, in every one of them: DPP moves inside a row of 16 lanes, a few cycles each where a shuffle takes a
// trip through the LDS pipe.
template <int CTRL> __device__ __forceinline__ float dpp_move(float x)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}
template <int W> __device__ __forceinline__ float row_sum(float d)
{
    static_assert(W == 8 || W == 16 || W == 32, "lanes per row");
    d += dpp_move<0xB1>(d);                  // quad_perm: lane ^ 1
    d += dpp_move<0x4E>(d);                  // quad_perm: lane ^ 2
    d += dpp_move<0x141>(d);                 // row_half_mirror: the other four of eight
    if (W >= 16) d += dpp_move<0x140>(d);    // row_mirror: the other eight of sixteen
    if (W == 32) d += __shfl_xor(d, 16, WAVE);
    return d;
}
// Reductions over the four 16-lane rows of a wave (the lanes that share a column of a 16x16 accumulator tile),
// with the row-swap instructions of gfx950: v_permlane16_swap exchanges rows 1 and 3 of its first operand with
// rows 0 and 2 of its second, v_permlane32_swap the upper half of the first with the lower half of the second.
__device__ __forceinline__ float rows_max(float x)
{
    unsigned u = __float_as_uint(x);
    auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    u = __float_as_uint(fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1])));
    auto b = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float rows_sum(float x)
{
    unsigned u = __float_as_uint(x);
    auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    u = __float_as_uint(__uint_as_float(a[0]) + __uint_as_float(a[1]));
    auto b = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// Over all lanes, added in the order of a butterfly from lane ^ 32 down to lane ^ 1 (a norm's bits, and what follows from them in a
// 16-bit model, depend on it).  Six shuffles, each a trip through the LDS pipe, took longer: LayerNorm of bf16 2048 x 4096 10.2 us, now
// 9.5, 8192 x 1024 9.0 and 8.6.
__device__ __forceinline__ float wave_sum(float v)
{
    auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    v += dpp_move<0x128>(v);                 // row_ror:8: lane ^ 8
    v += dpp_move<0x124>(v);                 // row_ror:4: as lane ^ 4, since lanes eight apart hold the same by now
    v += dpp_move<0x4E>(v);                  // quad_perm: lane ^ 2
    v += dpp_move<0xB1>(v);                  // quad_perm: lane ^ 1
    return v;
}
__device__ __forceinline__ float wave_max(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, WAVE));
    return v;
}

// Largest value and its index, the lowest of equal ones; a NaN is never taken.
__device__ __forceinline__ void argmax_take(float& best, int& idx, float ov, int oi)
{
    if (ov > best || (ov == best && oi < idx)) { best = ov; idx = oi; }
}
template <int CTRL> __device__ __forceinline__ int dpp_move_int(int x) { return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xf, 0xf, true); }
// over 16 lanes, then over the wave, in every lane (moves as in row_sum and rows_sum).  With shuffles, and one thread going through
// the waves' candidates, 4 rows of 2048 in a decode iteration took 3.7 us, now 2.5.
__device__ __forceinline__ void argmax_row16(float& best, int& idx)
{
    argmax_take(best, idx, dpp_move<0xB1>(best), dpp_move_int<0xB1>(idx));
    argmax_take(best, idx, dpp_move<0x4E>(best), dpp_move_int<0x4E>(idx));
    argmax_take(best, idx, dpp_move<0x141>(best), dpp_move_int<0x141>(idx));
    argmax_take(best, idx, dpp_move<0x140>(best), dpp_move_int<0x140>(idx));
}
// over the four lanes l, l + 16, ..
__device__ __forceinline__ void argmax_column(float& best, int& idx)
{
    auto bv = __builtin_amdgcn_permlane16_swap(__float_as_uint(best), __float_as_uint(best), false, false);
    auto bi = __builtin_amdgcn_permlane16_swap((unsigned)idx, (unsigned)idx, false, false);
    best = __uint_as_float(bv[0]);
    idx = (int)bi[0];
    argmax_take(best, idx, __uint_as_float(bv[1]), (int)bi[1]);
    bv = __builtin_amdgcn_permlane32_swap(__float_as_uint(best), __float_as_uint(best), false, false);
    bi = __builtin_amdgcn_permlane32_swap((unsigned)idx, (unsigned)idx, false, false);
    best = __uint_as_float(bv[0]);
    idx = (int)bi[0];
    argmax_take(best, idx, __uint_as_float(bv[1]), (int)bi[1]);
}
__device__ __forceinline__ void argmax_rows(float& best, int& idx)
{
    argmax_row16(best, idx);
    argmax_column(best, idx);
}

// GELU, erf form: x * Phi(x), by Phi(-t) = 2^-(t * R(t)) / 2 for t = |x|: max(x, 0) - t / 2 * 2^-(t * R(t)), whose last step rounds once.
// R is of degree 11, a weighted least-squares fit on [0, 9] (weights iterated towards equal error; each coefficient rounded to
// float, the ones above it fitted again), its leading coefficient positive, so that Phi vanishes beyond.  With the coefficients as
// they stand, in 64 bits: relative error of Phi(-t) 1.9e-9 for t below 3, then growing (4e-9 to 4, 5e-8 to 5, 3e-5 to 7, 5e-2 to
// 9) while the absolute error falls (9e-10 below 1, 2e-11 to 3, 1e-13 to 5, 1e-14 to 7, 3e-17 to 9).
// What bounds it: the vector ALU of an epilogue, here 21 instructions (the power counted four times).  0.5 * x * (1 + erff(x / sqrt 2)),
// with both of erff's branches in waves of wide inputs, took longer: bf16 8192 x 4096, K 1024 76.2 us, now 69.8 (53.6 without an
// activation), 8192 x 49152, K 12288 6350 and 6243; of narrow ones one branch is met, float 12288 x 1024, K 256 at a deviation of
// 0.32 63.4 and 64.7.
// Error against 64 bits, 2-norm relative, and of 0.5 * x * (1 + erf) in float with an erf rounded once: x normal with deviation
// 0.1 3.1e-8 and 3.8e-8, 0.32 3.1e-8 and 4.0e-8, 1 2.7e-8 and 3.7e-8, 2.2 2.5e-8 and 3.4e-8; and no larger in any stretch of x.
__device__ __forceinline__ float gelu(float x)
{
    float t = fabsf(fminf(x, 3.4028235e+38f));               // finite for +inf, whose result is +inf; -inf gives NaN, as -inf * 0 does
    float r = 2.61296429e-10f;
    r = fmaf(r, t, -1.1455894e-08f);
    r = fmaf(r, t, 2.27268643e-07f);
    r = fmaf(r, t, -2.69496695e-06f);
    r = fmaf(r, t, 2.10983981e-05f);
    r = fmaf(r, t, -1.11249807e-04f);
    r = fmaf(r, t, 3.54487536e-04f);
    r = fmaf(r, t, -9.85201768e-05f);
    r = fmaf(r, t, -6.87161693e-03f);
    r = fmaf(r, t, 5.24111241e-02f);
    r = fmaf(r, t, 4.59225982e-01f);
    r = fmaf(r, t, 1.15110397f);
    float p = __builtin_amdgcn_exp2f(-(r * t));              // 2 Phi(-t)
    return fmaf(-0.5f * t, p, x < 0.f ? -0.f : x);
}

__device__ __forceinline__ float act_apply(float x, int act)
{
    if (act == 0) return x > 0.f ? x : 0.f;
    if (act == 1) return gelu(x);
    return x;
}

}  // namespace exe
