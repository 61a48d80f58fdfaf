// A float32 value as the sum of three bfloat16 values, the cells in which matrices of them lie (gemm_f32_split.hip), and the GELU of the
// float32 path.
#pragma once
#include "sti_internal.hpp"

namespace sti {

typedef float plane_f32x2 __attribute__((ext_vector_type(2)));
typedef float plane_f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t plane_u32x2 __attribute__((ext_vector_type(2)));

// Two values to planes h, m, l, each a dword of two bfloat16 (rounded to nearest even; one conversion instruction per pair).  Values that
// would round to infinity are cut to the largest bfloat16, so that h - infinity is never formed: an infinity then sits in l alone
// and meets only the other operand's h, a NaN likewise.
__device__ inline void split_pair(float a, float b, uint32_t (&plane)[3])
{
    constexpr float kLargest = 3.38953139e38f;
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    auto round2 = [](float x, float y) { return __builtin_bit_cast(uint32_t, __builtin_convertvector((plane_f32x2{x, y}), bf16x2)); };
    auto low = [](uint32_t u) { return __builtin_bit_cast(float, u << 16); };
    auto high = [](uint32_t u) { return __builtin_bit_cast(float, u & 0xFFFF0000u); };
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        plane[p] = round2(__builtin_amdgcn_fmed3f(a, -kLargest, kLargest), __builtin_amdgcn_fmed3f(b, -kLargest, kLargest));
        a -= low(plane[p]);
        b -= high(plane[p]);
    }
    plane[2] = round2(a, b);
}

// columns col .. col + 3 (a multiple of 4) of a row into a matrix of `cells` 64-column cells per row block
__device__ inline void store_planes4(uint16_t *planes, int row, int col, int cells, const plane_f32x4 x)
{
    uint16_t *cell = planes + ((int64_t)(row >> 5) * cells + (col >> 6)) * 6144 + ((col & 31) >> 3) * 512 + (((col >> 5) & 1) * 32 + (row & 31)) * 8 + (col & 7);
    uint32_t lo[3], hi[3];
    split_pair(x[0], x[1], lo);
    split_pair(x[2], x[3], hi);
#pragma unroll
    for (int k = 0; k < 3; ++k) *(plane_u32x2 *)(cell + k * 2048) = plane_u32x2{lo[k], hi[k]};
}

// z * Phi(z) with Phi(-|z|) = erfc(a) / 2, a = |z| / sqrt(2), and erfc(a) = t exp(-a^2 + P(t)), t = 1 / (1 + a / 2): P, of degree
// 9, is a minimax fit (float64, error 4.5e-8) of log(exp(a^2) erfc(a) / t); its coefficients carry the factor log2(e) of exp2.  19
// instructions and no branch; the erf of the mathematics library takes both of its branches in nearly every wave (FFN1 of 8 x 128
// tokens: 10 us of 37).  Error of the GELU of normal arguments (2-norm, relative): 3.3e-8, against 3.6e-8 of z / 2 (1 + erf(a)).
__device__ inline float gelu_f32(float z)
{
    const float a = fabsf(z) * 0.70710678118654752440f;
    const float t = __builtin_amdgcn_rcpf(fmaf(0.5f, a, 1.0f));
    float p = 2.051324397e-01f;
    p = fmaf(p, t, -9.608712196e-01f);
    p = fmaf(p, t, 1.619159222e+00f);
    p = fmaf(p, t, -9.393962026e-01f);
    p = fmaf(p, t, -1.686127335e-01f);
    p = fmaf(p, t, 2.919966169e-02f);
    p = fmaf(p, t, 4.089012742e-02f);
    p = fmaf(p, t, 5.596251488e-01f);
    p = fmaf(p, t, 1.440519691e+00f);
    p = fmaf(p, t, -1.825646043e+00f);
    const float tail = 0.5f * t * __builtin_amdgcn_exp2f(fmaf(-1.44269504088896340736f * a, a, p));
    return z * (z < 0.0f ? tail : 1.0f - tail);
}

}  // namespace sti
