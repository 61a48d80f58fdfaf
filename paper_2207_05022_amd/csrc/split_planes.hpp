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

// z * Phi(z) with Phi(-|z|) = exp(log(erfcx(a)) - a^2) / 2, a = |z| / sqrt(2) (erfcx: the scaled complementary error function), and
// log2(erfcx(a)) = u P(u), u = a / (a + 5): P, of degree 8, is a minimax fit in float64 over a <= 5 (error 1.3e-8; beyond, the sum is
// governed by a^2).  The exponent goes to zero with z, so that no rounding of a larger term is left in Phi near one half.  22
// instructions and no branch; the erf of the mathematics library takes both of its branches in nearly every wave (FFN1 of 8 x 128
// tokens: 10 us of 37).  Error of the GELU (2-norm, relative; in brackets that of z / 2 (1 + erf)): arguments with a standard deviation of
// 0.05 3.2e-8 (3.7e-8), 0.3 3.3e-8 (4.1e-8), 1 2.7e-8 (3.9e-8), 3 2.2e-8 (3.0e-8); the largest relative to the value 2.1e-7 (2.7e-7) above -1.
// A form with exponent P(1 / (1 + a / 2)) - a^2 in front of that factor had 9.5e-8, 6.7e-8, 3.8e-8 and 2.6e-8 for 0.2 % less time of 12
// BERT-base layers at 8 x 128 tokens.
__device__ inline float gelu_f32(float z)
{
    const float r = fabsf(z), m = __builtin_amdgcn_fmed3f(z, -3e38f, 3e38f);   // (cut, so that no infinity meets a zero)
    const float u = fabsf(m) * __builtin_amdgcn_rcpf(r + 7.07106781f);
    float p = -12.034221f;
    p = fmaf(p, u, 32.526283f);
    p = fmaf(p, u, -38.2196f);
    p = fmaf(p, u, 18.953194f);
    p = fmaf(p, u, 1.5620527f);
    p = fmaf(p, u, -7.010886f);
    p = fmaf(p, u, -0.47139093f);
    p = fmaf(p, u, 4.9669704f);
    p = fmaf(p, u, -8.139539f);
    const float tail = 0.5f * __builtin_amdgcn_exp2f(fmaf(-0.72134752044448170368f * r, r, u * p));
    return z < 0.0f ? z * tail : fmaf(-fabsf(m), tail, z);
}

}  // namespace sti
