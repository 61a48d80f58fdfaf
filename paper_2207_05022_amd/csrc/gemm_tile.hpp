// What the kernels for many tokens (gemm_wide.hip, gemm_large.hip) share.
#pragma once
#include "sti_internal.hpp"

namespace sti {

// GELU with the Gaussian CDF (the erf form, not the tanh form):  z * Phi(z),
// Phi(z) = 1/2 + z * R(z^2).  R is a degree-8 polynomial in u = 2 z^2 / 4.5^2 - 1, fitted in
// float64 (weighted least squares on Chebyshev nodes) to (Phi(z) - 1/2) / z on |z| <= 4.5;
// beyond that Phi is taken at the clamped argument (1 - Phi(4.5) = 3.4e-6).  Evaluated in
// float32 the absolute error of the result is below 5e-5 for all z (0.1 of a binary16 ulp at
// 0.35, the value at z = 0.6 where the error peaks) and its relative error below 1e-4 for
// z > -1; 13 arithmetic instructions per value and no transcendental ones, which matters
// because the epilogue of the FFN1 projection is bound by exactly these instructions.
__device__ inline float gelu_polynomial(float z)
{
    const float zc = __builtin_amdgcn_fmed3f(z, -4.5f, 4.5f);
    const float u = fmaf(zc * zc, 2.0f / 20.25f, -1.0f);
    float r = 3.174704981e-03f;
    r = fmaf(r, u, -9.158361878e-03f);
    r = fmaf(r, u, 1.244540513e-02f);
    r = fmaf(r, u, -1.696567595e-02f);
    r = fmaf(r, u, 2.754268719e-02f);
    r = fmaf(r, u, -4.047719455e-02f);
    r = fmaf(r, u, 5.482644199e-02f);
    r = fmaf(r, u, -7.717846451e-02f);
    r = fmaf(r, u, 1.569020774e-01f);
    return z * fmaf(zc, r, 0.5f);
}

struct ShardIds {   // original shard id of every weight block (selects the bias slice), four to a scalar-loadable dword
    uint32_t id4[kMaxShardsPerLayer / 4];
    __device__ inline int id(int block) const { return (id4[block >> 2] >> (8 * (block & 3))) & 0xFF; }
};
inline ShardIds shard_ids(const GemmBlocks &blocks)
{
    ShardIds ids;   // (the kernels take these instead of the block table: a shorter argument list is a cheaper launch)
    for (int b = 0; b < kMaxShardsPerLayer; b += 4)
        ids.id4[b / 4] = (uint32_t)blocks.b[b].shard | (uint32_t)blocks.b[b + 1].shard << 8 |
                         (uint32_t)blocks.b[b + 2].shard << 16 | (uint32_t)blocks.b[b + 3].shard << 24;
    return ids;
}

}  // namespace sti
