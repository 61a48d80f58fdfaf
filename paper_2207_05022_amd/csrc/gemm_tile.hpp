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

constexpr int kComputeUnits = 256;
constexpr int kGroupRows = 8;              // row tiles per band of the tile order ...
constexpr int kRowMajorColumnTiles = 12;   // ... used beyond this many column tiles

// Workgroups are handed to the 8 XCDs round-robin by linear id; each XCD has one contiguous range of the tile order: row by row up to
// kRowMajorColumnTiles column tiles; beyond that (d_model 2048: 22 column tiles) row by row would stream every weight column
// through the L2 once per row tile, and the order walks bands of kGroupRows row tiles column by column instead, so that the
// workgroups that run together share weight columns too (measured at d_model 2048, 4096 tokens: 720 -> 617 us per layer; at 8 to 11
// column tiles the two orders measure the same within run-to-run noise).
__device__ inline void locate_tile(int tile, int n_tiles, int m_tiles, uint32_t band_recip, int &tile_m, int &tile_n)   // band_recip: band_reciprocal(n_tiles)
{
    const int group = n_tiles > kRowMajorColumnTiles ? kGroupRows : 1;
    const int band = quotient(tile, group * n_tiles, band_recip);
    const int band_rows = min(group, m_tiles - band * group);   // the last band may be short
    const int in_band = tile - band * (group * n_tiles);
    tile_n = in_band;
    if (band_rows == kGroupRows) tile_n = in_band / kGroupRows;
    else if (band_rows > 1) tile_n = in_band / band_rows;
    tile_m = band * group + (in_band - tile_n * band_rows);
}
inline uint32_t band_reciprocal(int n_tiles) { return reciprocal((n_tiles > kRowMajorColumnTiles ? kGroupRows : 1) * n_tiles); }

}  // namespace sti
