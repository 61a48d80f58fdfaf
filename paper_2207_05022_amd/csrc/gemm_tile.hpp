// What the kernels for many tokens (gemm_wide.hip, gemm_large.hip) share.
#pragma once
#include "sti_internal.hpp"

namespace sti {

// GELU with the Gaussian CDF (the erf form, not the tanh form):  z Phi(z) = max(z, 0) - a Phi(-a),  a = |z|.
// log2 Phi(-a) is close to a parabola: a polynomial of degree 4, the minimax fit of a 2^p(a) to a Phi(-a) (linear program in float64) with
// p(0) = -1.  |error| < 9e-6, relative below 1e-4 for z > -1 and 2e-3 for z > -3; beyond a = 5.5 (a Phi(-a) = 1e-7) the clamped argument.
// none (zero_of) is 0, or NaN where z or another of eight values of the same token is infinite or NaN.  max(z, none) is max(z, 0) or z, so that -inf
// and NaN come out as such, as in the polynomial of degree 8 before it; what the others of the eight come out as then does not matter, since FFN2
// adds all neurons of a token up.  Eight instructions, one of them transcendental, and five for eight values' `none`: the epilogue of FFN1 is bound by
// exactly these.  That polynomial in z^2 took 13 (errors 4.1e-5, 2.5e-4, 5e-3).  Clocks for 128 x 384 outputs: 11440 so, 10960 now, 10690 with
// max(z, 0), which makes -inf a 0, 11400 with a product -0 z for each value.
__device__ inline float gelu_wide(float z, float none)
{
    const float a = __builtin_fminf(__builtin_fabsf(z), 5.5f);
    float p = 4.161671270e-03f;
    p = fmaf(p, a, -4.573547095e-02f);
    p = fmaf(p, a, -4.649304450e-01f);
    p = fmaf(p, a, -1.149567008f);
    p = fmaf(p, a, -1.0f);
    return fmaf(-a, __builtin_amdgcn_exp2f(p), __builtin_fmaxf(z, none));
}
__device__ inline float zero_of(const float (&z)[8])
{
    float most = __builtin_fabsf(z[0]);
#pragma unroll
    for (int e = 1; e < 8; ++e) most = __builtin_elementwise_maximum(most, __builtin_fabsf(z[e]));
    return most * 0.f;
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
