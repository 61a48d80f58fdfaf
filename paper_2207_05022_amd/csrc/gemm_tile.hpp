// What the kernels for many tokens (gemm_wide.hip, gemm_large.hip) share.
#pragma once
#include "sti_internal.hpp"

namespace sti {

// GELU with the Gaussian CDF (the erf form, not the tanh form):  z Phi(z) = max(z, 0) - a Phi(-a),  a = |z|.
// log2 Phi(-a) is close to a parabola: a polynomial of degree 4, the minimax fit of a 2^p(a) to a Phi(-a) (linear program in float64) with
// p(0) = -1.  |error| < 9e-6, relative below 1e-4 for z > -1 and 2e-3 for z > -3; beyond a = 5.5 (a Phi(-a) = 1e-7) the clamped argument.
// -0 z is a zero that is none where z is infinite or NaN: max(z, -0 z) is max(z, 0), but -inf gives -inf, as in the polynomial of degree 8
// before it, and NaN gives NaN.  Nine instructions, one of them transcendental: the epilogue of FFN1 is bound by exactly these.  That
// polynomial in z^2 took 13 (errors 4.1e-5, 2.5e-4, 5e-3): 11440 -> 10690 clocks for 128 x 384 outputs with
// max(z, 0), which loses -inf: 24 x 384 tokens of d_model 1024, 24 layers 7000 us so, 7030 with the product.
__device__ inline float gelu_wide(float z)
{
    const float a = __builtin_fminf(__builtin_fabsf(z), 5.5f);
    float p = 4.161671270e-03f;
    p = fmaf(p, a, -4.573547095e-02f);
    p = fmaf(p, a, -4.649304450e-01f);
    p = fmaf(p, a, -1.149567008f);
    p = fmaf(p, a, -1.0f);
    return fmaf(-a, __builtin_amdgcn_exp2f(p), __builtin_fmaxf(z, z * -0.f));
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
