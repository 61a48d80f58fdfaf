// Decompression of a float32 layer's shards into planes of three bfloat16 values (gemm_f32_split.hip): in a launch of its own there, and
// beside a LayerNorm (rowops.hip).
#pragma once
#include <type_traits>
#include "sti_internal.hpp"
#include "weight_loader.hpp"
#include "split_planes.hpp"

namespace sti {

// What a launch decodes: Q, K, V and O of every shard, or (skip: the cells of those) FFN1 and FFN2.
struct SplitDecodeJob {
    uint16_t *out;
    int32_t cells, skip, n_shards;
    CellMap map;
};
// d, dh and f multiples of 64; false: more cells than a grid has room for
inline bool split_decode_job(int n_shards, int d, int dh, int f, bool ffn, void *out, SplitDecodeJob *job)
{
    const int64_t attention_cells = (int64_t)d * 4 * dh / 2048, per_shard = ffn ? (int64_t)d * 2 * f / 2048 : attention_cells;
    const int64_t cells = per_shard * n_shards;
    if (d % 64 || dh % 64 || f % 64 || cells > 0x7FFFFFF0) return false;
    *job = SplitDecodeJob{(uint16_t *)out, (int32_t)cells, ffn ? (int32_t)attention_cells : 0, n_shards, cell_map(d, dh, f)};
    job->map.per_shard = (int)per_shard;
    job->map.recip_shard = reciprocal((uint32_t)per_shard);
    return true;
}

// Workgroup `block` of four waves, one wave per cell (Section "Submodel execution": the working buffer).
template <typename Table>
__device__ inline void decode_split_block(const SplitDecodeJob &job, const Table &tab, int block, u32x2 (&lut)[4][kLutEntries])
{
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int cell = block * 4 + wave;
    if (cell >= job.cells) return;   // whole wave; no workgroup barrier is used
    const CellMap &m = job.map;   // (per_shard: cells of a shard that the launch decodes)
    const int d = m.d, dh = m.dh, f = m.f;
    const int shard = quotient(cell, m.per_shard, m.recip_shard);
    const TiledCell t = locate_cell_of_shard(shard, cell - shard * m.per_shard + job.skip, m);
    const ShardDesc sd = tab.get(shard);
    const int64_t attention = (int64_t)4 * dh * d, ffn = (int64_t)f * d;
    const int64_t at = job.skip == 0 ? shard * attention + t.sub_off : (t.sub_off == attention ? job.n_shards + shard : shard) * ffn;
    u32x4 *cell_out = (u32x4 *)(job.out + at * 3) + ((int64_t)t.strip * (t.cols >> 6) + t.kt) * 768 + lane;
    const int64_t elem = t.sub_off + (int64_t)(t.strip * 32 + (lane & 31)) * t.cols + t.kt * 64 + (lane >> 5) * 32;
    auto store = [&](int q, const uint32_t (&x)[4][3]) {   // four pairs of weights
#pragma unroll
        for (int p = 0; p < 3; ++p) cell_out[(p * 4 + q) * 64] = u32x4{x[0][p], x[1][p], x[2][p], x[3][p]};
    };
    if (sd.bits == 32) {
        const f32x4 *src = (const f32x4 *)((const float *)sd.data + elem);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const f32x4 a = src[2 * q], b = src[2 * q + 1];
            uint32_t x[4][3];
            split_pair(a.x, a.y, x[0]);
            split_pair(a.z, a.w, x[1]);
            split_pair(b.x, b.y, x[2]);
            split_pair(b.z, b.w, x[3]);
            store(q, x);
        }
        return;
    }
    if (lane < (1 << sd.bits)) {
        uint32_t c[3];
        split_pair(sd.codebook[lane], 0.f, c);
        lut[wave][lane] = u32x2{(c[0] & 0xFFFFu) | c[1] << 16, c[2]};
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    auto packed = [&](auto width) {
        constexpr int BITS = decltype(width)::value;
        const Raw r = load_raw<BITS>((const uint8_t *)sd.data + (elem >> 5) * (BITS * 4));
        const uint32_t rv[8] = {r.a.x, r.a.y, r.a.z, r.a.w, r.b.x, r.b.y, r.b.z, r.b.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uint32_t x[4][3];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                u32x2 c[2];
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const int bit = (q * 8 + 2 * e + k) * BITS, dw = bit >> 5, sh = bit & 31;
                    uint32_t v = rv[dw] >> sh;
                    if (sh + BITS > 32) v |= rv[dw + 1] << (32 - sh);
                    c[k] = lut[wave][v & ((1u << BITS) - 1u)];
                }
                x[e][0] = (c[0].x & 0xFFFFu) | c[1].x << 16;
                x[e][1] = c[0].x >> 16 | (c[1].x & 0xFFFF0000u);
                x[e][2] = (c[0].y & 0xFFFFu) | c[1].y << 16;
            }
            store(q, x);
        }
    };
    switch (sd.bits) {
    case 2: packed(std::integral_constant<int, 2>{}); break;
    case 3: packed(std::integral_constant<int, 3>{}); break;
    case 4: packed(std::integral_constant<int, 4>{}); break;
    case 5: packed(std::integral_constant<int, 5>{}); break;
    default: packed(std::integral_constant<int, 6>{}); break;
    }
}

}  // namespace sti
