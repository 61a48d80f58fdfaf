// Sums and maxima over groups of lanes without LDS: rotations inside 16 lanes are part of the adding instruction (DPP), rows
// of 16 and halves of 32 change places through v_permlane16_swap / v_permlane32_swap.  A step is 4 to 8 clocks; a shuffle goes through
// the LDS pipe and costs its round trip of about 100.  Every lane of a group ends with the same bits.
// LayerNorm's two sums per row, attention's maxima and sums: 12 layers of BERT-base, 9 of 12 shards, 128 tokens 334 -> 322 us (the order of
// LayerNorm's arguments included); 11 x 93 tokens 683 -> 671; 24 layers of d_model 1024, 24 x 384 tokens 2.2 % faster.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sti {

template <int N>
__device__ inline float rotated(float v)   // by N lanes inside each row of 16
{
    const int r = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x120 + N, 0xf, 0xf, true);
    return __builtin_bit_cast(float, r);
}

struct LanePair {
    float a, b;   // a lane's value and its partner's, in the same order on both
};
__device__ inline LanePair across_16(float v)   // partner: lane ^ 16
{
    const uint32_t u = __builtin_bit_cast(uint32_t, v);
    const auto s = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const uint32_t a = s[0], b = s[1];
    return {__builtin_bit_cast(float, a), __builtin_bit_cast(float, b)};
}
__device__ inline LanePair across_32(float v)   // partner: lane ^ 32
{
    const uint32_t u = __builtin_bit_cast(uint32_t, v);
    const auto s = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    const uint32_t a = s[0], b = s[1];
    return {__builtin_bit_cast(float, a), __builtin_bit_cast(float, b)};
}
__device__ inline float pair_sum(LanePair p) { return p.a + p.b; }
__device__ inline float pair_max(LanePair p) { return fmaxf(p.a, p.b); }

// Sum over groups of LANES (16, 32 or 64) consecutive lanes, halves first: the order (and the bits) of butterflies of lane ^ 32, 16, 8, 4,
// 2, 1, as after each step the values repeat themselves with that step's distance.
template <int LANES>
__device__ inline float lane_sum(float v)
{
    static_assert(LANES == 16 || LANES == 32 || LANES == 64, "rows of 16 lanes");
    if constexpr (LANES >= 64) v = pair_sum(across_32(v));
    if constexpr (LANES >= 32) v = pair_sum(across_16(v));
    v += rotated<8>(v);
    v += rotated<4>(v);
    v += rotated<2>(v);
    v += rotated<1>(v);
    return v;
}

// ---- 32-bit integers, and 64-bit values as two halves ----
template <int CTRL, int ROWS = 0xf>
__device__ inline uint32_t moved(uint32_t v)   // by a DPP control; 0 where no lane of the group is there, or in rows that ROWS leaves out
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
}
template <int CTRL, int ROWS = 0xf>
__device__ inline uint64_t moved(uint64_t v)
{
    return (uint64_t)moved<CTRL, ROWS>((uint32_t)(v >> 32)) << 32 | moved<CTRL, ROWS>((uint32_t)v);
}
template <int CTRL>
__device__ inline double moved(double v)
{
    return __builtin_bit_cast(double, moved<CTRL>(__builtin_bit_cast(uint64_t, v)));
}

// inclusive sums over the wave (T: uint32_t or uint64_t)
template <typename T>
__device__ inline T lane_scan(T v)
{
    v += moved<0x111>(v);        // row_shr: 1, 2, 4 and 8 lanes inside each row of 16
    v += moved<0x112>(v);
    v += moved<0x114>(v);
    v += moved<0x118>(v);
    v += moved<0x142, 0xa>(v);   // row_bcast:15: a row's last lane to the next row (rows 1 and 3)
    v += moved<0x143, 0xc>(v);   // row_bcast:31: lane 31 to the upper half
    return v;
}

// A tree over lanes i and i + 32, 16, 8, 4, 2, 1, as lane 0 ends with it (the order of shuffles downwards).
template <typename Op>
__device__ inline double lane_tree(double v, Op op)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)u, (uint32_t)u, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
    const uint32_t l0 = lo[0], l1 = lo[1], h0 = hi[0], h1 = hi[1];
    v = op(__builtin_bit_cast(double, (uint64_t)h0 << 32 | l0), __builtin_bit_cast(double, (uint64_t)h1 << 32 | l1));
    const uint64_t t = __builtin_bit_cast(uint64_t, v);
    const auto lo2 = __builtin_amdgcn_permlane16_swap((uint32_t)t, (uint32_t)t, false, false);
    const auto hi2 = __builtin_amdgcn_permlane16_swap((uint32_t)(t >> 32), (uint32_t)(t >> 32), false, false);
    const uint32_t a0 = lo2[0], a1 = lo2[1], b0 = hi2[0], b1 = hi2[1];
    v = op(__builtin_bit_cast(double, (uint64_t)b0 << 32 | a0), __builtin_bit_cast(double, (uint64_t)b1 << 32 | a1));
    v = op(v, moved<0x108>(v));   // row_shl
    v = op(v, moved<0x104>(v));
    v = op(v, moved<0x102>(v));
    v = op(v, moved<0x101>(v));
    return v;
}

}  // namespace sti
