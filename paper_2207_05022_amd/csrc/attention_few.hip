// Attention for few tokens (Section "A primer on transformer": each head contributes its own attention
// score): Q, K and V arrive from the projection fragment-tiled (V transposed), so that every operand of both
// products is a contiguous 1 KiB load straight into registers, without LDS.
//
// A workgroup takes 32 queries of one (sequence, head); its W waves share out the 32-key blocks, each with
// a running maximum of its own, and combine at the end through LDS.  As in attention_core.hpp everything is
// computed transposed (S^T = K Q^T, O^T = V^T P^T): a lane pair l, l ^ 32 owns one query, and the
// probabilities are already in the layout of the second product's operand.
//
// Bound by latency: one round trip for all operands, two short products, one barrier.  One sequence of 128
// tokens, 12 heads: 3.5 us, against 5.7 us of the kernel that stages K and V of a whole head in LDS per workgroup.
#include <float.h>
#include "sti_internal.hpp"
#include "weight_loader.hpp"
#include "lane_ops.hpp"

namespace sti {
namespace {

typedef _Float16 half4 __attribute__((ext_vector_type(4)));

template <int W>
__global__ __launch_bounds__(W * 64) void attention_few_kernel(const _Float16 *qkv, _Float16 *ctx, int L, int m,
                                                               const int32_t *key_lengths)
{
    __shared__ f32x4 part[W > 1 ? W : 1][8][64];   // unnormalised context: [feature quarter-blocks][lane]
    __shared__ float part_max[W][64], part_sum[W][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 5, lr = lane & 31;
    const int head = blockIdx.y, b = blockIdx.z;
    const int blocks = (L + 31) >> 5;              // 32-row blocks of a sequence (one sequence, or L a multiple of 32)
    const int rb = b * blocks + blockIdx.x;        // the queries' row block
    const u32x4 *cells = (const u32x4 *)qkv;
    auto cell = [&](int row_block, int which) { return cells + ((int64_t)row_block * (3 * m) + head * 3 + which) * 256 + lane; };
    int Lk = L;
    if (key_lengths) Lk = min(max(key_lengths[b], 1), L);
    const int nkb = (Lk + 31) >> 5;
    u32x4 qf[4], kf[4], vf[4];
    auto request = [&](int kb) {
        const u32x4 *k = cell(b * blocks + kb, 1), *v = cell(b * blocks + kb, 2);
#pragma unroll
        for (int s = 0; s < 4; ++s) kf[s] = k[s * 64];
#pragma unroll
        for (int s = 0; s < 4; ++s) vf[s] = v[s * 64];
    };
    {
        const u32x4 *q = cell(rb, 0);
#pragma unroll
        for (int s = 0; s < 4; ++s) qf[s] = q[s * 64];
    }
    int kb = wave;
    if (kb < nkb) request(kb);
    const float scale = 0.125f * 1.44269504088896340736f;   // 1/sqrt(64) * log2(e)
    float run_max = -FLT_MAX, run_sum = 0.f;                // (of the scaled scores; finite: a block may hold none but -infinity)
    float16v o[2];
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[e][v] = 0.f;
    for (; kb < nkb; kb += W) {
        float16v s_acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) s_acc[v] = 0.f;
#pragma unroll
        for (int s = 0; s < 4; ++s)
            s_acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, kf[s]), __builtin_bit_cast(half8, qf[s]), s_acc, 0, 0, 0);
        u32x4 v_now[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) v_now[s] = vf[s];
        if (kb + W < nkb) request(kb + W);
        if (kb * 32 + 32 > Lk) {
            // keys past the last one (padding, rows past the last token): their probabilities are zero, and their values
            // have to be, since 0 times an infinity or NaN would reach every query.  Dword w of a fragment: two keys.
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const int key = kb * 32 + (s & 1) * 16 + (w >> 1) * 8 + g * 4 + (w & 1) * 2;
                    v_now[s][w] = key + 1 < Lk ? v_now[s][w] : key < Lk ? v_now[s][w] & 0xFFFFu : 0u;
                }
        }
        float bmax = -INFINITY;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int key = kb * 32 + (v >> 2) * 8 + g * 4 + (v & 3);
            const float x = (key < Lk) ? s_acc[v] * scale : -INFINITY;
            s_acc[v] = x;
            bmax = fmaxf(bmax, x);
        }
        bmax = pair_max(across_32(bmax));
        const float new_max = fmaxf(run_max, bmax);
        const float alpha = __builtin_amdgcn_exp2f(run_max - new_max);
        run_max = new_max;
        float psum = 0.f;
        uint32_t pk[8];
#pragma unroll
        for (int v = 0; v < 16; v += 2) {
            const float p0 = __builtin_amdgcn_exp2f(s_acc[v] - new_max);
            const float p1 = __builtin_amdgcn_exp2f(s_acc[v + 1] - new_max);
            psum += p0 + p1;
            pk[v / 2] = f16_pair_bits(p0, p1);
        }
        run_sum = run_sum * alpha + psum;
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int v = 0; v < 16; ++v) o[e][v] *= alpha;
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
            const u32x4 pv = {pk[4 * s2], pk[4 * s2 + 1], pk[4 * s2 + 2], pk[4 * s2 + 3]};
#pragma unroll
            for (int e = 0; e < 2; ++e)
                o[e] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, v_now[e * 2 + s2]), __builtin_bit_cast(half8, pv), o[e], 0, 0, 0);
        }
    }
    run_sum = pair_sum(across_32(run_sum));
    // o[e][4 v4 + i]: feature e*32 + v4*8 + g*4 + i of query lr -> 16-byte chunk (v4, e*32 + lr) of the context's cell
    _Float16 *out = ctx + ((int64_t)rb * m + head) * 2048 + g * 4;
    auto store = [&](int e, int v4, f32x4 x, float inv) {
        *(half4 *)(out + v4 * 512 + (e * 32 + lr) * 8) = half4{(_Float16)(x[0] * inv), (_Float16)(x[1] * inv), (_Float16)(x[2] * inv), (_Float16)(x[3] * inv)};
    };
    if constexpr (W == 1) {
        const float inv = 1.0f / run_sum;
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4)
                store(e, v4, f32x4{o[e][4 * v4], o[e][4 * v4 + 1], o[e][4 * v4 + 2], o[e][4 * v4 + 3]}, inv);
    } else {
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4)
                part[wave][e * 4 + v4][lane] = f32x4{o[e][4 * v4], o[e][4 * v4 + 1], o[e][4 * v4 + 2], o[e][4 * v4 + 3]};
        part_max[wave][lane] = run_max;
        part_sum[wave][lane] = run_sum;
        __syncthreads();
        float mx = -INFINITY, factor[W], total = 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w) mx = fmaxf(mx, part_max[w][lane]);
#pragma unroll
        for (int w = 0; w < W; ++w) {               // (waves without a key block: factor 0)
            factor[w] = __builtin_amdgcn_exp2f(part_max[w][lane] - mx);
            total += part_sum[w][lane] * factor[w];
        }
        const float inv = 1.0f / total;
#pragma unroll
        for (int j = 0; j < 8 / W; ++j) {
            const int ev = wave * (8 / W) + j;
            f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < W; ++w) x += part[w][ev][lane] * factor[w];
            store(ev >> 2, ev & 3, x, inv);
        }
    }
}

}  // namespace

bool attention_few_supported(int B, int L) { return B == 1 || L % 32 == 0; }

hipError_t launch_attention_few(const void *qkv, void *ctx, int B, int L, int m, int dh, const int32_t *key_lengths,
                                hipStream_t stream)
{
    if (B <= 0 || L <= 0 || m <= 0) return hipSuccess;
    if (dh != 64 || !attention_few_supported(B, L)) return hipErrorInvalidValue;
    const dim3 grid((L + 31) / 32, m, B);
    const _Float16 *q = (const _Float16 *)qkv;
    _Float16 *c = (_Float16 *)ctx;
    if (L <= 32) launch((attention_few_kernel<1>), grid, dim3(64), 0, stream, q, c, L, m, key_lengths);
    else if (L <= 64) launch((attention_few_kernel<2>), grid, dim3(128), 0, stream, q, c, L, m, key_lengths);
    else launch((attention_few_kernel<4>), grid, dim3(256), 0, stream, q, c, L, m, key_lengths);
    return hipGetLastError();
}

}  // namespace sti
