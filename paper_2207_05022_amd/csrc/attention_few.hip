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
#include <string.h>
#include <type_traits>
#include "sti_internal.hpp"
#include "weight_loader.hpp"
#include "lane_ops.hpp"
#include "few_tiles.hpp"

namespace sti {
namespace {

constexpr float kScale = 0.125f * 1.44269504088896340736f;   // 1/sqrt(64) * log2(e)

// One wave's queries (a row block) of one head, and what it has of their attention so far.
struct FewHead {
    u32x4 q[4];                 // the queries as an operand
    float16v o[2];              // unnormalised context
    float run_max, run_sum;     // (of the scaled scores; finite: a block may hold none but -infinity)
};
__device__ inline void request_cell(const u32x4 *cell, u32x4 (&x)[4])
{
#pragma unroll
    for (int s = 0; s < 4; ++s) x[s] = cell[s * 64];
}
__device__ inline void no_attention_yet(FewHead &t)
{
    t.run_max = -FLT_MAX;
    t.run_sum = 0.f;
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int v = 0; v < 16; ++v) t.o[e][v] = 0.f;
}
// scores of one block of keys, transposed: a lane's query against 16 of them
__device__ inline float16v scores(const u32x4 (&k)[4], const u32x4 (&q)[4])
{
    float16v s_acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) s_acc[v] = 0.f;
#pragma unroll
    for (int s = 0; s < 4; ++s)
        s_acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, k[s]), __builtin_bit_cast(half8, q[s]), s_acc, 0, 0, 0);
    return s_acc;
}
// that block's part of the softmax and of the context; val: its values
__device__ inline void attend_block(FewHead &t, float16v s_acc, u32x4 (&val)[4], int kb, int Lk, int g)
{
    if (kb * 32 + 32 > Lk) {
        // keys past the last one (padding, rows past the last token): their probabilities are zero, and their values
        // have to be, since 0 times an infinity or NaN would reach every query.  Dword w of a fragment: two keys.
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const int key = kb * 32 + (s & 1) * 16 + (w >> 1) * 8 + g * 4 + (w & 1) * 2;
                val[s][w] = key + 1 < Lk ? val[s][w] : key < Lk ? val[s][w] & 0xFFFFu : 0u;
            }
    }
    float bmax = -INFINITY;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int key = kb * 32 + (v >> 2) * 8 + g * 4 + (v & 3);
        const float x = (key < Lk) ? s_acc[v] * kScale : -INFINITY;
        s_acc[v] = x;
        bmax = fmaxf(bmax, x);
    }
    bmax = pair_max(across_32(bmax));
    const float new_max = fmaxf(t.run_max, bmax);
    const float alpha = __builtin_amdgcn_exp2f(t.run_max - new_max);
    t.run_max = new_max;
    float psum = 0.f;
    uint32_t pk[8];
#pragma unroll
    for (int v = 0; v < 16; v += 2) {
        const float p0 = __builtin_amdgcn_exp2f(s_acc[v] - new_max);
        const float p1 = __builtin_amdgcn_exp2f(s_acc[v + 1] - new_max);
        psum += p0 + p1;
        pk[v / 2] = f16_pair_bits(p0, p1);
    }
    t.run_sum = t.run_sum * alpha + psum;
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int v = 0; v < 16; ++v) t.o[e][v] *= alpha;
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2) {
        const u32x4 pv = {pk[4 * s2], pk[4 * s2 + 1], pk[4 * s2 + 2], pk[4 * s2 + 3]};
#pragma unroll
        for (int e = 0; e < 2; ++e)
            t.o[e] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, val[e * 2 + s2]), __builtin_bit_cast(half8, pv), t.o[e], 0, 0, 0);
    }
}

// store(e, v4, x): features e*32 + v4*8 + g*4 .. + 3 of query lr, the 16-byte chunk (v4, e*32 + lr) of the context's cell
template <typename Store>
__device__ inline void store_whole(const FewHead &t, Store store)   // one wave per head
{
    const float inv = 1.0f / t.run_sum;
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int v4 = 0; v4 < 4; ++v4)
            store(e, v4, f32x4{t.o[e][4 * v4], t.o[e][4 * v4 + 1], t.o[e][4 * v4 + 2], t.o[e][4 * v4 + 3]} * inv);
}
__device__ inline half4 rounded(f32x4 x) { return half4{(_Float16)x[0], (_Float16)x[1], (_Float16)x[2], (_Float16)x[3]}; }

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
    const int64_t block_stride = (int64_t)(3 * m) * 256;   // (from a row block's cell of a head to the next one's; values lie behind keys)
    const u32x4 *cells = (const u32x4 *)qkv + head * 3 * 256 + lane, *keys = cells + b * blocks * block_stride + 256;
    int Lk = L;
    if (key_lengths) Lk = min(max(key_lengths[b], 1), L);
    const int nkb = (Lk + 31) >> 5;
    FewHead t;
    u32x4 kf[4], vf[4];
    auto request = [&](int kb) {
        request_cell(keys + kb * block_stride, kf);
        request_cell(keys + kb * block_stride + 256, vf);
    };
    request_cell(cells + rb * block_stride, t.q);
    int kb = wave;
    if (kb < nkb) request(kb);
    no_attention_yet(t);
    for (; kb < nkb; kb += W) {
        const float16v s_acc = scores(kf, t.q);
        u32x4 v_now[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) v_now[s] = vf[s];
        if (kb + W < nkb) request(kb + W);
        attend_block(t, s_acc, v_now, kb, Lk, g);
    }
    t.run_sum = pair_sum(across_32(t.run_sum));
    _Float16 *out = ctx + ((int64_t)rb * m + head) * 2048 + g * 4;
    auto store = [&](int e, int v4, f32x4 x) { *(half4 *)(out + v4 * 512 + (e * 32 + lr) * 8) = rounded(x); };
    if constexpr (W == 1) {
        store_whole(t, store);
    } else {
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4)
                part[wave][e * 4 + v4][lane] = f32x4{t.o[e][4 * v4], t.o[e][4 * v4 + 1], t.o[e][4 * v4 + 2], t.o[e][4 * v4 + 3]};
        part_max[wave][lane] = t.run_max;
        part_sum[wave][lane] = t.run_sum;
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
            store(ev >> 2, ev & 3, x * inv);
        }
    }
}

// ---- attention and output projection in one launch -------------------------------------------------
// A workgroup of four waves: each the attention of one head for 32 queries, all keys (64 at most) requested at once, and then that head's part of the product (one
// 64-wide K tile) for one strip of 32 output columns.  The sums over the four heads leave as one plane of partial sums, which LayerNorm
// adds.
//
// Bound by latency, like its parts: it saves a launch and its round trip for an attention that is worked out once per strip and as
// many planes as there are groups of four heads.  One sequence, 9 heads of BERT-base, us: 23 tokens 3.2 + 3.8 and LayerNorm 2.6 -> 4.4 and 3.2,
// 64 tokens 3.3 + 3.9 and 3.2 -> 5.2 and 3.8; on the host a launch less of seven.  Workgroups of six heads 5.2 for 23 tokens, of twelve
// 6.2: the operands (12 KB per wave and key block) through one L1.
// The packed weights of the wave's tile (in one piece: rows of 64) go straight to LDS in the meantime: a switch on the
// bitwidth around loads into registers makes the compiler wait for them where its cases join.
constexpr int kOutHeads = 4;

struct FewOutSmem {
    union {
        unsigned char raw[8192];     // a wave's weights as stored
        f32x4 red[4][64];            // its products
    } wave[kOutHeads];
    _Float16 ctx[kOutHeads][2048];   // context cells
    uint16_t lut[kOutHeads][kLutEntries];
};

typedef __attribute__((address_space(3))) void lds_ptr;

// The 64-wide tile of strip `strip` of a weight block of 64 columns, as stored: 256 bytes per bit of a weight.  Chunks of 16 bytes of a float32
// row change places (by the row) so that a column of chunks does not lie in the same banks.
__device__ inline void request_strip(const GemmBlock &desc, int strip, int lane, unsigned char *raw)
{
    // (written as instructions: the compiler would wait for these in front of the next LDS read)
    uint32_t dst = (uint32_t)(size_t)(lds_ptr *)raw;
    const int bits = desc.bits;
    if (bits <= 6) {
        const uint8_t *base = (const uint8_t *)desc.w + (int64_t)strip * (256 * bits);
        for (int i = 0; i < bits; ++i)
            asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" :: "v"((uint32_t)(i * 256 + lane * 4)), "s"(base), "s"(dst + i * 256) : "memory", "m0");
        return;
    }
    const int kib = bits == kTiledBits ? 4 : 8;
    const uint8_t *base = (const uint8_t *)desc.w + (int64_t)strip * (1024 * kib);
    for (int i = 0; i < kib; ++i) {
        const int chunk = bits == kTiledBits ? lane & 15 : (lane & 15) ^ ((i * 4 + (lane >> 4)) & 15);
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" :: "v"((uint32_t)(i * 1024 + (lane >> 4) * 256 + chunk * 16)), "s"(base), "s"(dst + i * 1024) : "memory", "m0");
    }
}
__device__ inline void strip_fragments(int bits, const unsigned char *raw, float centroid, uint16_t *lut, int lane, half8 (&f)[4])
{
    lut[lane] = (uint16_t)f16_bits(centroid);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    wave_lds_fence();
    auto packed = [&](auto width) {   // (rows of 64 weights: two runs of 32; the lane's is run lane >> 5 of row lane & 31)
        constexpr int BITS = decltype(width)::value;
        decode_raw<BITS>(load_raw<BITS>(raw + ((lane & 31) * 2 + (lane >> 5)) * (BITS * 4)), lut, f);
    };
    switch (bits) {
    case 2: packed(std::integral_constant<int, 2>{}); break;
    case 3: packed(std::integral_constant<int, 3>{}); break;
    case 4: packed(std::integral_constant<int, 4>{}); break;
    case 5: packed(std::integral_constant<int, 5>{}); break;
    case 6: packed(std::integral_constant<int, 6>{}); break;
    case kTiledBits:
#pragma unroll
        for (int q = 0; q < 4; ++q) f[q] = *(const half8 *)(raw + q * 1024 + lane * 16);
        break;
    default:
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int chunk = (lane >> 5) * 8 + q * 2 + c;
                const f32x4 v = *(const f32x4 *)(raw + (lane & 31) * 256 + (chunk ^ (lane & 15)) * 16);
#pragma unroll
                for (int e = 0; e < 4; ++e) f[q][c * 4 + e] = (_Float16)v[e];
            }
    }
}

// grid: x = strip, y = group of heads, z = 32-row block; NKB: blocks of keys, at most; blocks_recip: quotients by the row blocks of a sequence
template <int NKB, int NB>
__global__ __launch_bounds__(kOutHeads * 64, 2) void attention_out_few_kernel(const _Float16 *qkv, const int32_t *key_lengths, float *out, int L, int m,
                                                                              int T, int N, uint32_t blocks_recip, int64_t partial_stride, FewBlocks<NB> blocks)
{
    __shared__ __attribute__((aligned(16))) FewOutSmem sm;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 5, lr = lane & 31;
    const int seq_blocks = (L + 31) >> 5, rb = blockIdx.z, b = quotient(rb, seq_blocks, blocks_recip);
    const int head = blockIdx.y * kOutHeads + wave, strip = blockIdx.x;
    float16v acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    if (head < m) {
        const int64_t block_stride = (int64_t)(3 * m) * 256;
        const u32x4 *cells = (const u32x4 *)qkv + head * 3 * 256 + lane, *keys = cells + (int64_t)b * seq_blocks * block_stride + 256;
        FewHead t;
        u32x4 k[NKB][4], val[NKB][4];
        request_cell(cells + rb * block_stride, t.q);
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {     // (padding, too: the length may not be there yet; blocks past the last one: that one)
            const u32x4 *cell = keys + min(kb, seq_blocks - 1) * block_stride;
            request_cell(cell, k[kb]);
            request_cell(cell + 256, val[kb]);
        }
        __builtin_amdgcn_sched_barrier(0);
        const GemmBlock desc = blocks.b[head];
        float centroid = 0.f;
        if (desc.bits <= 6) centroid = desc.codebook[lane & ((1 << desc.bits) - 1)];
        request_strip(desc, strip, lane, sm.wave[wave].raw);
        int Lk = L;
        if (key_lengths) Lk = min(max(key_lengths[b], 1), L);
        no_attention_yet(t);
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
            if (kb * 32 < Lk) attend_block(t, scores(k[kb], t.q), val[kb], kb, Lk, g);
        }
        t.run_sum = pair_sum(across_32(t.run_sum));
        _Float16 *ctx = sm.ctx[wave];
        store_whole(t, [&](int e, int v4, f32x4 x) { *(half4 *)(ctx + v4 * 512 + (e * 32 + lr) * 8 + g * 4) = rounded(x); });
        half8 f[4];
        strip_fragments(desc.bits, sm.wave[wave].raw, centroid, sm.lut[wave], lane, f);
        wave_lds_fence();
#pragma unroll
        for (int s = 0; s < 4; ++s)
            acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(f[s], *(const half8 *)(ctx + s * 512 + lane * 8), acc, 0, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) sm.wave[wave].red[q][lane] = f32x4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
    __syncthreads();
    const int row = rb * 32 + lr;
    f32x4 x[kOutHeads];
#pragma unroll
    for (int h = 0; h < kOutHeads; ++h) x[h] = sm.wave[h].red[wave][lane];
    if (row < T) *(f32x4 *)(out + blockIdx.y * partial_stride + (int64_t)row * N + strip * 32 + wave * 8 + g * 4) = (x[0] + x[1]) + (x[2] + x[3]);
}

template <int NKB, int NB>
hipError_t launch_attention_out(const GemmProblem &p, const GemmBlocks &blocks, const void *qkv, int L, const int32_t *key_lengths, int64_t partial_stride, hipStream_t stream)
{
    FewBlocks<NB> table;
    memcpy(table.b, blocks.b, sizeof(table.b));
    const dim3 grid(p.block_rows / 32, (p.n_blocks + kOutHeads - 1) / kOutHeads, (p.T + 31) / 32);
    launch((attention_out_few_kernel<NKB, NB>), grid, dim3(kOutHeads * 64), 0, stream, (const _Float16 *)qkv, key_lengths, (float *)p.C, L, p.n_blocks,
           p.T, p.block_rows, reciprocal((uint32_t)((L + 31) / 32)), partial_stride, table);
    return hipGetLastError();
}

inline int waves_per_head(int L) { return L <= 32 ? 1 : L <= 64 ? 2 : 4; }

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
    switch (waves_per_head(L)) {
    case 1: launch((attention_few_kernel<1>), grid, dim3(64), 0, stream, q, c, L, m, key_lengths); break;
    case 2: launch((attention_few_kernel<2>), grid, dim3(128), 0, stream, q, c, L, m, key_lengths); break;
    default: launch((attention_few_kernel<4>), grid, dim3(256), 0, stream, q, c, L, m, key_lengths); break;
    }
    return hipGetLastError();
}

int attention_out_few_planes(const GemmProblem &p, int B, int L)
{
    if (B <= 0 || L <= 0 || L > kFewOutKeys || p.d_head != 64 || p.block_cols != 64 || !attention_few_supported(B, L)) return 0;
    const int planes = (p.n_blocks + kOutHeads - 1) / kOutHeads;
    // Up to one and a half key blocks per compute unit: beyond, the repeated attention costs more than the launch.  12 layers, us, by itself /
    // in one (workgroups x blocks): BERT-base, 9 of 12 shards 64 tokens 306 / 280 (288), 2 x 64 tokens 318 / 320 (576), 8 x 32 tokens 383 / 388
    // (576); d_model 1024, 12 of 16 shards 23 tokens 322 / 305 (96), 64 tokens 339 / 328 (384), 4 x 32 tokens 376 / 372 (384), 2 x 64 tokens
    // 379 / 385 (768).  128 keys: 7.7 / 8.8 us, 7.2 with two waves per head.
    const int64_t workgroups = (int64_t)(p.block_rows / 32) * planes * ((p.T + 31) / 32);
    return workgroups * ((L + 31) / 32) <= 384 ? planes : 0;
}

hipError_t launch_attention_out_few(const GemmProblem &p, const GemmBlocks &blocks, const void *qkv, int B, int L, const int32_t *key_lengths,
                                    int64_t partial_stride, hipStream_t stream)
{
    if (p.n_blocks <= 0 || p.n_blocks > kMaxShardsPerLayer || p.block_rows % 32 || p.ldc != p.block_rows || p.T != B * L || attention_out_few_planes(p, B, L) < 1)
        return hipErrorInvalidValue;
#define STI_OUT(NKB) (p.n_blocks <= 16 ? launch_attention_out<NKB, 16>(p, blocks, qkv, L, key_lengths, partial_stride, stream) \
                                       : launch_attention_out<NKB, kMaxShardsPerLayer>(p, blocks, qkv, L, key_lengths, partial_stride, stream))
    return L <= 32 ? STI_OUT(1) : STI_OUT(2);
#undef STI_OUT
}

}  // namespace sti
