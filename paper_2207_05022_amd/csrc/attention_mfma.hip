// Per-head attention on the matrix cores: C = softmax(Q K^T / sqrt(dh)) V for
// one (sequence, present head) per workgroup column (Section "A primer on
// transformer": each head contributes its own attention score).
//
// Everything is computed transposed so that the softmax never crosses lanes:
//   S^T = K Q^T   -> a lane owns one query (MFMA column) and 16 keys per
//                    32-key block in its accumulator registers;
//   O^T = V^T P^T -> the probabilities are already in the register layout the
//                    B operand needs once the key order inside each k16 step
//                    is permuted, and V^T is read from LDS in that same order.
// The maximum and the sum of a query's row are per lane; lanes l and l^32 own the two
// halves of a query's keys and exchange their maxima (once in all for short sequences, once per
// key block with the running maximum of the online softmax otherwise).
//
// Padded sequences (the input length is fixed after padding, Section "Prerequisite: Offline
// Profiling"): with key_lengths, sequence b attends to its first key_lengths[b] positions only
// (clamped to 1..L); rows of padded positions are still computed, from those keys.
#include <float.h>
#include "sti_internal.hpp"
#include "attention_core.hpp"

namespace sti {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef float float16v __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int DH = 64;
constexpr int KPAD = DH + 8;   // padded K row (halves)

__device__ inline int vt_stride(int Lp) { return Lp + 8; }

// Sequences of at most 128 tokens: NW waves of 32 queries; all scores stay in registers, the row maximum is known before
// the first exponential, and the output accumulators are never rescaled (attention_core.hpp).
template <int NW>
__global__ __launch_bounds__(NW * 64, 2) void attention_mfma_kernel(const _Float16 *qkv, _Float16 *ctx,
                                                                 int L, int Lp, int m, int ctx_tiled,
                                                                 const int32_t *key_lengths, AttentionPieces pieces)
{
    constexpr int QB = NW * 32;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    _Float16 *Ks = (_Float16 *)smem_raw;                 // [Lp][KPAD]
    _Float16 *Vt = Ks + (size_t)Lp * KPAD;               // [DH][Lp + 8]
    const int vts = vt_stride(Lp);
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int g = lane >> 5, lr = lane & 31;
    const AttentionPiece piece = attention_piece(pieces, m, (L + QB - 1) / QB);
    if (piece.none) return;
    const int b = piece.sequence, p = piece.head;
    const int64_t ld = (int64_t)m * 3 * DH;
    const _Float16 *base = qkv + (int64_t)b * L * ld + (int64_t)p * 3 * DH;
    int Lk = L;   // keys that take part
    if (key_lengths) Lk = min(max(key_lengths[b], 1), L);

    // this lane's query row as the B operand of S^T = K Q^T (asked for first: the loads below
    // and these share one round trip to memory)
    const int q = piece.block * QB + wave * 32 + lr;
    half8 qf[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        u32x4 v = {0, 0, 0, 0};
        if (q < L) v = *(const u32x4 *)(base + (int64_t)q * ld + s * 16 + g * 8);
        qf[s] = __builtin_bit_cast(half8, v);
    }

    // Stage K (row-major; rows >= Lk are zero) and V transposed: all loads are issued
    // before the first LDS store, one round trip.
    //   K: a thread takes 16 bytes of rows tid/8 + 8 NW j;
    //   V: a lane takes two consecutive keys and 8 features, so that the 64 lanes of one LDS
    //      store write consecutive dwords of one V^T row (no bank conflicts).
    constexpr int KJ = 16 / NW;           // K rows per thread
    constexpr int VJ = 8 / NW;            // V key pairs per thread
    const int kc = (tid & 7) * 8;
    const int v_items = (Lp / 2) * 8;
    u32x4 kreg[KJ], v0[VJ], v1[VJ];
#pragma unroll
    for (int j = 0; j < KJ; ++j) {
        const int r = (tid >> 3) + NW * 8 * j;
        kreg[j] = u32x4{0, 0, 0, 0};
        if (r < Lk) kreg[j] = *(const u32x4 *)(base + (int64_t)r * ld + DH + kc);
    }
#pragma unroll
    for (int j = 0; j < VJ; ++j) {
        const int item = tid + NW * 64 * j;
        const int pair = item % (Lp / 2), c = (item / (Lp / 2)) * 8;
        const int r0 = 2 * pair;
        v0[j] = u32x4{0, 0, 0, 0};
        v1[j] = u32x4{0, 0, 0, 0};
        if (item < v_items && r0 < Lk) v0[j] = *(const u32x4 *)(base + (int64_t)r0 * ld + 2 * DH + c);
        if (item < v_items && r0 + 1 < Lk) v1[j] = *(const u32x4 *)(base + (int64_t)(r0 + 1) * ld + 2 * DH + c);
    }
#pragma unroll
    for (int j = 0; j < KJ; ++j) {
        const int r = (tid >> 3) + NW * 8 * j;
        if (r < Lp) *(u32x4 *)(Ks + (size_t)r * KPAD + kc) = kreg[j];
    }
#pragma unroll
    for (int j = 0; j < VJ; ++j) {
        const int item = tid + NW * 64 * j;
        if (item >= v_items) continue;
        const int pair = item % (Lp / 2), c = (item / (Lp / 2)) * 8;
        const int r0 = 2 * pair;
        const uint32_t a[4] = {v0[j].x, v0[j].y, v0[j].z, v0[j].w}, bq[4] = {v1[j].x, v1[j].y, v1[j].z, v1[j].w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t lo = (a[i] & 0xFFFFu) | (bq[i] << 16);          // feature c + 2i
            const uint32_t hi = (a[i] >> 16) | (bq[i] & 0xFFFF0000u);      // feature c + 2i + 1
            *(uint32_t *)(Vt + (size_t)(c + 2 * i) * vts + r0) = lo;
            *(uint32_t *)(Vt + (size_t)(c + 2 * i + 1) * vts + r0) = hi;
        }
    }
    __syncthreads();

    float16v o[2];
    const float run_sum = attention_scores_in_registers<4>(qf, Ks, KPAD, Vt, vts, Lk, lane, o);
    if (q >= L) return;
    const float inv = 1.0f / run_sum;
    // (a tiled context: chunk v4 of half e of the head's cell; the strides of e and v4 in elements)
    _Float16 *out = ctx + ((int64_t)b * L + q) * ((int64_t)m * DH) + (int64_t)p * DH;
    int e_step = 32, v4_step = 8;
    if (ctx_tiled) {
        out = ctx + tiled_offset(b * L + q, p * DH, m);
        e_step = 256;
        v4_step = 512;
    }
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int v4 = 0; v4 < 4; ++v4) {
            half4 h;
#pragma unroll
            for (int i = 0; i < 4; ++i) h[i] = (_Float16)(o[e][v4 * 4 + i] * inv);
            *(half4 *)(out + e * e_step + v4 * v4_step + g * 4) = h;
        }
}

// Longer sequences: NW waves of 32 queries walk the keys in blocks of 64 that are staged
// in LDS one block ahead (two buffers, one barrier per block), so that several workgroups share a
// compute unit whatever the length.  Online softmax; the output accumulators are only rescaled when some
// query's maximum moves.
// Bound by the softmax's vector instructions (about 1200 clocks per wave and block, 512 of matrix
// work).  24 sequences of 384 tokens, 16 heads (14.5 GFLOP): 32 us, against 71 us of the kernel that kept all keys of
// a head in LDS (105 KB: one workgroup of four waves per compute unit).  The block that the last key cuts is
// behind the loop, 32 keys at a time: inside it, masked as a whole, it cost the loop 8 spilled registers and the half
// without keys its time (8 sequences of 160 tokens, 12 heads: 8.1 us, now 6.7; the kernel with all keys in LDS 7.5).
constexpr int SB = 64;            // keys per block
constexpr int SV = SB + 8;        // padded V^T row (halves)

template <int NW>
__global__ __launch_bounds__(NW * 64, 4) void attention_stream_kernel(const _Float16 *qkv, _Float16 *ctx, int L, int m, int ctx_tiled,
                                                                   const int32_t *key_lengths, AttentionPieces pieces)
{
    __shared__ __attribute__((aligned(16))) _Float16 Ks[2][SB * KPAD];
    __shared__ __attribute__((aligned(16))) _Float16 Vt[2][DH * SV];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int g = lane >> 5, lr = lane & 31;
    const AttentionPiece piece = attention_piece(pieces, m, (L + NW * 32 - 1) / (NW * 32));
    if (piece.none) return;
    const int b = piece.sequence, p = piece.head;
    const int64_t ld = (int64_t)m * 3 * DH;
    const _Float16 *base = qkv + (int64_t)b * L * ld + (int64_t)p * 3 * DH;
    int Lk = L;   // keys that take part
    if (key_lengths) Lk = min(max(key_lengths[b], 1), L);
    const int q = piece.block * (NW * 32) + wave * 32 + lr;
    half8 qf[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) qf[s] = *(const half8 *)(base + (int64_t)min(q, L - 1) * ld + s * 16 + g * 8);

    // a thread's share of a block: 16 bytes of K rows tid/8 + 8 NW j; two consecutive keys x 8 features of V,
    // stored transposed as dwords (a wave writes consecutive dwords of V^T rows)
    constexpr int KJ = SB / (8 * NW), VJ = SB * 4 / (NW * 64);
    const int kr = tid >> 3, kc = (tid & 7) * 8;
    const char *bytes = (const char *)base;                 // scalar base, 32-bit lane offsets (a sequence has < 2^24 bytes)
    const uint32_t row_bytes = (uint32_t)(ld * 2);
    u32x4 kreg[KJ], v0[VJ], v1[VJ];
    auto request = [&](int kb) {   // (keys past Lk: the last one again; their probabilities are zero)
#pragma unroll
        for (int j = 0; j < KJ; ++j)
            kreg[j] = *(const u32x4 *)(bytes + (uint32_t)min(kb + kr + 8 * NW * j, Lk - 1) * row_bytes + (DH + kc) * 2);
#pragma unroll
        for (int j = 0; j < VJ; ++j) {
            const int item = tid + NW * 64 * j, r0 = kb + 2 * (item & 31), c = (item >> 5) * 8;
            v0[j] = *(const u32x4 *)(bytes + (uint32_t)min(r0, Lk - 1) * row_bytes + (2 * DH + c) * 2);
            v1[j] = *(const u32x4 *)(bytes + (uint32_t)min(r0 + 1, Lk - 1) * row_bytes + (2 * DH + c) * 2);
        }
    };
    auto put = [&](int buf) {
#pragma unroll
        for (int j = 0; j < KJ; ++j) *(u32x4 *)(Ks[buf] + (kr + 8 * NW * j) * KPAD + kc) = kreg[j];
#pragma unroll
        for (int j = 0; j < VJ; ++j) {
            const int item = tid + NW * 64 * j, r0 = 2 * (item & 31), c = (item >> 5) * 8;
            const uint32_t a[4] = {v0[j].x, v0[j].y, v0[j].z, v0[j].w}, d[4] = {v1[j].x, v1[j].y, v1[j].z, v1[j].w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                *(uint32_t *)(Vt[buf] + (c + 2 * i) * SV + r0) = (a[i] & 0xFFFFu) | (d[i] << 16);
                *(uint32_t *)(Vt[buf] + (c + 2 * i + 1) * SV + r0) = (a[i] >> 16) | (d[i] & 0xFFFF0000u);
            }
        }
    };
    const float scale = 0.125f * 1.44269504088896340736f;   // 1/sqrt(64) * log2(e)
    float run_max = -FLT_MAX, run_sum = 0.f;                // (of the unscaled scores, finite: a block may hold none but -infinity; sum: this lane's keys only)
    float16v o[2];
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[e][v] = 0.f;
    request(0);
    put(0);
    __syncthreads();
    auto scores = [&](int buf, int t) {   // of 32 keys
        float16v s;
#pragma unroll
        for (int v = 0; v < 16; ++v) s[v] = 0.f;
#pragma unroll
        for (int f = 0; f < 4; ++f)
            s = __builtin_amdgcn_mfma_f32_32x32x16_f16(*(const half8 *)(Ks[buf] + (t * 32 + lr) * KPAD + f * 16 + g * 8), qf[f], s, 0, 0, 0);
        return s;
    };
    auto rescale = [&](float bmax) {
        bmax = pair_max(across_32(bmax));
        if (__ballot(bmax > run_max)) {
            const float new_max = fmaxf(run_max, bmax);
            const float alpha = __builtin_amdgcn_exp2f((run_max - new_max) * scale);
            run_max = new_max;
            run_sum *= alpha;
#pragma unroll
            for (int e = 0; e < 2; ++e)
#pragma unroll
                for (int v = 0; v < 16; ++v) o[e][v] *= alpha;
        }
    };
    auto weigh = [&](const float16v &s, int buf, int t, float shift) {
        uint32_t pk[8];
#pragma unroll
        for (int v = 0; v < 16; v += 2) {
            const float p0 = __builtin_amdgcn_exp2f(fmaf(s[v], scale, shift));
            const float p1 = __builtin_amdgcn_exp2f(fmaf(s[v + 1], scale, shift));
            run_sum += p0 + p1;
            pk[v / 2] = f16_pair_bits(p0, p1);
        }
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
            const u32x4 pv = {pk[4 * s2], pk[4 * s2 + 1], pk[4 * s2 + 2], pk[4 * s2 + 3]};
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const _Float16 *vrow = Vt[buf] + (e * 32 + lr) * SV + t * 32 + s2 * 16 + g * 4;
                const u32x2 lo = *(const u32x2 *)vrow, hi = *(const u32x2 *)(vrow + 8);
                const u32x4 vv = {lo.x, lo.y, hi.x, hi.y};
                o[e] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, vv), __builtin_bit_cast(half8, pv), o[e], 0, 0, 0);
            }
        }
    };
    int kb = 0, buf = 0;
    for (; kb + SB <= Lk; kb += SB, buf ^= 1) {
        if (kb + SB < Lk) request(kb + SB);
        __builtin_amdgcn_sched_barrier(0);
        const float16v sc[2] = {scores(buf, 0), scores(buf, 1)};
        float bmax = -INFINITY;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) bmax = fmaxf(bmax, sc[t][v]);
        rescale(bmax);
        const float shift = -run_max * scale;
#pragma unroll
        for (int t = 0; t < 2; ++t) weigh(sc[t], buf, t, shift);
        __builtin_amdgcn_sched_barrier(0);
        if (kb + SB < Lk) put(buf ^ 1);
        __syncthreads();
    }
    // the block that the last key cuts: 32 keys at a time, as far as there are any
#pragma unroll 1
    for (int t = 0; kb + t * 32 < Lk; ++t) {
        float16v s = scores(buf, t);
        float bmax = -INFINITY;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int key = kb + t * 32 + (v >> 2) * 8 + g * 4 + (v & 3);
            s[v] = key < Lk ? s[v] : -INFINITY;
            bmax = fmaxf(bmax, s[v]);
        }
        rescale(bmax);
        weigh(s, buf, t, -run_max * scale);
    }
    run_sum = pair_sum(across_32(run_sum));
    // (worked out again instead of kept: the loop uses all 128 registers of four waves per SIMD)
    int t2 = threadIdx.x;
    asm volatile("" : "+v"(t2));
    const int q2 = piece.block * (NW * 32) + (t2 >> 6) * 32 + (t2 & 31), g2 = (t2 >> 5) & 1;
    if (q2 >= L) return;
    const float inv = 1.0f / run_sum;
    _Float16 *out = ctx + ((int64_t)b * L + q2) * ((int64_t)m * DH) + (int64_t)p * DH;
    int e_step = 32, v4_step = 8;
    if (ctx_tiled) {
        out = ctx + tiled_offset(b * L + q2, p * DH, m);
        e_step = 256;
        v4_step = 512;
    }
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int v4 = 0; v4 < 4; ++v4) {
            half4 h;
#pragma unroll
            for (int i = 0; i < 4; ++i) h[i] = (_Float16)(o[e][v4 * 4 + i] * inv);
            *(half4 *)(out + e * e_step + v4 * v4_step + g2 * 4) = h;
        }
}

}  // namespace

hipError_t launch_attention_mfma(const void *qkv, void *ctx, ActLayout ctx_layout, int B, int L, int m, int dh,
                                 const int32_t *key_lengths, hipStream_t stream)
{
    if (B <= 0 || L <= 0 || m <= 0) return hipSuccess;
    if (dh != DH) return hipErrorInvalidValue;
    const int Lp = (L + 31) / 32 * 32;
    const size_t lds = ((size_t)Lp * KPAD + (size_t)DH * (Lp + 8)) * sizeof(_Float16);
    const _Float16 *in = (const _Float16 *)qkv;
    _Float16 *out = (_Float16 *)ctx;
    const int tiled = (int)ctx_layout;
    // The kernel with all keys in LDS up to its 128 keys (93 tokens, 11 x 12 heads: 5.3 us against 6.1); few (sequence,
    // head) pairs: 64 queries per workgroup put twice as many workgroups on the chip.
    const int blocks = L > 128 ? (L + 127) / 128 : (int64_t)B * m < 128 && L > 32 ? (L + 63) / 64 : 1;
    const AttentionPieces pieces = attention_pieces(B, m, blocks);
    const dim3 grid(8 * pieces.per_xcd);
    if (L > 128) launch((attention_stream_kernel<4>), grid, dim3(256), 0, stream, in, out, L, m, tiled, key_lengths, pieces);
    else if ((int64_t)B * m < 128 && L > 32) launch((attention_mfma_kernel<2>), grid, dim3(128), lds, stream, in, out, L, Lp, m, tiled, key_lengths, pieces);
    else launch((attention_mfma_kernel<4>), grid, dim3(256), lds, stream, in, out, L, Lp, m, tiled, key_lengths, pieces);
    return hipGetLastError();
}

}  // namespace sti
