// float32 kernels of the layer: the decompress-into-a-working-buffer route of
// the paper (Section "Submodel execution": shards are decompressed into a
// buffer holding one layer of FP32 weights, then the layer is computed), with
// float32 storage and arithmetic.  Any dimensions are accepted.  The projections of larger layers without outlier dictionaries whose
// dimensions are multiples of 64 go through gemm_f32_split.hip instead, three bfloat16 values to a float32; attention and LayerNorm
// are those of this path.
//
// Products run on the matrix cores in float32 (v_mfma_f32_16x16x4_f32: 256 flops per clock and
// compute unit, float32 multiply and accumulate), in the projections as well as in the attention.
#include <float.h>
#include <type_traits>
#include "sti_internal.hpp"
#include "lane_ops.hpp"
#include "split_planes.hpp"

namespace sti {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kComputeUnits = 256;

// ---------------------------------------------------------------------------
// Projections: C[T x N] = A[T x K] * W^T.
//
// A workgroup of four waves owns a (16 WM RM) x (16 WN CN) tile (WM x WN waves of RM x CN blocks
// of 16 x 16) and walks K in tiles of 32: the tile after next is requested from memory into
// registers while the current one is multiplied out of LDS (two LDS buffers, one barrier per
// tile).  The order of K inside a 16-wide step is permuted (lane group g takes k = 4g .. 4g+3),
// identically for both operands, so that a lane's operands of four MFMAs are one 16-byte LDS read; rows of 36
// floats make those reads conflict free.  The weight is the first operand: a lane's accumulators
// are four consecutive output columns of one token.
//
// Bound by the float32 matrix rate (157 TFLOP/s at the published clock), at few tokens by latency: tile
// sizes and K splits come from choose_f32 below.  BERT-base, 8 x 128 tokens, one layer's four
// projections (14.5 GFLOP, 92 us at that rate): 150 us, against 1150 us of the LDS-tiled product on
// the vector units that this replaces.
//
// VEC: every row of A and W starts on a 16-byte boundary, K is a multiple of 4, the weight blocks span
// less than 4 GiB, and with K split over blocks a block is a whole number of K tiles.
// O and FFN2 leave raw sums (of the K range of split blockIdx.y, at C + split * partial_stride);
// bias, residual and LayerNorm follow in the row kernel.
// ---------------------------------------------------------------------------
constexpr int BK = 32;
constexpr int LDK = BK + 4;

struct F32Args {
    const float *A, *w0;
    int64_t w_stride;                    // distance of two weight blocks (floats)
    float *C;
    int64_t partial_stride;
    const float *bias0, *bias1, *bias2;
    int32_t T, N, K, lda, ldc, block_rows, block_cols, d_head, m_fastest;
    int8_t shard[kMaxShardsPerLayer];    // original shard id of block b (selects the bias slice)
};

template <int KIND, int WM, int RM, int CN, bool VEC>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const F32Args p)
{
    constexpr bool n_split = (KIND == GEMM_QKV || KIND == GEMM_FFN_UP);
    constexpr int WN = 4 / WM;
    constexpr int BM = 16 * WM * RM, BN = 16 * WN * CN;
    __shared__ __attribute__((aligned(16))) float As[2][BM * LDK];
    __shared__ __attribute__((aligned(16))) float Bs[2][BN * LDK];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = wave / WM;
    const int g = lane >> 4, lr = lane & 15;
    // workgroups go to the 8 XCDs in turn: each XCD takes one contiguous range of the tile order, in which
    // the smaller of the two operands is the one every XCD reads in full
    const int n_tiles = (p.N + BN - 1) / BN, m_tiles = (p.T + BM - 1) / BM;
    const int total = n_tiles * m_tiles, per_xcd = (total + 7) / 8;
    const int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per_xcd || tile >= total) return;
    const int tile_m = p.m_fastest ? tile % m_tiles : tile / n_tiles;
    const int tile_n = p.m_fastest ? tile / m_tiles : tile % n_tiles;
    const int m0 = tile_m * BM, n0 = tile_n * BN;
    const int k_tiles = (p.K + BK - 1) / BK;
    const int kt0 = (int)((int64_t)k_tiles * blockIdx.y / gridDim.y);
    const int kt1 = (int)((int64_t)k_tiles * (blockIdx.y + 1) / gridDim.y);

    // ---- loads: VEC: thread = (row tid / 8, 4 floats tid % 8) + 32 rows per item, a scalar base that walks
    //      along K plus a 32-bit offset; else (row tid / 32, 1 float) + 8 rows per item ----
    constexpr int RPI = VEC ? 32 : 8;
    constexpr int AI = (BM + RPI - 1) / RPI, BI = (BN + RPI - 1) / RPI;
    const int row_t = VEC ? tid >> 3 : tid >> 5, col_t = VEC ? (tid & 7) * 4 : tid & 31;
    typedef typename std::conditional<VEC, f32x4, float>::type item_t;
    typedef typename std::conditional<VEC, uint32_t, int64_t>::type offset_t;
    offset_t a_off[AI], b_off[BI];   // VEC: bytes, column included; else: elements of the row's start
    const float *a_base = p.A + (int64_t)m0 * p.lda, *b_base = p.w0;
#pragma unroll
    for (int i = 0; i < AI; ++i) {   // (rows past T or N: the last one again)
        const offset_t row = (offset_t)min(row_t + i * RPI, p.T - 1 - m0) * (offset_t)p.lda;
        a_off[i] = VEC ? (row + col_t) * 4 : row;
    }
#pragma unroll
    for (int i = 0; i < BI; ++i) {
        const int n = min(n0 + row_t + i * RPI, p.N - 1);
        offset_t row = (offset_t)n * (offset_t)p.block_cols;
        if constexpr (n_split) {
            const int blk = n / p.block_rows;
            row = (offset_t)blk * (offset_t)p.w_stride + (offset_t)(n - blk * p.block_rows) * (offset_t)p.block_cols;
        }
        b_off[i] = VEC ? (row + col_t) * 4 : row;
    }
    struct Stage {
        item_t a[AI], b[BI];
    };
    const int k_tail = p.K % BK;
    int kf = kt0;                   // next tile to request
    int kb_rem = 0;                 // K-split kinds: its first k inside its weight block
    if constexpr (VEC) {
        a_base += (int64_t)kt0 * BK;
        if constexpr (n_split) {
            b_base += (int64_t)kt0 * BK;
        } else {
            const int blk = kt0 * BK / p.block_cols;
            kb_rem = kt0 * BK - blk * p.block_cols;
            b_base += blk * p.w_stride + kb_rem;
        }
    }
    // Tiles past the end: the last one again (loaded, never used).
    auto fetch = [&](Stage &st) {
        if constexpr (VEC) {
            if (kf == k_tiles - 1 && k_tail) {   // columns past K: the tile's first ones (zeroed in put())
                const uint32_t back = col_t < k_tail ? 0 : col_t * 4;
#pragma unroll
                for (int i = 0; i < AI; ++i) a_off[i] -= back;
#pragma unroll
                for (int i = 0; i < BI; ++i) b_off[i] -= back;
            }
#pragma unroll
            for (int i = 0; i < AI; ++i)
                if (BM % RPI == 0 || row_t + i * RPI < BM) st.a[i] = *(const item_t *)((const char *)a_base + a_off[i]);
#pragma unroll
            for (int i = 0; i < BI; ++i)
                if (BN % RPI == 0 || row_t + i * RPI < BN) st.b[i] = *(const item_t *)((const char *)b_base + b_off[i]);
            if (kf < k_tiles - 1) {
                a_base += BK;
                b_base += BK;
                if constexpr (!n_split) {
                    kb_rem += BK;
                    if (kb_rem == p.block_cols) {   // (VEC: whole tiles per block)
                        kb_rem = 0;
                        b_base += p.w_stride - p.block_cols;
                    }
                }
            }
        } else {
            const int kk = min(kf * BK + col_t, p.K - 1);
            int64_t kb = kk;
            if constexpr (!n_split) {
                const int blk = kk / p.block_cols;
                kb = blk * p.w_stride + (kk - blk * p.block_cols);
            }
#pragma unroll
            for (int i = 0; i < AI; ++i)
                if (BM % RPI == 0 || row_t + i * RPI < BM) st.a[i] = a_base[a_off[i] + kk];
#pragma unroll
            for (int i = 0; i < BI; ++i)
                if (BN % RPI == 0 || row_t + i * RPI < BN) st.b[i] = b_base[b_off[i] + kb];
        }
        ++kf;
    };
    auto put = [&](int buf, Stage &st, int kt) {
        if (kt == k_tiles - 1 && k_tail && col_t >= k_tail) {
#pragma unroll
            for (int i = 0; i < AI; ++i) st.a[i] = item_t{};
#pragma unroll
            for (int i = 0; i < BI; ++i) st.b[i] = item_t{};
        }
#pragma unroll
        for (int i = 0; i < AI; ++i)
            if (BM % RPI == 0 || row_t + i * RPI < BM) *(item_t *)&As[buf][(row_t + i * RPI) * LDK + col_t] = st.a[i];
#pragma unroll
        for (int i = 0; i < BI; ++i)
            if (BN % RPI == 0 || row_t + i * RPI < BN) *(item_t *)&Bs[buf][(row_t + i * RPI) * LDK + col_t] = st.b[i];
    };

    f32x4 acc[RM][CN];
#pragma unroll
    for (int i = 0; i < RM; ++i)
#pragma unroll
        for (int j = 0; j < CN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    struct Frags {   // the operands of one 16-wide K step
        f32x4 a[RM], b[CN];
    };
    const int a_at = (wm * 16 * RM + lr) * LDK + g * 4, b_at = (wn * 16 * CN + lr) * LDK + g * 4;
    auto read = [&](int buf, int s, Frags &f) {
#pragma unroll
        for (int i = 0; i < RM; ++i) f.a[i] = *(const f32x4 *)&As[buf][a_at + i * 16 * LDK + s * 16];
#pragma unroll
        for (int j = 0; j < CN; ++j) f.b[j] = *(const f32x4 *)&Bs[buf][b_at + j * 16 * LDK + s * 16];
    };
    auto multiply = [&](const Frags &f) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < RM; ++i)
#pragma unroll
                for (int j = 0; j < CN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(f.b[j][e], f.a[i][e], acc[i][j], 0, 0, 0);
    };

    // At step kt: LDS buffer kt & 1 holds tile kt and f0 its first K step; `next` holds tile kt + 1 (on its
    // way), `after` takes tile kt + 2.  Every LDS read and the barrier have products of the other K
    // step behind them.  Nothing is conditional (tiles past the range are loaded and dropped), so that
    // the waits in front of put() leave the loads of tile kt + 2 in flight; the scheduling barriers
    // keep the requests in front of the products.
    static_assert(BK == 32, "two K steps per tile");
    Frags f0, f1;
    auto step = [&](int kt, Stage &next, Stage &after) {
        const int buf = (kt - kt0) & 1;
        read(buf, 1, f1);
        fetch(after);
        __builtin_amdgcn_sched_barrier(0);
        multiply(f0);
        __builtin_amdgcn_sched_barrier(0);
        put(buf ^ 1, next, kt + 1);
        __syncthreads();
        read(buf ^ 1, 0, f0);
        __builtin_amdgcn_sched_barrier(0);
        multiply(f1);
        __builtin_amdgcn_sched_barrier(0);
    };
    if (kt0 < kt1) {
        Stage s0, s1;
        fetch(s0);
        fetch(s1);
        put(0, s0, kt0);
        __syncthreads();
        read(0, 0, f0);
        int kt = kt0;
        for (; kt + 1 < kt1; kt += 2) {
            step(kt, s1, s0);
            step(kt + 1, s0, s1);
        }
        if (kt < kt1) {
            read(0, 1, f1);
            multiply(f0);
            multiply(f1);
        }
    }

    // ---- epilogue: block (i, j): token lr, columns 4g .. 4g + 3 ----
#pragma unroll
    for (int j = 0; j < CN; ++j) {
        const int n = n0 + (wn * CN + j) * 16 + g * 4;
        if (n >= p.N) continue;
        f32x4 bias = {0.f, 0.f, 0.f, 0.f};
        if constexpr (n_split) {
            if (VEC) {   // block_rows and d_head are multiples of 4: one look-up for the four columns
                const int blk = n / p.block_rows, r = n - blk * p.block_rows;
                const float *src;
                if constexpr (KIND == GEMM_QKV) {
                    const int which = r / p.d_head;
                    src = (which == 0 ? p.bias0 : (which == 1 ? p.bias1 : p.bias2)) + p.shard[blk] * p.d_head + r - which * p.d_head;
                } else {
                    src = p.bias0 + p.shard[blk] * p.block_rows + r;
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) bias[v] = src[v];
            } else {
                for (int v = 0; v < 4; ++v) {
                    const int nv = min(n + v, p.N - 1);
                    const int blk = nv / p.block_rows, r = nv - blk * p.block_rows;
                    if constexpr (KIND == GEMM_QKV) {
                        const int which = r / p.d_head;
                        bias[v] = (which == 0 ? p.bias0 : (which == 1 ? p.bias1 : p.bias2))[p.shard[blk] * p.d_head + r - which * p.d_head];
                    } else {
                        bias[v] = p.bias0[p.shard[blk] * p.block_rows + r];
                    }
                }
            }
        }
#pragma unroll
        for (int i = 0; i < RM; ++i) {
            const int m = m0 + (wm * RM + i) * 16 + lr;
            if (m >= p.T) continue;
            f32x4 x = acc[i][j];
            if constexpr (n_split) x += bias;
            if constexpr (KIND == GEMM_FFN_UP) {
#pragma unroll
                for (int v = 0; v < 4; ++v) x[v] = gelu_f32(x[v]);
            }
            float *dst = p.C + (n_split ? 0 : (int64_t)blockIdx.y * p.partial_stride) + (int64_t)m * p.ldc + n;
            if (VEC) {
                *(f32x4 *)dst = x;
            } else {
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (n + v < p.N) dst[v] = x[v];
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Attention: a workgroup of four waves takes 64 queries of one (sequence, head), 16 per wave, and
// walks the keys in blocks of 64 staged in LDS.  S^T = K Q^T leaves a lane with four keys per 16-key block of one
// query, O^T = V^T P^T takes exactly those as its second operand (the K order of the product is
// permuted to it), so probabilities never leave their lane; the row maximum is carried along
// (online softmax).  DB = 16-feature blocks of a head.
// Bound by latency (BERT-base, 8 x 128 tokens: 0.4 GFLOP, 12 us); one wave per query row, which this
// replaces up to 128 features per head, took 68 us there.
// ---------------------------------------------------------------------------
constexpr int KB = 64;   // keys per block

// PLANES: the context goes to the output projection as planes of bfloat16 values (gemm_f32_split.hip).
template <int DB, bool VEC, bool PLANES>
__global__ __launch_bounds__(256) void attention_f32_mfma_kernel(const float *qkv, void *ctx, int L, int m, int dh,
                                                                 const int32_t *key_lengths, AttentionPieces pieces)
{
    constexpr int DP = DB * 16;        // padded features
    constexpr int LDR = DP + 4;        // LDS row (floats): conflict-free in both products
    __shared__ __attribute__((aligned(16))) float Ks[KB * LDR];
    __shared__ __attribute__((aligned(16))) float Vs[KB * LDR];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = lane >> 4, lr = lane & 15;
    const AttentionPiece piece = attention_piece(pieces, m, (L + 63) / 64);
    if (piece.none) return;
    const int b = piece.sequence, head = piece.head;
    const int64_t ld = (int64_t)m * 3 * dh;
    const float *base = qkv + (int64_t)b * L * ld + (int64_t)head * 3 * dh;
    int Lk = L;
    if (key_lengths) Lk = min(max(key_lengths[b], 1), L);
    const int q = piece.block * 64 + wave * 16 + lr;
    const float *qp = base + (int64_t)min(q, L - 1) * ld;
    f32x4 qf[DB];
#pragma unroll
    for (int c = 0; c < DB; ++c) {
        const int e = c * 16 + g * 4;
        if (VEC) {
            qf[c] = *(const f32x4 *)(qp + min(e, dh - 4));
            if (e >= dh) qf[c] = f32x4{0.f, 0.f, 0.f, 0.f};
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v) qf[c][v] = e + v < dh ? qp[min(e + v, dh - 1)] : 0.f;
        }
    }
    const float scale = 1.0f / sqrtf((float)dh);
    float run_max = -FLT_MAX, run_sum = 0.f;   // (finite: a block may hold no score but -infinity)
    f32x4 o[DB];
#pragma unroll
    for (int c = 0; c < DB; ++c) o[c] = f32x4{0.f, 0.f, 0.f, 0.f};

    constexpr int PER_ROW = VEC ? DP / 4 : DP;      // items of a row
    constexpr int ITEMS = (KB * PER_ROW) / 256;     // per thread
    typedef typename std::conditional<VEC, f32x4, float>::type item_t;
    constexpr int W = VEC ? 4 : 1;
    static_assert(ITEMS * 256 == KB * PER_ROW, "whole passes");
    for (int kb = 0; kb < Lk; kb += KB) {
        // keys past Lk: the last one again (their probabilities are zero); features past dh: zero
        item_t kr[VEC ? ITEMS : 1], vr[VEC ? ITEMS : 1];
        auto source = [&](int item, int &row, int &e) -> const float * {
            row = item / PER_ROW;
            e = (item - row * PER_ROW) * W;
            return base + (int64_t)min(kb + row, Lk - 1) * ld + dh + min(e, dh - W);
        };
        if constexpr (VEC) {
#pragma unroll
            for (int i = 0; i < ITEMS; ++i) {
                int row, e;
                const float *src = source(tid + 256 * i, row, e);
                kr[i] = *(const item_t *)src;
                vr[i] = *(const item_t *)(src + dh);
                if (e >= dh) kr[i] = vr[i] = item_t{};
            }
        }
        __syncthreads();   // every wave is done with the previous block
        if constexpr (VEC) {
#pragma unroll
            for (int i = 0; i < ITEMS; ++i) {
                const int item = tid + 256 * i, row = item / PER_ROW, e = (item - row * PER_ROW) * W;
                *(item_t *)&Ks[row * LDR + e] = kr[i];
                *(item_t *)&Vs[row * LDR + e] = vr[i];
            }
        } else {
#pragma unroll 4
            for (int i = 0; i < ITEMS; ++i) {
                int row, e;
                const float *src = source(tid + 256 * i, row, e);
                Ks[row * LDR + e] = e < dh ? src[0] : 0.f;
                Vs[row * LDR + e] = e < dh ? src[dh] : 0.f;
            }
        }
        __syncthreads();
        const int nk = min(Lk - kb, KB), sub = (nk + 15) / 16;   // 16-key blocks that hold a key
        f32x4 s[KB / 16];
        float mx = -INFINITY;
#pragma unroll
        for (int t = 0; t < KB / 16; ++t) {
            s[t] = f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
            if (t >= sub) continue;   // uniform
            f32x4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < DB; ++c) {
                const f32x4 kf = *(const f32x4 *)&Ks[(t * 16 + lr) * LDR + c * 16 + g * 4];
#pragma unroll
                for (int e = 0; e < 4; ++e) a = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[e], qf[c][e], a, 0, 0, 0);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float x = (t * 16 + g * 4 + v < nk) ? a[v] * scale : -INFINITY;
                s[t][v] = x;
                mx = fmaxf(mx, x);
            }
        }
        mx = pair_max(across_32(pair_max(across_16(mx))));
        const float new_max = fmaxf(run_max, mx);
        const float alpha = expf(run_max - new_max);
        run_max = new_max;
        float sum = 0.f;
#pragma unroll
        for (int t = 0; t < KB / 16; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                s[t][v] = expf(s[t][v] - new_max);
                sum += s[t][v];
            }
        run_sum = run_sum * alpha + sum;
#pragma unroll
        for (int c = 0; c < DB; ++c) o[c] *= alpha;
#pragma unroll
        for (int t = 0; t < KB / 16; ++t) {
            if (t >= sub) continue;
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int c = 0; c < DB; ++c)
                    o[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(Vs[(t * 16 + g * 4 + v) * LDR + c * 16 + lr], s[t][v], o[c], 0, 0, 0);
        }
    }
    run_sum = pair_sum(across_32(pair_sum(across_16(run_sum))));
    if (q >= L) return;
    const float inv = 1.0f / run_sum;
    float *out = (float *)ctx + ((int64_t)b * L + q) * ((int64_t)m * dh) + (int64_t)head * dh;
#pragma unroll
    for (int c = 0; c < DB; ++c) {
        const int e = c * 16 + g * 4;
        if constexpr (PLANES) {
            store_planes4((uint16_t *)ctx, b * L + q, head * 64 + e, m, o[c] * inv);
        } else if (VEC) {
            if (e < dh) *(f32x4 *)(out + e) = o[c] * inv;
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (e + v < dh) out[e + v] = o[c][v] * inv;
        }
    }
}

__device__ inline float wave_max(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ inline float wave_sum(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Heads of more than 128 features.  One wave per query row: scores over all keys,
// wavefront-reduction softmax, then the context row.  Dynamic LDS: 4 waves x (L + dh) floats.
// With key_lengths, sequence b attends to its first key_lengths[b] positions only (clamped to 1..L).
__global__ __launch_bounds__(256) void attention_f32_wide_head_kernel(const float *qkv, float *ctx, int L,
                                                                      int m, int dh, const int32_t *key_lengths)
{
    extern __shared__ float smem[];
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    float *prob = smem + (size_t)wave * (L + dh);
    float *qrow = prob + L;
    const int b = blockIdx.z, p = blockIdx.y;
    const int i = blockIdx.x * 4 + wave;
    if (i >= L) return;  // whole wave leaves; no workgroup barrier below
    int Lk = L;
    if (key_lengths) Lk = min(max(key_lengths[b], 1), L);
    const int64_t ld = (int64_t)m * 3 * dh;
    const float *base = qkv + (int64_t)b * L * ld + (int64_t)p * 3 * dh;
    const float *q = base + (int64_t)i * ld;
    for (int e = lane; e < dh; e += 64) qrow[e] = q[e];
    __builtin_amdgcn_wave_barrier();
    const float scale = 1.0f / sqrtf((float)dh);
    float mx = -INFINITY;
    for (int j = lane; j < Lk; j += 64) {
        const float *k = base + (int64_t)j * ld + dh;
        float s = 0.f;
        for (int e = 0; e < dh; ++e) s = fmaf(qrow[e], k[e], s);
        s *= scale;
        prob[j] = s;
        mx = fmaxf(mx, s);
    }
    mx = wave_max(mx);
    float den = 0.f;
    for (int j = lane; j < Lk; j += 64) {
        float e = expf(prob[j] - mx);
        prob[j] = e;
        den += e;
    }
    den = wave_sum(den);
    const float inv = 1.0f / den;
    __builtin_amdgcn_wave_barrier();
    float *out = ctx + ((int64_t)b * L + i) * ((int64_t)m * dh) + (int64_t)p * dh;
    for (int e = lane; e < dh; e += 64) {
        float acc = 0.f;
        for (int j = 0; j < Lk; ++j) acc = fmaf(prob[j], base[(int64_t)j * ld + 2 * dh + e], acc);
        out[e] = acc * inv;
    }
}

// Tile shapes: {waves along M, 16-row blocks per wave, 16-column blocks per wave}
struct TileShape {
    int wm, rm, cn;
    int bm() const { return 16 * wm * rm; }
    int bn() const { return 16 * (4 / wm) * cn; }
};
constexpr TileShape kTiles[] = {{4, 2, 6}, {4, 2, 4}, {4, 1, 6}, {4, 1, 4}, {4, 1, 3}, {4, 1, 2}, {2, 1, 2}, {2, 1, 1}, {1, 1, 1}};
constexpr int kTileCount = (int)(sizeof(kTiles) / sizeof(kTiles[0]));

struct F32Choice {
    int tile, splits;
};

// Shape and K splits with the least estimated time: the busiest compute unit's matrix work at 256
// flops per clock (25 and 10 % more for a unit that holds one or two workgroups: their waves wait at the
// same barriers), a start-up and epilogue of 3000 clocks per round of workgroups, and for the K-split
// kinds the float32 planes that LayerNorm has to read (about 2 KB per clock over the chip).  At BERT-base,
// 8 x 128 tokens, the choices are within 3 % of the best of all shapes and 1, 2, 4 splits.
F32Choice choose_f32(const GemmProblem &p, int N, int K, int max_splits)
{
    const bool n_split = (p.kind == GEMM_QKV || p.kind == GEMM_FFN_UP);
    const int k_tiles = (K + BK - 1) / BK;
    F32Choice best = {0, 1};
    double best_t = 0.0;
    bool any = false;
    for (int c = 0; c < kTileCount; ++c) {
        const int bm = kTiles[c].bm(), bn = kTiles[c].bn();
        const int64_t tiles = (int64_t)((N + bn - 1) / bn) * ((p.T + bm - 1) / bm);
        for (int s = 1; s <= (n_split ? 1 : max_splits) && s * 4 <= k_tiles + 3; ++s) {
            const int64_t per_cu = (tiles * s + kComputeUnits - 1) / kComputeUnits;
            const double work = (double)bm * bn * ((K + s - 1) / s) * 2.0 / 256.0;
            double t = (double)per_cu * work * (per_cu == 1 ? 1.25 : per_cu == 2 ? 1.1 : 1.0) + 3000.0 * (per_cu < 2 ? 1 : (per_cu + 1) / 2);
            if (!n_split) t += (double)s * p.T * N * 8.0 / 2048.0;
            if (!any || t < best_t * 0.999) {
                any = true;
                best_t = t;
                best = {c, s};
            }
        }
    }
    return best;
}

template <int KIND, int WM, int RM, int CN>
hipError_t launch_tile(const F32Args &a, bool vec, int splits, hipStream_t stream)
{
    constexpr int BM = 16 * WM * RM, BN = 16 * (4 / WM) * CN;
    const int64_t tiles = (int64_t)((a.N + BN - 1) / BN) * ((a.T + BM - 1) / BM);
    if (tiles > 0x7FFFFFF0) return hipErrorInvalidValue;
    const dim3 grid((uint32_t)((tiles + 7) / 8 * 8), (uint32_t)splits);
    if (vec) launch((gemm_f32_kernel<KIND, WM, RM, CN, true>), grid, dim3(256), 0, stream, a);
    else launch((gemm_f32_kernel<KIND, WM, RM, CN, false>), grid, dim3(256), 0, stream, a);
    return hipGetLastError();
}

template <int KIND>
hipError_t launch_f32_kind(const F32Args &a, int tile, bool vec, int splits, hipStream_t stream)
{
    switch (tile) {
    case 0: return launch_tile<KIND, 4, 2, 6>(a, vec, splits, stream);
    case 1: return launch_tile<KIND, 4, 2, 4>(a, vec, splits, stream);
    case 2: return launch_tile<KIND, 4, 1, 6>(a, vec, splits, stream);
    case 3: return launch_tile<KIND, 4, 1, 4>(a, vec, splits, stream);
    case 4: return launch_tile<KIND, 4, 1, 3>(a, vec, splits, stream);
    case 5: return launch_tile<KIND, 4, 1, 2>(a, vec, splits, stream);
    case 6: return launch_tile<KIND, 2, 1, 2>(a, vec, splits, stream);
    case 7: return launch_tile<KIND, 2, 1, 1>(a, vec, splits, stream);
    default: return launch_tile<KIND, 1, 1, 1>(a, vec, splits, stream);
    }
}

template <bool VEC>
void launch_attention_blocks(const float *qkv, void *ctx, int B, int L, int m, int dh, const int32_t *key_lengths,
                             hipStream_t stream)
{
    const AttentionPieces pieces = attention_pieces(B, m, (L + 63) / 64);
    const dim3 grid(8 * pieces.per_xcd);
#define STI_ATT_F32(DB) \
    launch((attention_f32_mfma_kernel<DB, VEC, false>), grid, dim3(256), 0, stream, qkv, ctx, L, m, dh, key_lengths, pieces)
    if (dh <= 32) STI_ATT_F32(2);
    else if (dh <= 64) STI_ATT_F32(4);
    else if (dh <= 96) STI_ATT_F32(6);
    else STI_ATT_F32(8);
#undef STI_ATT_F32
}

}  // namespace

hipError_t launch_gemm_f32(const GemmProblem &p, const GemmBlocks &blocks, int max_splits, int *splits_used, hipStream_t stream)
{
    const bool n_split = (p.kind == GEMM_QKV || p.kind == GEMM_FFN_UP);
    const int N = n_split ? p.n_blocks * p.block_rows : p.block_rows;
    const int K = n_split ? p.block_cols : p.n_blocks * p.block_cols;
    *splits_used = 1;
    if (p.T <= 0 || N <= 0 || K <= 0) return hipSuccess;
    F32Args a;
    a.A = (const float *)p.A; a.w0 = (const float *)blocks.b[0].w;
    a.w_stride = p.n_blocks > 1 ? (const float *)blocks.b[1].w - (const float *)blocks.b[0].w : 0;
    a.C = (float *)p.C; a.partial_stride = p.partial_stride;
    a.bias0 = p.bias0; a.bias1 = p.bias1; a.bias2 = p.bias2;
    a.T = p.T; a.N = N; a.K = K; a.lda = p.lda; a.ldc = p.ldc;
    a.block_rows = p.block_rows; a.block_cols = p.block_cols; a.d_head = p.d_head;
    a.m_fastest = p.T <= N;
    for (int b = 0; b < p.n_blocks; ++b) {
        if ((const float *)blocks.b[b].w != a.w0 + b * a.w_stride) return hipErrorInvalidValue;
        a.shard[b] = (int8_t)blocks.b[b].shard;
    }
    auto al16 = [](const void *q) { return ((uintptr_t)q & 15) == 0; };
    const bool vec = p.lda % 4 == 0 && p.ldc % 4 == 0 && p.block_cols % 4 == 0 && p.block_rows % 4 == 0 && p.d_head % 4 == 0 &&
                     a.w_stride % 4 == 0 && p.partial_stride % 4 == 0 && al16(a.A) && al16(a.w0) && al16(a.C) &&
                     (n_split || p.block_cols % BK == 0) &&
                     (uint64_t)(p.n_blocks - 1) * a.w_stride + (uint64_t)p.block_rows * p.block_cols < (1u << 30) &&
                     (uint64_t)p.lda * 128 < (1u << 30);   // (at most 128 rows per tile)
    const F32Choice ch = choose_f32(p, N, K, max_splits < 1 ? 1 : max_splits);
    *splits_used = ch.splits;
    switch (p.kind) {
    case GEMM_QKV: return launch_f32_kind<GEMM_QKV>(a, ch.tile, vec, ch.splits, stream);
    case GEMM_FFN_UP: return launch_f32_kind<GEMM_FFN_UP>(a, ch.tile, vec, ch.splits, stream);
    default: return launch_f32_kind<GEMM_OUT>(a, ch.tile, vec, ch.splits, stream);   // O and FFN2: the same kernel
    }
}

hipError_t launch_attention_f32(const float *qkv, void *ctx, bool planes, int B, int L, int m, int dh,
                                const int32_t *key_lengths, hipStream_t stream)
{
    if (B <= 0 || L <= 0 || m <= 0) return hipSuccess;
    if (planes) {
        if (dh != 64 || ((uintptr_t)qkv & 15) || ((uintptr_t)ctx & 15)) return hipErrorInvalidValue;
        const AttentionPieces pieces = attention_pieces(B, m, (L + 63) / 64);
        launch((attention_f32_mfma_kernel<4, true, true>), dim3(8 * pieces.per_xcd), dim3(256), 0, stream, qkv, ctx, L, m, dh, key_lengths, pieces);
        return hipGetLastError();
    }
    if (dh <= 128) {
        const bool vec = dh % 4 == 0 && ((uintptr_t)qkv & 15) == 0 && ((uintptr_t)ctx & 15) == 0;
        if (vec) launch_attention_blocks<true>(qkv, ctx, B, L, m, dh, key_lengths, stream);
        else launch_attention_blocks<false>(qkv, ctx, B, L, m, dh, key_lengths, stream);
        return hipGetLastError();
    }
    dim3 grid((L + 3) / 4, m, B);
    size_t lds = (size_t)4 * (L + dh) * sizeof(float);
    launch(attention_f32_wide_head_kernel, grid, dim3(256), lds, stream, qkv, (float *)ctx, L, m, dh, key_lengths);
    return hipGetLastError();
}

}  // namespace sti
