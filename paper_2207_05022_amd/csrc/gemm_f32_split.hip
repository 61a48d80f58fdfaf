// float32 layers on the bfloat16 matrix cores (any number of tokens that fills them; d_model and neurons multiples of 64,
// heads of 64 features): every float32 operand is the sum of three bfloat16 values,
//   x = h + m + l,   h = bf16(x), m = bf16(x - h), l = bf16(x - h - m)
// (three times 8 significant bits, rounded to nearest: all 24 of x, unless l is too small for a bfloat16), and a product keeps six terms,
//   h h' + (h m' + m h') + (m m' + h l' + l h');
// the other three come to 2^-23 of it at worst, over random pairs 2^-24.2 at most and 2^-27.4 in the 2-norm.  Six products at 16 times the rate of the float32 matrix instruction.  (The method is that of G. Henry, P. T. P.
// Tang and A. Heinecke, "Leveraging the bfloat16 artificial intelligence datatype for higher-precision computations", 2019.)
//
// Products of bfloat16 values are exact in float32; the terms are added smallest first.  Measured against float64, random operands, K = 768
// and 3072: 3.9e-7 and 8.6e-7 (2-norm, relative); v_mfma_f32_16x16x4_f32 5.0e-7 and 1.01e-6, which is what one rounding per
// product gives.
//
// What bounds it: BERT-base, 8 x 128 tokens, us per launch, float32 against these matrix instructions: Q/K/V 34 / 27, O 13 / 12, FFN1 43 / 33,
// FFN2 43 / 31; the K loops run at 1.1 to 1.4 PFLOP/s of bfloat16 products, near what the chip's clock under this load allows, around them
// start-up and epilogue of the one tile per compute unit.  Planes cost the two LayerNorms 6 us more, and as much again since they carry the
// decompression beside them, which took two launches of 7 us: a layer 178 -> 148 -> 136 us.  Error of 12 layers against float64 (2-norm, relative): 1.28e-6 -> 0.92e-6.
//
// Layout: an operand matrix is cut into cells of 32 rows x 64 columns as the binary16 working buffer is (weight_loader.hpp), a cell
// holding its three planes one after the other: [row block][column cell][plane][fragment q][lane][8 values], 12 KiB.
#include <algorithm>
#include "sti_internal.hpp"
#include "weight_loader.hpp"
#include "split_planes.hpp"
#include "split_decode.hpp"

namespace sti {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int BK = 64;
constexpr int kComputeUnits = 256;

struct SplitTail {   // what only the end of a workgroup needs
    void *C;
    const float *bias0, *bias1, *bias2;
    int64_t partial_stride;
    int32_t ldc;
    int8_t shard[kMaxShardsPerLayer];   // original shard id of block b (selects the bias slice)
};

// A workgroup of four waves owns 128 rows x (32 CN) columns: a wave 32 rows, whose fragments go straight into its registers, all
// columns, whose weights the four waves share through LDS.  Of K tile kt + 1 everything is requested before tile kt is
// multiplied: 24 CN matrix instructions of 32 clocks per tile and wave, 12 + 3 CN requests of 1 KiB, and of k-step s + 1 the
// weight fragments are read while step s is multiplied.
// grid: x = tiles (an XCD takes a contiguous range, row tiles fastest), y = K split.
template <int KIND, int CN>
__global__ __launch_bounds__(256, 1) void gemm_split_kernel(
    const void *A, const void *W, int32_t T, int32_t nkt, int32_t N, int32_t tiles_per_block /* strips (N split) or K tiles */,
    uint32_t block_recip, uint32_t row_tiles_recip, int32_t block_stride_kib, int32_t kt_per_split, SplitTail tail)
{
    constexpr bool n_split = (KIND == GEMM_QKV || KIND == GEMM_FFN_UP);
    __shared__ u32x4 Ws[2][CN][12][64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 5, lr = lane & 31;
    const int m_tiles = (T + 127) >> 7, n_tiles = (N + 32 * CN - 1) / (32 * CN);
    const int total = m_tiles * n_tiles, per_xcd = (total + 7) >> 3;
    const int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per_xcd || tile >= total) return;
    const int tile_n = quotient(tile, m_tiles, row_tiles_recip), tile_m = tile - tile_n * m_tiles;
    const int kt0 = blockIdx.y * kt_per_split, kt1 = min(kt0 + kt_per_split, nkt);
    const int rb = min(tile_m * 4 + wave, (T - 1) >> 5);   // (row blocks past the last one: that one again, never stored)
    const char *a_base = (const char *)A + (int64_t)rb * nkt * 12288;   // (uniform)
    const uint32_t lane16 = lane * 16, tid16 = tid * 16;

    // strip j of this tile, K tile kt (strips past the last one: that one again, never stored)
    auto w_cell = [&](int j, int kt) -> const char * {
        const int strip = min(tile_n * CN + j, (N >> 5) - 1);
        int blk, cell;
        if (n_split) {
            blk = quotient(strip, tiles_per_block, block_recip);
            cell = (strip - blk * tiles_per_block) * nkt + kt;
        } else {
            blk = quotient(kt, tiles_per_block, block_recip);
            cell = strip * tiles_per_block + kt - blk * tiles_per_block;
        }
        return (const char *)W + (int64_t)blk * block_stride_kib * 1024 + (int64_t)cell * 12288;
    };
    struct Stage {
        u32x4 a[3][4], w[CN][3];
    };
    // requests lo .. hi - 1 of a tile's 3 CN + 12
    auto request = [&](int kt, Stage &st, int lo, int hi) {
#pragma unroll
        for (int j = 0; j < CN; ++j)
#pragma unroll
            for (int r = 0; r < 3; ++r)
                if (j * 3 + r >= lo && j * 3 + r < hi) st.w[j][r] = *(const u32x4 *)(w_cell(j, kt) + (tid16 + r * 4096u));
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
            for (int s = 0; s < 4; ++s)
                if (3 * CN + p * 4 + s >= lo && 3 * CN + p * 4 + s < hi)
                    st.a[p][s] = *(const u32x4 *)(a_base + (int64_t)kt * 12288 + (lane16 + (p * 4 + s) * 1024u));
    };
    auto put = [&](int buf, const Stage &st) {
#pragma unroll
        for (int j = 0; j < CN; ++j)
#pragma unroll
            for (int r = 0; r < 3; ++r) (&Ws[buf][j][0][0])[tid + 256 * r] = st.w[j][r];
    };
    float16v acc[CN];
#pragma unroll
    for (int j = 0; j < CN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
    struct Frags {
        u32x4 w[CN][3];
    };
    auto read = [&](int buf, int s, Frags &f) {
#pragma unroll
        for (int j = 0; j < CN; ++j)
#pragma unroll
            for (int p = 0; p < 3; ++p) f.w[j][p] = Ws[buf][j][p * 4 + s][lane];
    };
    auto multiply = [&](const Frags &f, const u32x4 (&a)[3][4], int s) {
        constexpr int term[6][2] = {{2, 0}, {0, 2}, {1, 1}, {1, 0}, {0, 1}, {0, 0}};   // planes of W and A, smallest first
#pragma unroll
        for (int t = 0; t < 6; ++t)
#pragma unroll
            for (int j = 0; j < CN; ++j)
                acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, f.w[j][term[t][0]]),
                                                                __builtin_bit_cast(bf16x8, a[term[t][1]][s]), acc[j], 0, 0, 0);
    };
    // Two matrix instructions, one read out of LDS, now and then a request or a write into LDS: with all of a tile's requests in front of its
    // products the four waves first stood 1300 clocks at the address unit.
    auto interleave = [&](auto writes) {
#pragma unroll
        for (int i = 0; i < 3 * CN; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);                                 // matrix
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                                 // LDS read
            if constexpr (decltype(writes)::value) __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);   // LDS write
            __builtin_amdgcn_sched_group_barrier(0x020, (CN + 4 + 3 * CN - 1) / (3 * CN), 0);  // request
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    constexpr int REQ = 3 * CN + 12;
    Frags f0, f1;
    auto step = [&](int kt, Stage &cur, Stage &next, Stage &after) {
        const int buf = (kt - kt0) & 1, ahead = min(kt + 2, kt1 - 1);   // (past the end: the last tile again, never used)
        read(buf, 1, f1);
        request(ahead, after, 0, REQ / 3);
        multiply(f0, cur.a, 0);
        interleave(std::false_type{});
        read(buf, 2, f0);
        request(ahead, after, REQ / 3, 2 * REQ / 3);
        multiply(f1, cur.a, 1);
        interleave(std::false_type{});
        read(buf, 3, f1);
        put(buf ^ 1, next);
        request(ahead, after, 2 * REQ / 3, REQ);
        multiply(f0, cur.a, 2);
        interleave(std::true_type{});
        __syncthreads();
        read(buf ^ 1, 0, f0);
        multiply(f1, cur.a, 3);
        interleave(std::false_type{});
    };
    if (kt0 < kt1) {
        Stage s0, s1, s2;
        request(kt0, s0, 0, REQ);
        request(min(kt0 + 1, kt1 - 1), s1, 0, REQ);
        put(0, s0);
        __syncthreads();
        read(0, 0, f0);
        // (whole rounds of three, the rest behind them: steps that can be skipped make the loop copy its sums and wait at its
        // top for requests of the step before)
        int kt = kt0;
        for (; kt + 2 < kt1; kt += 3) {
            step(kt, s0, s1, s2);
            step(kt + 1, s1, s2, s0);
            step(kt + 2, s2, s0, s1);
        }
        if (kt < kt1) step(kt, s0, s1, s2);
        if (kt + 1 < kt1) step(kt + 1, s1, s2, s0);
    }

    // ---- epilogue: block j: token lr, columns v4 * 8 + g * 4 .. + 4 ----
    const int t = (tile_m * 4 + wave) * 32 + lr;
    if ((tile_m * 4 + wave) * 32 >= T) return;
#pragma unroll
    for (int j = 0; j < CN; ++j) {
        const int strip = tile_n * CN + j;
        if (strip * 32 >= N) continue;
        const float *bp = nullptr;
        if constexpr (n_split) {
            const int blk = quotient(strip, tiles_per_block, block_recip), r = (strip - blk * tiles_per_block) * 32;
            const int shard = tail.shard[blk];
            if constexpr (KIND == GEMM_QKV) {
                const int which = r >> 6;
                bp = (which == 0 ? tail.bias0 : which == 1 ? tail.bias1 : tail.bias2) + shard * 64 + r - which * 64;
            } else {
                bp = tail.bias0 + shard * tiles_per_block * 32 + r;
            }
        }
#pragma unroll
        for (int v4 = 0; v4 < 4; ++v4) {
            const int n = strip * 32 + v4 * 8 + g * 4;
            f32x4 x = {acc[j][v4 * 4], acc[j][v4 * 4 + 1], acc[j][v4 * 4 + 2], acc[j][v4 * 4 + 3]};
            if constexpr (n_split) x += *(const f32x4_any *)(bp + v4 * 8 + g * 4);
            if constexpr (KIND == GEMM_FFN_UP) {
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = gelu_f32(x[e]);
                store_planes4((uint16_t *)tail.C, t, n, tail.ldc >> 6, x);   // (rows past T: inside the last row block)
            } else if (t < T) {
                *(f32x4 *)((float *)tail.C + (n_split ? 0 : (int64_t)blockIdx.y * tail.partial_stride) + (int64_t)t * tail.ldc + n) = x;
            }
        }
    }
}

// Rows of float32 to planes: a thread takes 8 columns, consecutive threads the rows of a 32-row block first, so that a wave's
// stores are whole fragments.
__global__ __launch_bounds__(256) void split_rows_kernel(const float *src, uint16_t *dst, int T, int d)
{
    const int chunks = d >> 3, i = blockIdx.x * 256 + threadIdx.x;
    const int row = i / (32 * chunks) * 32 + i % 32, c = i / 32 % chunks * 8;
    if (row >= T) return;
    const f32x4 *p = (const f32x4 *)(src + (int64_t)row * d + c);
    store_planes4(dst, row, c, d >> 6, p[0]);
    store_planes4(dst, row, c + 4, d >> 6, p[1]);
}

// A layer's shards to planes, one wave per cell
template <typename Table>
__global__ __launch_bounds__(256) void decode_split_kernel(SplitDecodeJob job, Table tab)
{
    __shared__ u32x2 lut[4][kLutEntries];
    decode_split_block(job, tab, blockIdx.x, lut);
}

struct SplitChoice {
    int cn, splits;
};

// Columns of a tile and K splits with the least estimated time in clocks: 768 per K tile and 32 columns at 0.8 of the matrix
// rate, start-up and epilogue of a round of workgroups, and for the K-split kinds the planes LayerNorm adds (about 2 KB a clock).
SplitChoice choose_split(const GemmProblem &p, int N, int nkt, int max_splits)
{
    const bool n_split = (p.kind == GEMM_QKV || p.kind == GEMM_FFN_UP);
    SplitChoice best = {1, 1};
    double best_t = 0.0;
    for (int cn = 4; cn >= 1; --cn)
        for (int s = 1; s <= (n_split ? 1 : max_splits) && s <= nkt; ++s) {
            const int64_t tiles = (int64_t)((p.T + 127) / 128) * ((N + 32 * cn - 1) / (32 * cn)) * s;
            const int64_t rounds = (tiles + kComputeUnits - 1) / kComputeUnits;
            double t = (double)rounds * (((nkt + s - 1) / s) * (cn * 768.0 / 0.8 + 250.0) + 6000.0);
            if (!n_split) t += (double)s * p.T * N * 8.0 / 2048.0;
            if (best_t == 0.0 || t < best_t * 0.999) {
                best_t = t;
                best = {cn, s};
            }
        }
    return best;
}

template <int KIND, int CN>
hipError_t launch_cn(const GemmProblem &p, const void *W, int64_t block_stride, int N, int nkt, int splits, const SplitTail &tail, hipStream_t stream)
{
    constexpr bool n_split = (KIND == GEMM_QKV || KIND == GEMM_FFN_UP);
    const int m_tiles = (p.T + 127) / 128, total = m_tiles * ((N + 32 * CN - 1) / (32 * CN));
    const int per_block = n_split ? p.block_rows / 32 : p.block_cols / BK;
    launch((gemm_split_kernel<KIND, CN>), dim3((total + 7) / 8 * 8, splits), dim3(256), 0, stream, p.A, W, p.T, nkt, N, per_block,
           reciprocal(per_block), reciprocal(m_tiles), (int32_t)(block_stride / 1024), (nkt + splits - 1) / splits, tail);
    return hipGetLastError();
}

template <int KIND>
hipError_t launch_split_kind(const GemmProblem &p, const void *W, int64_t block_stride, int N, int nkt, SplitChoice ch, const SplitTail &tail, hipStream_t stream)
{
    switch (ch.cn) {
    case 1: return launch_cn<KIND, 1>(p, W, block_stride, N, nkt, ch.splits, tail, stream);
    case 2: return launch_cn<KIND, 2>(p, W, block_stride, N, nkt, ch.splits, tail, stream);
    case 3: return launch_cn<KIND, 3>(p, W, block_stride, N, nkt, ch.splits, tail, stream);
    default: return launch_cn<KIND, 4>(p, W, block_stride, N, nkt, ch.splits, tail, stream);
    }
}

}  // namespace

int gemm_split_k_splits(const GemmProblem &p, int max_splits)
{
    return choose_split(p, p.block_rows, p.n_blocks * p.block_cols / BK, max_splits < 1 ? 1 : max_splits).splits;
}

hipError_t launch_gemm_split(const GemmProblem &p, const GemmBlocks &blocks, int max_splits, int *splits_used, hipStream_t stream)
{
    const bool n_split = (p.kind == GEMM_QKV || p.kind == GEMM_FFN_UP);
    const int N = n_split ? p.n_blocks * p.block_rows : p.block_rows;
    const int K = n_split ? p.block_cols : p.n_blocks * p.block_cols;
    *splits_used = 1;
    if (p.T <= 0 || N <= 0 || K <= 0) return hipSuccess;
    const int64_t stride = p.n_blocks > 1 ? (const uint8_t *)blocks.b[1].w - (const uint8_t *)blocks.b[0].w : 0;
    if (p.block_rows % 32 || p.block_cols % BK || p.ldc % 4 || stride % 1024 || stride < 0 || stride / 1024 > INT32_MAX ||
        (p.kind == GEMM_FFN_UP && p.ldc % 64) || (p.kind == GEMM_QKV && (p.d_head != 64 || p.block_rows != 192)))
        return hipErrorInvalidValue;
    SplitTail tail = {p.C, p.bias0, p.bias1, p.bias2, p.partial_stride, p.ldc, {}};
    for (int b = 0; b < p.n_blocks; ++b) {
        if ((const uint8_t *)blocks.b[b].w != (const uint8_t *)blocks.b[0].w + b * stride) return hipErrorInvalidValue;
        tail.shard[b] = (int8_t)blocks.b[b].shard;
    }
    const SplitChoice ch = choose_split(p, N, K / BK, max_splits < 1 ? 1 : max_splits);
    *splits_used = ch.splits;
    switch (p.kind) {
    case GEMM_QKV: return launch_split_kind<GEMM_QKV>(p, blocks.b[0].w, stride, N, K / BK, ch, tail, stream);
    case GEMM_FFN_UP: return launch_split_kind<GEMM_FFN_UP>(p, blocks.b[0].w, stride, N, K / BK, ch, tail, stream);
    default: return launch_split_kind<GEMM_OUT>(p, blocks.b[0].w, stride, N, K / BK, ch, tail, stream);   // O and FFN2
    }
}

hipError_t launch_split_rows(const float *src, void *dst, int T, int d, hipStream_t stream)
{
    if (T <= 0 || d <= 0) return hipSuccess;
    if (d % 64) return hipErrorInvalidValue;
    const int64_t threads = (int64_t)((T + 31) / 32) * 32 * (d / 8);
    if (threads > 0x7FFFFF00) return hipErrorInvalidValue;
    launch(split_rows_kernel, dim3((uint32_t)((threads + 255) / 256)), dim3(256), 0, stream, src, (uint16_t *)dst, T, d);
    return hipGetLastError();
}

hipError_t launch_decode_split(const InlineShardTable &table, int n_shards, int d, int dh, int f, bool ffn, void *out, hipStream_t stream)
{
    SplitDecodeJob job;
    if (!split_decode_job(n_shards, d, dh, f, ffn, out, &job)) return hipErrorInvalidValue;
    if (job.cells == 0) return hipSuccess;
    with_inline_table(table, n_shards, [&](auto t) {
        launch((decode_split_kernel<decltype(t)>), dim3((uint32_t)((job.cells + 3) / 4)), dim3(256), 0, stream, job, t);
    });
    return hipGetLastError();
}

}  // namespace sti
