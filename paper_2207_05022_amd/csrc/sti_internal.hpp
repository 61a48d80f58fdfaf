// Internal declarations shared by the translation units of libsti (HIP, gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>
#include "sti.h"

namespace sti {

constexpr int kMaxShardsPerLayer = 64;   // sti_dims.n_heads upper bound
constexpr int kInlineShards = 64;        // shard tables up to this size travel as kernel arguments

// Device-side view of one shard version.
struct ShardDesc {
    const void *data;       // packed stream or float32 values
    const float *codebook;  // 2^bits centroids (unused for 32)
    int32_t bits;           // 2..6 or 32
    int32_t tag;            // original shard id inside its layer
    const uint32_t *outlier_pos;   // distinct offsets of the outlier dictionary
    const float *outlier_val;      // their original float32 weights
    uint32_t n_outliers;
    uint32_t pad;
};

struct InlineShardTable {
    ShardDesc d[kInlineShards];
};

// A shard table among a kernel's arguments, with room for as few descriptors as the call has: the host copies an argument list
// to the device (64 descriptors are 3 KiB: 12 shards of BERT-base with dictionaries to float32 7.2 us, 6.9 with room for 16; 2 shards 5.4 and
// 5.1 with room for four).
template <int N>
struct TableInline {
    ShardDesc d[N];
    __device__ inline ShardDesc get(uint32_t s) const { return d[s]; }
};
template <typename Go>
inline auto with_inline_table(const InlineShardTable &table, int n_shards, Go go)   // go(a TableInline of 4, 16 or 64)
{
    auto cut = [&](auto &t) {
        for (size_t i = 0; i < sizeof(t.d) / sizeof(t.d[0]); ++i) t.d[i] = table.d[i];
        return go(t);
    };
    if (n_shards <= 4) {
        TableInline<4> t;
        return cut(t);
    }
    if (n_shards <= 16) {
        TableInline<16> t;
        return cut(t);
    }
    TableInline<kInlineShards> t;
    return cut(t);
}

// ---- decode.hip -----------------------------------------------------------
// Decode n_shards shards of n weights each into out[s*n + j] and put the bookkept outliers back:
// out[s*n + pos] = round_to(out_dtype, val) for every entry of every shard's outlier dictionary
// (offsets >= n are ignored).  `table` is a device pointer to n_shards descriptors, or NULL to use
// `inline_table`; max_outliers: the largest dictionary.
hipError_t launch_decode(const ShardDesc *table, const InlineShardTable *inline_table, int n_shards,
                         uint32_t max_outliers, uint64_t n, void *out, sti_dtype out_dtype, hipStream_t stream);

// Copy `count` descriptors from pinned host memory to the device; `done` is recorded by the launch itself.
hipError_t launch_fetch_table(const ShardDesc *pinned, ShardDesc *table, size_t count, hipStream_t stream, hipEvent_t done);

// Put outliers back into the fragment-tiled binary16 working buffer written by launch_decode_tiled.
hipError_t launch_patch_outliers_tiled(const InlineShardTable &table, int n_shards,
                                       uint32_t max_outliers, int d, int dh, int f, void *out,
                                       hipStream_t stream);

// Decode n_shards shards of a layer (d, dh, f geometry) into the fragment-tiled binary16
// working buffer out[n_shards][Wsh] used by the matrix-core GEMM (see weight_loader.hpp).
hipError_t launch_decode_tiled(const InlineShardTable &table, int n_shards, int d, int dh, int f,
                               void *out, hipStream_t stream);
// Same with the table in device memory (any number of shards, e.g. every layer of a model in
// one launch): shard p is written at out + p * Wsh * 2 bytes.
hipError_t launch_decode_tiled_table(const ShardDesc *device_table, int n_shards, int d, int dh, int f,
                                     void *out, hipStream_t stream);

// ---- layer kernels ----------------------------------------------------------
// The four projections of a layer over its present shards, seen as GEMMs
// C[T x N] = A[T x K] * W^T whose weight operand is cut into per-shard blocks:
enum GemmKind : int32_t {
    GEMM_QKV = 0,       // blocks along N: block p = [3*dh x d] (Wq,Wk,Wv of shard p); + bq|bk|bv
    GEMM_FFN_UP = 1,    // blocks along N: block p = [f x d];   + b1 slice, then GELU
    GEMM_OUT = 2,       // blocks along K: block p = [d x dh];  + bo[n] + residual
    GEMM_FFN_DOWN = 3,  // blocks along K: block p = [d x f];   + b2[n] + residual
    // wide-tile kernel only, sequences of exactly 128 tokens: a 128 x 384 tile is the Q, K, V of
    // two heads of one sequence, and the workgroup goes on to those heads' attention; C is then
    // the context buffer [T x m*dh] and no Q/K/V buffer is written
    GEMM_QKV_ATTN = 4
};

// How an activation matrix lies in memory: row by row, or (few tokens) in the cells of the weights' working
// buffer: 32 rows x 64 columns = 4 KiB, [row block][column cell][fragment q][lane][8 values], lane l of
// fragment q owning row l % 32, columns (l / 32) * 32 + q * 8 .. + 8 - a matrix-core operand of a wave is one contiguous
// 1 KiB load.  Buffers of tiled matrices hold whole row blocks; what lies in rows past the last token is arbitrary.
// LAYOUT_ROWS_F32: row by row in float32 (the caller's x, read by the few-token Q/K/V projection and as a residual).
enum ActLayout : int32_t { LAYOUT_ROWS = 0, LAYOUT_TILED = 1, LAYOUT_ROWS_F32 = 2 };

// element offset of (row, col) in a tiled matrix of `cells` 64-column cells per row block
__host__ __device__ inline int64_t tiled_offset(int row, int col, int cells)
{
    return ((int64_t)(row >> 5) * cells + (col >> 6)) * 2048 + ((col & 31) >> 3) * 512 + (((col >> 5) & 1) * 32 + (row & 31)) * 8 +
           (col & 7);
}

// Quotients by a divisor that is the same for a whole launch: 5 instructions instead of the 35 dependent ones of a division of two
// scalars.  q = c * floor(2^32 / d) / 2^32 is the quotient or one less, for every c.
__host__ __device__ inline uint32_t reciprocal(uint32_t d) { return d <= 1 ? 0xFFFFFFFFu : (uint32_t)(((uint64_t)1 << 32) / d); }
__device__ inline int quotient(int c, int d, uint32_t recip)   // c >= 0, d > 0
{
    const uint32_t q = __umulhi((uint32_t)c, recip);
    return (int)(q + ((uint32_t)c - q * (uint32_t)d >= (uint32_t)d ? 1u : 0u));
}

// between a wave's own writes to LDS and its reads of what other lanes wrote
__device__ inline void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Workgroups are handed to the eight XCDs in turn.  Pieces of work that lie behind each other in memory go to one XCD, an eighth of
// them to each, so that what they share is fetched into one L2.
__host__ __device__ inline int pieces_per_xcd(int pieces) { return (pieces + 7) >> 3; }
__device__ inline int piece_of_block(int block, int per_xcd) { return (block & 7) * per_xcd + (block >> 3); }   // (of 8 per_xcd blocks; some past the last piece)

// The (sequence, head, block of queries) triples of an attention launch in that order: the blocks of a head share its keys and values, the
// heads of a sequence the cache lines of its rows.  24 x 384 tokens, 16 heads: 32.8 -> 29.9 us; 11 x 93, 10 heads 5.6 -> 5.35; float32
// 8 x 128, 12 heads 12.8 -> 12.3.
struct AttentionPieces {
    int total, per_xcd;
    uint32_t heads_recip, blocks_recip;
};
inline AttentionPieces attention_pieces(int sequences, int heads, int blocks)
{
    const int total = sequences * heads * blocks;   // (below 2^31: at most 2^24 tokens, 64 heads, blocks of 64 queries or more)
    return {total, pieces_per_xcd(total), reciprocal((uint32_t)heads), reciprocal((uint32_t)blocks)};
}
struct AttentionPiece {
    int sequence, head, block;
    bool none;
};
__device__ inline AttentionPiece attention_piece(const AttentionPieces &p, int heads, int blocks)
{
    const int i = piece_of_block(blockIdx.x, p.per_xcd), pair = quotient(i, blocks, p.blocks_recip);
    AttentionPiece out;
    out.none = i >= p.total;
    out.block = i - pair * blocks;
    out.sequence = quotient(pair, heads, p.heads_recip);
    out.head = pair - out.sequence * heads;
    return out;
}

// two values rounded to binary16 (nearest even) in one dword: one conversion instruction
__device__ inline uint32_t f16_pair_bits(float lo, float hi)
{
    typedef _Float16 half2v __attribute__((ext_vector_type(2)));
    const half2v h = {(_Float16)lo, (_Float16)hi};
    return __builtin_bit_cast(uint32_t, h);
}

struct CellMap {       // cells of the fragment-tiled working buffer (weight_loader.hpp): what a launch's cells have in common
    int d, dh, f, per_shard;
    uint32_t recip_shard, recip_d, recip_dh, recip_f;
};
inline CellMap cell_map(int d, int dh, int f)
{
    const int per_shard = (3 * dh / 32) * (d / 64) + (d / 32) * (dh / 64) + (f / 32) * (d / 64) + (d / 32) * (f / 64);
    return CellMap{d, dh, f, per_shard, reciprocal(per_shard), reciprocal(d / 64), reciprocal(dh / 64), reciprocal(f / 64)};
}

struct GemmBlock {
    const void *w;          // start of the block's weights: float32 values, or a k-bit stream
    const float *codebook;  // centroids when bits <= 6
    int32_t bits;           // 2..6, 32; 17 = fragment-tiled binary16 working buffer
    int32_t shard;          // original shard id (selects the bias slice)
};

struct GemmBlocks {
    GemmBlock b[kMaxShardsPerLayer];
};

struct GemmProblem {
    GemmKind kind;
    int32_t T;          // rows of A and C
    int32_t n_blocks;   // present shards
    int32_t block_rows; // N-split: rows per block; K-split: N (= d)
    int32_t block_cols; // N-split: K (= d);        K-split: columns per block
    int32_t d_head;     // QKV bias selection
    const void *A;      // [T x K], row stride lda elements
    int32_t lda;
    void *C;            // [T x N], row stride ldc elements
    int32_t ldc;
    const float *bias0, *bias1, *bias2;  // QKV: bq,bk,bv; FFN_UP: b1; OUT/FFN_DOWN: bias[N]
    const void *resid;  // OUT/FFN_DOWN: [T x N] residual, row stride ldr
    int32_t ldr;
    ActLayout a_layout, c_layout;   // few-token kernel; tiled: lda / ldc are the matrices' widths
    // wide-tile kernel, OUT/FFN_DOWN only: with k_splits > 0 the K range is split over
    // that many workgroups per tile, C is float32 and takes the raw sums of split s
    // at C + s * partial_stride (bias and residual are left to launch_layernorm)
    int32_t k_splits;
    int64_t partial_stride;
    const int32_t *key_lengths;   // GEMM_QKV_ATTN: real positions per sequence (device, may be null)
    // wide-tile kernel, GEMM_QKV and GEMM_QKV_ATTN: workgroups beyond those of the tiles (next_workgroups of them, on compute
    // units the tiles leave idle) decompress next_shards shards - the next layer's - from the device
    // table next_table into the working buffer next_out; next_workgroups == 0: nothing of the kind
    const ShardDesc *next_table;
    void *next_out;
    int32_t next_shards, next_workgroups, next_ffn_per_shard;
    // wide-tile kernel, GEMM_OUT and GEMM_FFN_DOWN: with next_outliers > 0 workgroups beyond those of the tiles put the outlier dictionaries
    // of the next_shards shards of next_table (at most next_outliers entries each) into next_out
    int32_t next_outliers;
    CellMap next_cells;   // (filled in by the launch)
};

// float32 path (layer_f32.hip): A and C are float32; weights are float32 blocks at a constant distance.
// QKV / FFN_UP apply bias (and GELU); OUT / FFN_DOWN leave raw sums for launch_layernorm, those of
// K split s at C + s * partial_stride, with at most max_splits of them (the number comes back in splits_used).
hipError_t launch_gemm_f32(const GemmProblem &p, const GemmBlocks &blocks, int max_splits, int *splits_used,
                           hipStream_t stream);
// The same on the bfloat16 matrix cores (gemm_f32_split.hip): A and the weight blocks are planes of three bfloat16 values per
// float32, in cells; FFN_UP leaves planes, the others as above.
hipError_t launch_gemm_split(const GemmProblem &p, const GemmBlocks &blocks, int max_splits, int *splits_used, hipStream_t stream);
int gemm_split_k_splits(const GemmProblem &p, int max_splits);   // those of O or FFN2
// rows [T x d] of float32 -> planes; a layer's shards (no outlier dictionaries) -> planes, Q, K, V and O shard by shard, or (ffn) all of
// FFN2 and then all of FFN1
hipError_t launch_split_rows(const float *src, void *dst, int T, int d, hipStream_t stream);
hipError_t launch_decode_split(const InlineShardTable &table, int n_shards, int d, int dh, int f, bool ffn, void *out, hipStream_t stream);
// qkv [T x m*3*dh] float32 (per shard: q, k, v each dh wide) -> ctx [T x m*dh] float32, or planes (heads of 64 features).
// key_lengths (device, [B], may be null): keys of sequence b beyond key_lengths[b] take no part.
hipError_t launch_attention_f32(const float *qkv, void *ctx, bool planes, int B, int L, int m, int dh,
                                const int32_t *key_lengths, hipStream_t stream);

// binary16 MFMA path (gemm_wide.hip, attention_mfma.hip): A and C are binary16.  QKV / FFN_UP
// apply bias (and GELU); OUT / FFN_DOWN add bias[N] and the binary16 residual, leaving the
// LayerNorm to launch_layernorm_f16in (or, with k_splits > 0, leave float32 sums that
// launch_layernorm completes, like the few-token variant below).  Every block is a cell array
// of the fragment-tiled binary16 working buffer (bits == kTiledBits).
hipError_t launch_gemm_wide(const GemmProblem &p, const GemmBlocks &blocks, hipStream_t stream);
bool gemm_wide_out_carries(GemmProblem out, GemmProblem down, int entries);
bool gemm_wide_supported(const GemmProblem &p, const GemmBlocks &blocks);
// the same in tiles of 64 row_blocks x 256 (gemm_large.hip): N a multiple of 64, at least two K tiles, no next_* work, on top of what
// launch_gemm_wide has checked
hipError_t launch_gemm_large(const GemmProblem &p, const GemmBlocks &blocks, int N, int row_blocks, hipStream_t stream);
// whether the Q/K/V projection of B sequences of L tokens over m heads should go out as GEMM_QKV_ATTN
bool gemm_wide_fuses_attention(int B, int L, int m, int dh);
// workgroups a Q/K/V launch (GEMM_QKV or GEMM_QKV_ATTN; kind, T, n_blocks, block_rows, block_cols, next_shards,
// next_ffn_per_shard set) should give to the next layer's decompression: one per compute unit that its tiles leave idle
// (0: none to spare, or a launch of its own costs less; grouped: that launch takes several layers)
int gemm_wide_spare_workgroups(const GemmProblem &p, bool grouped);
// k_splits of this problem, and the most planes that can be for T tokens and N output columns (workspace sizing; rows in binary16
// lie in a plane, too)
int gemm_wide_sum_planes(const GemmProblem &p);
int gemm_wide_max_sum_planes(int64_t T, int N);
// the most tokens for which it can be `splits` (2 or 4)
int64_t gemm_wide_most_tokens(int splits, int N);
// ctx_layout: how the context is left behind (the Q/K/V matrix is row-major)
hipError_t launch_attention_mfma(const void *qkv, void *ctx, ActLayout ctx_layout, int B, int L, int m, int dh,
                                 const int32_t *key_lengths, hipStream_t stream);
// Few tokens: Q/K/V and context tiled, the V cells transposed as the few-token GEMM leaves them
// (attention_few.hip; one sequence, or sequences of a multiple of 32 tokens).
bool attention_few_supported(int B, int L);
hipError_t launch_attention_few(const void *qkv, void *ctx, int B, int L, int m, int dh, const int32_t *key_lengths,
                                hipStream_t stream);

// The same attention and the output projection (p: GEMM_OUT) in one launch: partial sums in planes of a group of heads each.
// How many planes, or 0 where the two by themselves are faster or the forms do not fit.
constexpr int kFewOutKeys = 64;
int attention_out_few_planes(const GemmProblem &p, int B, int L);   // (0 beyond kFewOutKeys keys)
hipError_t launch_attention_out_few(const GemmProblem &p, const GemmBlocks &blocks, const void *qkv, int B, int L, const int32_t *key_lengths,
                                    int64_t partial_stride, hipStream_t stream);

// Few-token variant of the MFMA GEMM (gemm_few.hip): T <= kFewMaxTokens, split-K inside the
// workgroup and, for the K-split kinds, across `k_splits` workgroups that write float32
// partial sums at C + s * partial_stride (to be added by launch_layernorm).
constexpr int kFewMaxTokens = 1024;
constexpr int kFewMaxSplits = 8;
int few_k_splits(const GemmProblem &p);
// whether the Q/K/V projection of T tokens takes float32 rows as they are
bool few_takes_f32_rows(int T, int n_blocks, int block_rows, int d_model);
int few_max_k_splits(int k_tiles);   // the most it can be for up to so many 64-wide K tiles (workspace sizing)
hipError_t launch_gemm_few(const GemmProblem &p, const GemmBlocks &blocks, int k_splits,
                              int64_t partial_stride, hipStream_t stream);

// A launch_decode_split that goes out with a LayerNorm that leaves planes, of up to kRideFeatures features (longer rows: registers for one
// workgroup of four waves per unit): n_shards of the table, of d_model d.  Nothing that LayerNorm reads or writes lies in `out`.
constexpr int kRideFeatures = 1024;
struct SplitRide {
    const InlineShardTable *table;
    int n_shards, d_head, ffn_per_shard;
    bool ffn;
    void *out;
};

// rowops.hip
// v = sum_{s < n_partials} pre[s * partial_stride + t*d + :] + bias[:] + resid[t][:]  (n_partials may be 0);
// y[t][:] = LayerNorm(v) * g + b.  pre float32; bias (float32 [d]) and resid (binary16, or float32
// with resid_f32, [T x d]) may be NULL; y of out_dtype.  A residual or a binary16 y may be tiled.  planes (may be NULL;
// float32 y and resid_f32, rows read with wide loads): y as planes of bfloat16 values, too.
bool layernorm_reads_wide(const float *pre, int64_t partial_stride, const float *bias, const void *resid, const void *y, const float *g, const float *b, int d);
hipError_t launch_layernorm(const float *pre, int n_partials, int64_t partial_stride,
                            const float *bias, const void *resid, bool resid_f32, ActLayout resid_layout, void *y,
                            sti_dtype out_dtype, ActLayout y_layout,
                            const float *g, const float *b, int T, int d, float eps,
                            hipStream_t stream, void *planes = nullptr, const SplitRide *ride = nullptr);
// y[t][:] = LayerNorm(pre_f16[t][:]) * g + b for rows that already hold sum + bias + residual.
hipError_t launch_layernorm_f16in(const void *pre_f16, void *y, sti_dtype out_dtype, const float *g,
                                  const float *b, int T, int d, float eps, hipStream_t stream);
// rows of src -> binary16, tiled (d a multiple of 64)
hipError_t launch_tile_rows(const void *src, sti_dtype src_dtype, void *dst, int T, int d, hipStream_t stream);
// elementwise conversion between activation types
hipError_t launch_convert(const void *src, sti_dtype src_dtype, void *dst, sti_dtype dst_dtype,
                          uint64_t n, hipStream_t stream);

// Kernel launches of the entry points go through launch(): while per-kernel timing is on
// (sti_profile_begin), the launch carries the two events the profiler handed out, which then
// hold the dispatch's own begin and end time stamps -- the same stamps a kernel trace reads.
// (Two events recorded around a launch read about 2.5 us more than the kernel lasts: the
// record-to-start latency.)  Without timing it is an ordinary launch.
struct LaunchEvents {
    hipEvent_t start = nullptr, stop = nullptr;
};
LaunchEvents take_launch_events();   // api.hip; nulls unless a timed launch is pending on this thread

template <typename T>
struct SameType {
    typedef T type;
};
// (the launch call itself: the triple chevrons pass grid and stream through a thread's stack of configurations first, 0.35 us of
// 3.6 with 400 bytes of arguments)
template <typename... P>
inline void launch_arguments(void (*kernel)(P...), dim3 grid, dim3 block, size_t lds_bytes, hipStream_t stream, typename SameType<P>::type... values)
{
    void *arguments[] = {(void *)&values...};
    (void)hipLaunchKernel((const void *)kernel, grid, block, arguments, lds_bytes, stream);   // (its error is the caller's hipGetLastError)
}

template <typename... P, typename... A>
inline void launch(void (*kernel)(P...), dim3 grid, dim3 block, size_t lds_bytes, hipStream_t stream, A... args)
{
    const LaunchEvents ev = take_launch_events();
    if (ev.start)
        hipExtLaunchKernelGGL(kernel, grid, block, (uint32_t)lds_bytes, stream, ev.start, ev.stop, 0, (P)args...);
    else
        launch_arguments(kernel, grid, block, lds_bytes, stream, P(args)...);
}

}  // namespace sti
