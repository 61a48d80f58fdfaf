// Projections for few tokens: the regime of single-sequence inference, where every weight is used once
// or a few times and a layer is a chain of short dependent launches (Section "Submodel execution" runs one
// input at a time).
//
// A workgroup owns one 32-column strip of the output, one or two 32-row blocks of tokens and a range of
// K; its waves take one 64-wide K tile each (split-K inside the workgroup), decode the tile's weights in
// registers and add their products through LDS.  The O and FFN2 products are also split over
// workgroups, which leave float32 partial sums that the LayerNorm kernel adds in a fixed order.
//
// What bounds it: latency.  Clocks inside a workgroup (Q/K/V of BERT-base, 128 tokens; about 2100 to a us), version before
// this one and now: 2560 / 750 until the descriptor is there, 3900 / 2650 until weights and activations are (both
// through the L1 at 64 bytes per clock: 150 KB per compute unit), 5040 / 4020 decoded, 7770 / 6090 all waves done, 8800 / 7200
// stored.  Hence:
//   - no integer division and nothing that only some bitwidths need in front of the first requests (a third of the time);
//   - activations come fragment-tiled (tiled_offset below, the layout of the weights' working buffer): a fragment load is
//     1 KiB contiguous, 16 clocks of the address unit; 32 rows of a row-major matrix take 64;
//   - one switch on the bitwidth per tile with the whole way from request to fragment inside each case: a switch
//     for the loads alone made the compiler wait for them where the cases join;
//   - one tile per wave wherever the tiles allow (4 to 16 waves), so that nothing is requested late;
//   - all waves take part in the sum, four columns of one token per thread, and store what they have
//     added; a wave's store instruction covers whole 512-byte runs of the tiled output.
// Per layer: BERT-base 128 tokens, 9 of 12 shards 32.0 -> 29.0 us; d_model 1024, 12 of 16 shards, 256 tokens 48 -> 41 us.
#include <string.h>
#include <type_traits>
#include "sti_internal.hpp"
#include "weight_loader.hpp"
#include "few_tiles.hpp"

namespace sti {
namespace {

constexpr int BK = 64;

__device__ inline float gelu_fast(float z)
{
    // erf by Abramowitz & Stegun 7.1.26 (|error| < 1.5e-7); results are rounded to binary16
    const float x = fabsf(z) * 0.70710678118654752440f;
    const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, x, 1.0f));
    float poly = fmaf(1.061405429f, t, -1.453152027f);
    poly = fmaf(poly, t, 1.421413741f);
    poly = fmaf(poly, t, -0.284496736f);
    poly = fmaf(poly, t, 0.254829592f);
    const float e = __builtin_amdgcn_exp2f(-x * x * 1.44269504088896340736f);
    const float erf_abs = 1.0f - poly * t * e;
    return 0.5f * z * (1.0f + (z < 0.f ? -erf_abs : erf_abs));
}

constexpr int kF32Row = BK + 8;      // LDS row of a float32 tile on its way to fragments (halves)

template <int RA>
struct FewWave {                     // one wave's part of LDS
    union {
        f32x4 red[RA][4][64];        // its partial sums
        _Float16 tile[32][kF32Row];
    };
};
template <int NW, int RA>
struct FewSmem {
    FewWave<RA> wave[NW];
    uint16_t lut[NW][kLutEntries];
};

// A float32 tile on its way to fragments: whole 256-byte rows are requested (16 lanes each), rounded, and
// turned into the fragment layout through LDS.
struct FloatTile {
    f32x4 v[8];
};
__device__ inline void request_floats(const float *src, uint32_t ld, int lane, FloatTile &t)   // src: uniform
{
    const uint32_t at = (uint32_t)(lane >> 4) * ld + (lane & 15) * 4;
#pragma unroll
    for (int j = 0; j < 8; ++j) t.v[j] = *(const f32x4 *)((const char *)src + (at + 4 * j * ld) * 4);   // (32 rows of at most 2^16 floats)
}
__device__ inline void float_fragments(const FloatTile &t, _Float16 (*tile)[kF32Row], int lane, half8 (&f)[4])
{
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const half4 h = {(_Float16)t.v[j].x, (_Float16)t.v[j].y, (_Float16)t.v[j].z, (_Float16)t.v[j].w};
        *(half4 *)&tile[4 * j + (lane >> 4)][(lane & 15) * 4] = h;
    }
    wave_lds_fence();
#pragma unroll
    for (int q = 0; q < 4; ++q) f[q] = *(const half8 *)&tile[lane & 31][(lane >> 5) * 32 + q * 8];
    wave_lds_fence();
}

struct FewTail {   // what only the end of a workgroup needs
    void *C;
    const float *bias0, *bias1, *bias2;
    int32_t ldc, c_layout;
};

constexpr int kDHead = 64;   // features of a head on this path

// grid: x = 32-column strip (KIND QKV, FFN_UP: of a weight block), y = weight block (QKV, FFN_UP) or K split (OUT, which
// stands for FFN_DOWN too), z = group of RA row blocks.  ONE: no wave has more than one K tile.  Otherwise the waves
// walk K side by side (a cache line of packed weights holds 3 to 8 tiles of a row).
// AF32: A is the caller's float32 rows, rounded on arrival.
template <int KIND, int NW, int RA, int NB, bool ONE, bool AF32>
__global__ __launch_bounds__(NW * 64) void gemm_few_kernel(
    // leading scalar arguments arrive preloaded in scalar registers: what the first loads of a workgroup depend on, with
    // every quotient already formed.  (A division of two scalars is 35 dependent instructions of 4 to 8 clocks.)
    const void *hot_A, int32_t hot_T, int32_t hot_lda, int32_t hot_nkt, int32_t hot_block_rows, int32_t hot_block_cols,
    int32_t hot_kt_per_split, uint32_t hot_kblock_magic, int32_t a_rows, int64_t partial_stride,
    FewTail tail, FewBlocks<NB> blocks)
{
    static_assert(!AF32 || (KIND == GEMM_QKV && ONE), "the first projection, one tile per wave");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    FewSmem<NW, RA> &sm = *reinterpret_cast<FewSmem<NW, RA> *>(smem_raw);
    constexpr bool n_split = (KIND == GEMM_QKV || KIND == GEMM_FFN_UP);
    const int nkt = hot_nkt;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 5, lr = lane & 31;
    const int row = blockIdx.x * 32;            // first row of the strip in its weight block(s)
    const int nblk = n_split ? blockIdx.y : 0, split = n_split ? 0 : blockIdx.y;
    const int nw = nblk * hot_block_rows + row; // first output column of the strip
    const int rb0 = blockIdx.z * RA;            // first 32-row block
    const int kt_begin = split * hot_kt_per_split, kt_end = n_split ? nkt : min(kt_begin + hot_kt_per_split, nkt);

    float16v acc[RA];
#pragma unroll
    for (int i = 0; i < RA; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;
    // this thread finishes columns n .. n + 3 (of every row block it comes to)
    const int v4 = wave & 3;
    const int n = nw + v4 * 8 + g * 4;
    f32x4 bias = {0.f, 0.f, 0.f, 0.f};
    const int part = KIND == GEMM_QKV ? row / kDHead : 0;   // Q/K/V: 0, 1, 2 (the strip lies inside one)
    auto request_bias = [&](int shard) {
        if constexpr (!n_split) return;
        const float *bp = KIND == GEMM_QKV ? (part == 0 ? tail.bias0 : part == 1 ? tail.bias1 : tail.bias2) + shard * kDHead + (row - part * kDHead)
                                           : tail.bias0 + shard * hot_block_rows + row;
        bias = *(const f32x4_any *)(bp + v4 * 8 + g * 4);
    };

    typedef u32x4 Operand[4];
    // fragments of row block rb0 + i, K tile kt (row blocks past the last one: the last one again, rows past the last token: the
    // last one; never stored)
    auto request_a = [&](int l, int kt, int i, Operand &a) {
        const int rb = min(rb0 + i, (hot_T - 1) >> 5);
        uint32_t at = (uint32_t)(rb * nkt + kt) * 4096u + l * 16, step = 1024;   // (below 2^32: rows and columns of this route)
        if (a_rows) {
            at = ((uint32_t)min(rb * 32 + (l & 31), hot_T - 1) * (uint32_t)hot_lda + kt * BK + (l >> 5) * 32) * 2;
            step = 16;
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) a[s] = *(const u32x4 *)((const char *)hot_A + (at + s * step));
    };
    // the weight is the first operand: a lane's accumulators are runs of four output columns of token lr
    auto multiply = [&](const half8 (&f)[4], const Operand (&a)[RA]) {
#pragma unroll
        for (int i = 0; i < RA; ++i)
#pragma unroll
            for (int s = 0; s < 4; ++s)
                acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(f[s], __builtin_bit_cast(half8, a[i][s]), acc[i], 0, 0, 0);
    };
    // count K tiles of weight block blk: k, k + NW, ...
    auto tiles = [&](int k, int count, int blk, bool first) {
        // (what follows is invariant, but not to be formed for every bitwidth before the first request)
        int l = lane;
        if constexpr (!ONE) asm volatile("" : "+v"(l));
        const GemmBlock desc = blocks.b[blk];
        const int ktb = n_split ? k : k - blk * (hot_block_cols / BK);
        Operand a[RA];
        FloatTile fa[AF32 ? RA : 1];
        // (row blocks past the last one: the last one again; the last 32 rows at most begin before the first of their block)
        auto request_rows = [&](int i) {
            const int r0 = min((rb0 + i) * 32, (hot_T - 1) & ~31);
#pragma unroll
            for (int j = 0; j < 8; ++j)
                fa[AF32 ? i : 0].v[j] = *(const f32x4 *)((const float *)hot_A + (uint32_t)min(r0 + 4 * j + (l >> 4), hot_T - 1) * (uint32_t)hot_lda + k * BK + (l & 15) * 4);
        };
        if constexpr (AF32) request_rows(0);
        else request_a(l, k, 0, a[0]);
        __builtin_amdgcn_sched_barrier(0);
        // behind the first request for weights: the other row blocks, and what the epilogue adds
        auto request_rest = [&]() {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 1; i < RA; ++i) {
                if constexpr (AF32) request_rows(i);
                else request_a(l, k, i, a[i]);
            }
            if (first) request_bias(desc.shard);
            __builtin_amdgcn_sched_barrier(0);
        };
        const int64_t start = (int64_t)row * hot_block_cols + ktb * BK;                    // of the tile in its block, uniform
        const uint32_t lane_elem = (uint32_t)(l & 31) * hot_block_cols + (l >> 5) * 32;     // of the lane in the tile
        auto rows_to_operands = [&]() {
            if constexpr (AF32) {
#pragma unroll
                for (int i = 0; i < RA; ++i) {
                    half8 f[4];
                    float_fragments(fa[i], sm.wave[wave].tile, l, f);
#pragma unroll
                    for (int s = 0; s < 4; ++s) a[i][s] = __builtin_bit_cast(u32x4, f[s]);
                }
            }
        };
        // One tile after the other: the next one's weights and this one's activations are on their way while fragments(raw, f)
        // turns its weights into operands
        auto walk = [&](auto request, auto fragments, auto &raw) {
            auto step = [&](int j, int cur) {
                if (j > 0) {
#pragma unroll
                    for (int i = 0; i < RA; ++i) request_a(l, k + j * NW, i, a[i]);
                }
                if (j + 1 < count) request(j + 1, raw[cur ^ 1]);
                __builtin_amdgcn_sched_barrier(0);
                half8 f[4];
                fragments(raw[cur], f);
                multiply(f, a);
            };
            if constexpr (ONE || !n_split) {
                half8 f[4];
                fragments(raw[0], f);
                rows_to_operands();
                multiply(f, a);
            } else {
                for (int j = 0; j < count; j += 2) {
                    step(j, 0);
                    if (j + 1 < count) step(j + 1, 1);
                }
            }
        };
        auto packed = [&](auto width) {
            constexpr int BITS = decltype(width)::value;
            uint16_t *lut = sm.lut[wave];
            const uint8_t *base = (const uint8_t *)desc.w + (start >> 5) * (BITS * 4);
            const uint32_t at = (lane_elem >> 5) * (BITS * 4);
            Raw raw[ONE || !n_split ? 1 : 2];
            auto request = [&](int j, Raw &r) { r = load_raw<BITS>(base + (at + j * (NW * 2 * BITS * 4))); };
            const float centroid = desc.codebook[l & ((1 << BITS) - 1)];
            request(0, raw[0]);
            request_rest();
            wave_lds_fence();                    // (the table of the wave's previous tiles is read)
            lut[l] = (uint16_t)f16_bits(centroid);
            wave_lds_fence();
            walk(request, [&](const Raw &r, half8 (&f)[4]) { decode_raw<BITS>(r, lut, f); }, raw);
        };
        switch (desc.bits) {
        case 2: packed(std::integral_constant<int, 2>{}); break;
        case 3: packed(std::integral_constant<int, 3>{}); break;
        case 4: packed(std::integral_constant<int, 4>{}); break;
        case 5: packed(std::integral_constant<int, 5>{}); break;
        case 6: packed(std::integral_constant<int, 6>{}); break;
        case kTiledBits: {
            const uint8_t *base = (const uint8_t *)desc.w + tiled_cell_offset(row >> 5, ktb, hot_block_cols);
            Raw raw[ONE || !n_split ? 1 : 2];
            auto request = [&](int j, Raw &r) { r = load_tiled(base + j * (NW * 4096), l); };
            request(0, raw[0]);
            request_rest();
            walk(request, [&](const Raw &r, half8 (&f)[4]) { decode_raw<16>(r, nullptr, f); }, raw);
            break;
        }
        default: {
            const float *base = (const float *)desc.w + start;
            for (int j = 0; j < count; ++j) {
                FloatTile t;
                request_floats(base + j * (NW * BK), hot_block_cols, l, t);
                if (j == 0) {
                    request_rest();
                } else {
#pragma unroll
                    for (int i = 0; i < RA; ++i) request_a(l, k + j * NW, i, a[i]);
                }
                half8 f[4];
                float_fragments(t, sm.wave[wave].tile, l, f);
                rows_to_operands();
                multiply(f, a);
                if constexpr (ONE || !n_split) break;
            }
        }
        }
    };
    auto block_of = [&](int kt) { return n_split ? nblk : hot_kblock_magic == 0 ? kt : (int)__umulhi((uint32_t)kt, hot_kblock_magic); };
    const int kt0 = kt_begin + wave;            // this wave's tiles: kt0, kt0 + NW, ...
    if (kt0 >= kt_end) {
        if constexpr (n_split) request_bias(blocks.b[nblk].shard);   // (a wave without a K tile finishes columns, too)
    } else if constexpr (ONE) {
        tiles(kt0, 1, block_of(kt0), true);
    } else if constexpr (n_split) {
        tiles(kt0, (kt_end - kt0 + NW - 1) / NW, nblk, true);
    } else {
        for (int kt = kt0; kt < kt_end; kt += NW) tiles(kt, 1, block_of(kt), false);
    }

#pragma unroll
    for (int i = 0; i < RA; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            sm.wave[wave].red[i][q][lane] = f32x4{acc[i][4 * q], acc[i][4 * q + 1], acc[i][4 * q + 2], acc[i][4 * q + 3]};
    __syncthreads();
    for (int i = wave >> 2; i < RA; i += NW / 4) {
        const int t = (rb0 + i) * 32 + lr;      // token
        f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < NW; w += 4) {
            f32x4 q[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) q[j] = sm.wave[w + j].red[i][v4][lane];
            s += (q[0] + q[1]) + (q[2] + q[3]);
        }
        if (!n_split) {
            if (t < hot_T) *(f32x4 *)((float *)tail.C + split * partial_stride + (int64_t)t * tail.ldc + n) = s;
            continue;
        }
        s += bias;
        if constexpr (KIND == GEMM_FFN_UP) {
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] = gelu_fast(s[e]);
        }
        half4 h = {(_Float16)s[0], (_Float16)s[1], (_Float16)s[2], (_Float16)s[3]};
        _Float16 *C = (_Float16 *)tail.C;
        if (tail.c_layout == LAYOUT_ROWS) {
            if (t < hot_T) *(half4 *)(C + (int64_t)t * tail.ldc + n) = h;
        } else if ((rb0 + i) * 32 >= hot_T) {
            continue;                           // (a row block past the last one)
        } else if (KIND == GEMM_QKV && part == 2) {
            // V transposed for the attention's second product (attention_few.hip)
            _Float16 *cell = C + ((int64_t)(rb0 + i) * (tail.ldc >> 6) + (n >> 6)) * 2048;
            const int half = (n >> 5) & 1, s2 = lr >> 4, gk = (lr >> 2) & 1, pos = ((lr >> 3) & 1) * 4 + (lr & 3);
#pragma unroll
            for (int e = 0; e < 4; ++e) cell[(half * 2 + s2) * 512 + (gk * 32 + (n & 31) + e) * 8 + pos] = h[e];
        } else {
            *(half4 *)(C + tiled_offset(t, n, tail.ldc >> 6)) = h;
        }
    }
}

template <int KIND, int NW, int RA, int NB, bool ONE, bool AF32 = false>
hipError_t launch_few(const GemmProblem &p, const GemmBlocks &blocks, int k_splits, int64_t partial_stride, hipStream_t stream)
{
    constexpr bool n_split = (KIND == GEMM_QKV || KIND == GEMM_FFN_UP);
    const int row_blocks = (p.T + 31) / 32, nkt = (n_split ? p.block_cols : p.n_blocks * p.block_cols) / BK;
    const dim3 grid(p.block_rows / 32, n_split ? p.n_blocks : k_splits, (row_blocks + RA - 1) / RA);
    constexpr size_t lds = sizeof(FewSmem<NW, RA>);
    static_assert(lds <= 160 * 1024, "one workgroup's partial sums");
    // more than 64 KiB of dynamic LDS needs an explicit opt-in: once per instantiation, and safe
    // when several host threads make their first call together
    static const hipError_t attr_status =
        hipFuncSetAttribute((const void *)gemm_few_kernel<KIND, NW, RA, NB, ONE, AF32>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (attr_status != hipSuccess) return attr_status;
    FewBlocks<NB> table;
    memcpy(table.b, blocks.b, sizeof(table.b));
    const int per_split = (nkt + k_splits - 1) / k_splits;
    const FewTail tail = {p.C, p.bias0, p.bias1, p.bias2, p.ldc, (int32_t)p.c_layout};
    // kt / tiles = the upper half of kt * ceil(2^32 / tiles) while kt * tiles < 2^32 (kt < 2^16, tiles <= 2^10); 0: one tile per block
    const uint32_t tiles = p.block_cols / BK, magic = tiles == 1 ? 0u : (uint32_t)((((uint64_t)1 << 32) + tiles - 1) / tiles);
    launch((gemm_few_kernel<KIND, NW, RA, NB, ONE, AF32>), grid, dim3(NW * 64), lds, stream, p.A, p.T, p.lda, nkt, p.block_rows, p.block_cols,
           per_split, magic, (int32_t)(p.a_layout == LAYOUT_ROWS), partial_stride, tail, table);
    return hipGetLastError();
}

template <int KIND, int NW, int RA, bool ONE>
hipError_t launch_blocks(const GemmProblem &p, const GemmBlocks &blocks, int k_splits, int64_t partial_stride, hipStream_t stream)
{
    if (p.a_layout == LAYOUT_ROWS_F32) {
        if constexpr (KIND == GEMM_QKV && ONE && NW <= 12) return launch_few<KIND, NW, RA, 16, ONE, true>(p, blocks, k_splits, partial_stride, stream);
        return hipErrorInvalidValue;
    }
    if (p.n_blocks <= 16) return launch_few<KIND, NW, RA, 16, ONE>(p, blocks, k_splits, partial_stride, stream);
    return launch_few<KIND, NW, RA, kMaxShardsPerLayer, ONE>(p, blocks, k_splits, partial_stride, stream);
}

template <int NW, int RA, bool ONE>
hipError_t launch_kind(const GemmProblem &p, const GemmBlocks &blocks, int k_splits, int64_t partial_stride, hipStream_t stream)
{
    switch (p.kind) {
    case GEMM_QKV: return launch_blocks<GEMM_QKV, NW, RA, ONE>(p, blocks, k_splits, partial_stride, stream);
    case GEMM_FFN_UP: return launch_blocks<GEMM_FFN_UP, NW, RA, ONE>(p, blocks, k_splits, partial_stride, stream);
    default: return launch_blocks<GEMM_OUT, NW, RA, ONE>(p, blocks, k_splits, partial_stride, stream);
    }
}

constexpr int kComputeUnits = 256;
constexpr int kMaxWaves = 16;
constexpr int kSharedWorkgroups = 3 * kComputeUnits;   // four-wave workgroups that the chip holds at once

inline int k_tiles(const GemmProblem &p)
{
    return ((p.kind == GEMM_QKV || p.kind == GEMM_FFN_UP) ? p.block_cols : p.n_blocks * p.block_cols) / BK;
}
inline int splits_of(int tiles, int per_split)
{
    const int s = (tiles + per_split - 1) / per_split;
    return s < 1 ? 1 : (s > kFewMaxSplits ? kFewMaxSplits : s);
}

}  // namespace

// K splits of O and FFN2: 12 K tiles each, or 16 where that saves a round of workgroups (LayerNorm adds the partial sums of
// all of them).  12 layers, us, 16 against 12 tiles: BERT-base 320 tokens 471 / 461, 512 tokens 526 / 513, 640 tokens (two
// rounds with 12) 570 / 594; d_model 1024 256 tokens (24 layers) 1003 / 979, 384 tokens (two rounds) 599 / 636.
int few_k_splits(const GemmProblem &p)
{
    if (p.kind == GEMM_QKV || p.kind == GEMM_FFN_UP) return 1;
    const int fine = splits_of(k_tiles(p), 12), coarse = splits_of(k_tiles(p), 16);
    const int64_t per_split = (int64_t)(p.block_rows / 32) * ((p.T + 63) / 64);
    auto rounds = [&](int splits) { return (per_split * splits + kSharedWorkgroups - 1) / kSharedWorkgroups; };
    return rounds(coarse) < rounds(fine) ? coarse : fine;
}

int few_max_k_splits(int tiles) { return splits_of(tiles, 12); }

namespace {

struct FewShape {
    int ra, nw;   // row blocks and waves of a workgroup
};
FewShape few_shape(int T, int strips, int k_splits, int tiles)   // tiles: of a K split
{
    // 32 rows to a workgroup where every workgroup then has a compute unit of its own (half the activations to fetch and the
    // sums to exchange per unit: BERT-base with 9 of 12 shards, 128 tokens 361 -> 354 us per 12 layers; 320 or 512 workgroups:
    // 362 to 371), else 64.  One wave per K tile while workgroups have units of their own; beyond that four waves, so that
    // three workgroups share a unit and cover each other's round trips (BERT-base, 256 tokens 442 us, 476 with eight waves).
    const int row_blocks = (T + 31) / 32;
    const int ra = row_blocks < 2 || (int64_t)strips * k_splits * row_blocks <= kComputeUnits ? 1 : 2;
    const int64_t workgroups = (int64_t)strips * k_splits * ((row_blocks + ra - 1) / ra);
    return {ra, tiles <= 4 || workgroups > kComputeUnits ? 4 : tiles <= 8 || tiles > kMaxWaves ? 8 : tiles <= 12 ? 12 : 16};
}

}  // namespace

// One tile per wave and no more than twelve waves (registers for two row blocks of float32).  The rows are twice the bytes and pass
// through LDS, but the launch that would round and tile them is on the chain: 2 us, and 2.8 on the host.
bool few_takes_f32_rows(int T, int n_blocks, int block_rows, int d_model)
{
    const FewShape sh = few_shape(T, n_blocks * block_rows / 32, 1, d_model / BK);
    return n_blocks > 0 && n_blocks <= 16 && d_model / BK <= sh.nw && sh.nw <= 12;
}

hipError_t launch_gemm_few(const GemmProblem &p, const GemmBlocks &blocks, int k_splits,
                           int64_t partial_stride, hipStream_t stream)
{
    const bool n_split = (p.kind == GEMM_QKV || p.kind == GEMM_FFN_UP);
    const int N = n_split ? p.n_blocks * p.block_rows : p.block_rows;
    if (p.T <= 0 || N <= 0) return hipSuccess;
    if (N % 32 || p.block_rows % 32 || p.block_cols % BK || p.ldc % 4 || k_splits < 1 || (p.c_layout != LAYOUT_ROWS && p.ldc % 64) ||
        (p.a_layout == LAYOUT_ROWS && p.lda % 8) || (p.a_layout == LAYOUT_ROWS_F32 && (p.lda % 4 || p.kind != GEMM_QKV)) || (p.kind == GEMM_QKV && p.d_head != kDHead))
        return hipErrorInvalidValue;
    const int tiles = (k_tiles(p) + k_splits - 1) / k_splits;
    const FewShape sh = few_shape(p.T, N / 32, k_splits, tiles);
    const int nw = sh.nw, ra = sh.ra;
#define STI_FEW(NW, RA, ONE) case NW * 4 + RA * 2 + ONE: return launch_kind<NW, RA, ONE>(p, blocks, k_splits, partial_stride, stream)
    switch (nw * 4 + ra * 2 + (tiles <= nw)) {
    STI_FEW(4, 1, true); STI_FEW(4, 2, true); STI_FEW(4, 1, false); STI_FEW(4, 2, false);
    STI_FEW(8, 1, true); STI_FEW(8, 2, true); STI_FEW(8, 1, false); STI_FEW(8, 2, false);
    STI_FEW(12, 1, true); STI_FEW(12, 2, true);
    STI_FEW(16, 1, true); STI_FEW(16, 2, true);
    }
#undef STI_FEW
    return hipErrorInvalidValue;
}

}  // namespace sti
