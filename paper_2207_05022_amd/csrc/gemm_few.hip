// Projections for few tokens: the regime of single-sequence inference, where every weight is used once
// or a few times and a layer is a chain of short dependent launches (Section "Submodel execution" runs one
// input at a time).
//
// A workgroup owns one 32-column strip of the output, one or two 32-row blocks of tokens and a range of
// K; its waves take one 64-wide K tile each (split-K inside the workgroup), decode the tile's weights in
// registers and add their products through LDS.  The O and FFN2 products are also split over
// workgroups, which leave float32 partial sums that the LayerNorm kernel adds in a fixed order.
//
// What bounds it: latency.  Of 7.0 us inside a workgroup of the version this replaces (Q/K/V of BERT-base,
// 128 tokens) 3.7 us went by until the weights had arrived and 1.5 us each in the products and in
// the epilogue.  Hence:
//   - activations come fragment-tiled (tiled_offset below, the layout of the weights' working buffer): a fragment load is
//     1 KiB contiguous, 16 clocks of the address unit; 32 rows of a row-major matrix take 64;
//   - one switch on the bitwidth per tile with the whole way from request to fragment inside each case: a switch
//     for the loads alone made the compiler wait for them where the cases join;
//   - one tile per wave wherever the tiles allow (4 to 12 waves), so that nothing is requested late;
//   - all waves take part in the sum, four columns of one token per thread, and store what they have
//     added; a wave's store instruction covers whole 512-byte runs of the tiled output.
#include <string.h>
#include "sti_internal.hpp"
#include "weight_loader.hpp"

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

typedef _Float16 half4 __attribute__((ext_vector_type(4)));

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

__device__ inline void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int BITS>
__device__ inline void packed_fragments(const uint8_t *src, const float *codebook, uint16_t *lut, int lane, half8 (&f)[4])
{
    const float centroid = codebook[lane & ((1 << BITS) - 1)];
    const Raw raw = load_raw<BITS>(src);
    lut[lane] = (uint16_t)f16_bits(centroid);
    wave_lds_fence();
    decode_raw<BITS>(raw, lut, f);
}

// Fragments of a float32 tile: whole 256-byte rows are requested (16 lanes each), rounded, and
// turned into the fragment layout through LDS.
__device__ inline void float_fragments(const float *src, int64_t ld, _Float16 (*tile)[kF32Row], int lane, half8 (&f)[4])
{
    f32x4 v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = *(const f32x4 *)(src + (int64_t)(4 * j + (lane >> 4)) * ld + (lane & 15) * 4);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const half4 h = {(_Float16)v[j].x, (_Float16)v[j].y, (_Float16)v[j].z, (_Float16)v[j].w};
        *(half4 *)&tile[4 * j + (lane >> 4)][(lane & 15) * 4] = h;
    }
    wave_lds_fence();
#pragma unroll
    for (int q = 0; q < 4; ++q) f[q] = *(const half8 *)&tile[lane & 31][(lane >> 5) * 32 + q * 8];
    wave_lds_fence();
}

// NB: room for weight blocks among the arguments (an argument list of 64 blocks costs the host 1.2 us more per launch)
template <int NB>
struct FewBlocks {
    GemmBlock b[NB];
};

// grid: x = 32-column strip, y = K split, z = group of RA row blocks
template <int NW, int RA, int NB>
__global__ __launch_bounds__(NW * 64) void gemm_few_kernel(
    // leading scalar arguments arrive preloaded in scalar registers: what the first loads of a
    // workgroup depend on (of p, only the other fields are read)
    const void *hot_A, int32_t hot_T, int32_t hot_lda, int32_t hot_n_blocks, int32_t hot_block_rows,
    int32_t hot_block_cols, int32_t hot_kind, int32_t k_splits, int32_t a_rows, int64_t partial_stride,
    GemmProblem p, FewBlocks<NB> blocks)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    FewSmem<NW, RA> &sm = *reinterpret_cast<FewSmem<NW, RA> *>(smem_raw);
    const bool n_split = (hot_kind == GEMM_QKV || hot_kind == GEMM_FFN_UP);
    const int K = n_split ? hot_block_cols : hot_n_blocks * hot_block_cols;
    const int nkt = K / BK;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 5, lr = lane & 31;
    const int nw = blockIdx.x * 32;             // first output column of the strip
    const int rb0 = blockIdx.z * RA;            // first 32-row block
    const int split = blockIdx.y;
    const int kt_begin = nkt * split / k_splits, kt_end = nkt * (split + 1) / k_splits;
    int nblk = 0, nrow0 = nw;
    if (n_split) {
        nblk = nw / hot_block_rows;
        nrow0 = nw - nblk * hot_block_rows;
    }
    const int tiles_per_kblock = hot_block_cols / BK;

    float16v acc[RA];
#pragma unroll
    for (int i = 0; i < RA; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;

    for (int kt = kt_begin + wave; kt < kt_end; kt += NW) {
        u32x4 a[RA][4];
#pragma unroll
        for (int i = 0; i < RA; ++i) {
            // (row blocks past the last one: the last one again, rows past the last token: the last one; never stored)
            const int rb = min(rb0 + i, (hot_T - 1) >> 5);
            const u32x4 *src = (const u32x4 *)hot_A + ((int64_t)rb * nkt + kt) * 256 + lane;
            if (a_rows) src = (const u32x4 *)((const _Float16 *)hot_A + (int64_t)min(rb * 32 + lr, hot_T - 1) * hot_lda + kt * BK + g * 32);
            const int step = a_rows ? 1 : 64;
#pragma unroll
            for (int s = 0; s < 4; ++s) a[i][s] = src[s * step];
        }
        const int blk = n_split ? nblk : kt / tiles_per_kblock;
        const int ktb = n_split ? kt : kt - blk * tiles_per_kblock, row = n_split ? nrow0 : nw;
        const GemmBlock desc = blocks.b[blk];
        const int bits = desc.bits;
        half8 f[4];
        const int64_t elem = (int64_t)(row + lr) * hot_block_cols + ktb * BK + g * 32;
        const uint8_t *packed = (const uint8_t *)desc.w + (elem >> 5) * (bits * 4);
        uint16_t *lut = sm.lut[wave];
        switch (bits) {
        case 2: packed_fragments<2>(packed, desc.codebook, lut, lane, f); break;
        case 3: packed_fragments<3>(packed, desc.codebook, lut, lane, f); break;
        case 4: packed_fragments<4>(packed, desc.codebook, lut, lane, f); break;
        case 5: packed_fragments<5>(packed, desc.codebook, lut, lane, f); break;
        case 6: packed_fragments<6>(packed, desc.codebook, lut, lane, f); break;
        case kTiledBits: {
            const Raw raw = load_tiled((const uint8_t *)desc.w + tiled_cell_offset(row >> 5, ktb, hot_block_cols), lane);
            decode_raw<16>(raw, nullptr, f);
            break;
        }
        default:
            float_fragments((const float *)desc.w + (int64_t)row * hot_block_cols + ktb * BK, hot_block_cols, sm.wave[wave].tile, lane, f);
        }
        // the weight is the first operand: a lane's accumulators are runs of four output columns of token lr
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int i = 0; i < RA; ++i)
                acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(f[s], __builtin_bit_cast(half8, a[i][s]), acc[i], 0, 0, 0);
    }

    // ---- this thread finishes columns n .. n + 3 (of every row block it comes to) ----
    const int v4 = wave & 3;
    const int n = nw + v4 * 8 + g * 4;
    f32x4 bias = {0.f, 0.f, 0.f, 0.f};
    int part = 0;                               // Q/K/V: 0, 1, 2 (the strip lies inside one)
    if (n_split) {
        const int shard = blocks.b[nblk].shard, nrow = nrow0 + v4 * 8 + g * 4;
        if (hot_kind == GEMM_QKV) {
            part = nrow0 / p.d_head;
            const float *bp = part == 0 ? p.bias0 : (part == 1 ? p.bias1 : p.bias2);
            bias = *(const f32x4_any *)(bp + shard * p.d_head + nrow - part * p.d_head);
        } else {
            bias = *(const f32x4_any *)(p.bias0 + shard * hot_block_rows + nrow);
        }
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
            if (t < hot_T) *(f32x4 *)((float *)p.C + split * partial_stride + (int64_t)t * p.ldc + n) = s;
            continue;
        }
        s += bias;
        if (hot_kind == GEMM_FFN_UP) {
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] = gelu_fast(s[e]);
        }
        half4 h = {(_Float16)s[0], (_Float16)s[1], (_Float16)s[2], (_Float16)s[3]};
        _Float16 *C = (_Float16 *)p.C;
        if (p.c_layout == LAYOUT_ROWS) {
            if (t < hot_T) *(half4 *)(C + (int64_t)t * p.ldc + n) = h;
        } else if ((rb0 + i) * 32 >= hot_T) {
            continue;                           // (a row block past the last one)
        } else if (hot_kind == GEMM_QKV && part == 2) {
            // V transposed for the attention's second product (attention_few.hip)
            _Float16 *cell = C + ((int64_t)(rb0 + i) * (p.ldc >> 6) + (n >> 6)) * 2048;
            const int half = (n >> 5) & 1, s2 = lr >> 4, gk = (lr >> 2) & 1, pos = ((lr >> 3) & 1) * 4 + (lr & 3);
#pragma unroll
            for (int e = 0; e < 4; ++e) cell[(half * 2 + s2) * 512 + (gk * 32 + (n & 31) + e) * 8 + pos] = h[e];
        } else {
            *(half4 *)(C + tiled_offset(t, n, p.ldc >> 6)) = h;
        }
    }
}

template <int NW, int RA, int NB>
hipError_t launch_few(const GemmProblem &p, const GemmBlocks &blocks, int N, int k_splits, int64_t partial_stride, hipStream_t stream)
{
    const int row_blocks = (p.T + 31) / 32;
    const dim3 grid(N / 32, k_splits, (row_blocks + RA - 1) / RA);
    constexpr size_t lds = sizeof(FewSmem<NW, RA>);
    static_assert(lds <= 160 * 1024, "one workgroup's partial sums");
    // more than 64 KiB of dynamic LDS needs an explicit opt-in: once per instantiation, and safe
    // when several host threads make their first call together
    static const hipError_t attr_status =
        hipFuncSetAttribute((const void *)gemm_few_kernel<NW, RA, NB>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (attr_status != hipSuccess) return attr_status;
    FewBlocks<NB> table;
    memcpy(table.b, blocks.b, sizeof(table.b));
    launch((gemm_few_kernel<NW, RA, NB>), grid, dim3(NW * 64), lds, stream, p.A, p.T, p.lda, p.n_blocks, p.block_rows,
           p.block_cols, (int32_t)p.kind, k_splits, (int32_t)(p.a_layout == LAYOUT_ROWS), partial_stride, p, table);
    return hipGetLastError();
}

template <int NW, int RA>
hipError_t launch_blocks(const GemmProblem &p, const GemmBlocks &blocks, int N, int k_splits, int64_t partial_stride, hipStream_t stream)
{
    if (p.n_blocks <= 16) return launch_few<NW, RA, 16>(p, blocks, N, k_splits, partial_stride, stream);
    return launch_few<NW, RA, kMaxShardsPerLayer>(p, blocks, N, k_splits, partial_stride, stream);
}

constexpr int kComputeUnits = 256;
constexpr int kMaxWaves = 12;   // (16 waves leave a lane 128 registers: spills, FFN2 12 us instead of 5.6)

}  // namespace

// As few splits as leave every wave at most one K tile (LayerNorm adds the partial sums of all of them).
int few_k_splits(const GemmProblem &p)
{
    const bool n_split = (p.kind == GEMM_QKV || p.kind == GEMM_FFN_UP);
    if (n_split) return 1;
    const int s = (p.n_blocks * p.block_cols / BK + kMaxWaves - 1) / kMaxWaves;
    return s < 1 ? 1 : (s > kFewMaxSplits ? kFewMaxSplits : s);
}

hipError_t launch_gemm_few(const GemmProblem &p, const GemmBlocks &blocks, int k_splits,
                           int64_t partial_stride, hipStream_t stream)
{
    const bool n_split = (p.kind == GEMM_QKV || p.kind == GEMM_FFN_UP);
    const int N = n_split ? p.n_blocks * p.block_rows : p.block_rows;
    if (p.T <= 0 || N <= 0) return hipSuccess;
    if (N % 32 || p.block_rows % 32 || p.block_cols % BK || p.ldc % 4 || k_splits < 1 || (p.c_layout != LAYOUT_ROWS && p.ldc % 64) ||
        (p.a_layout == LAYOUT_ROWS && p.lda % 8))
        return hipErrorInvalidValue;
    const int tiles = ((n_split ? p.block_cols : p.n_blocks * p.block_cols) / BK + k_splits - 1) / k_splits;
    // One wave per K tile while every workgroup has a compute unit of its own.  Beyond that four waves, so
    // that four workgroups share a unit and cover each other's round trips (BERT-base, 512 tokens, per layer:
    // 46 us; 12 or 8 waves in rounds 56 - 58, 128-row tiles 50).
    const int row_blocks = (p.T + 31) / 32, ra = row_blocks < 2 ? 1 : 2;
    const int64_t workgroups = (int64_t)(N / 32) * k_splits * ((row_blocks + ra - 1) / ra);
    const int nw = tiles <= 4 || workgroups > kComputeUnits ? 4 : tiles <= 8 ? 8 : 12;
#define STI_FEW(NW, RA) case NW * 8 + RA: return launch_blocks<NW, RA>(p, blocks, N, k_splits, partial_stride, stream)
    switch (nw * 8 + ra) {
    STI_FEW(4, 1); STI_FEW(4, 2);
    STI_FEW(8, 1); STI_FEW(8, 2);
    STI_FEW(12, 1); STI_FEW(12, 2);
    }
#undef STI_FEW
    return hipErrorInvalidValue;
}

}  // namespace sti
