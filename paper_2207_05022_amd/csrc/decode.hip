// Shard decompression: k-bit dictionary indexes -> centroids (Section
// "quantization per shard"; the substitution loop of Section "Implementation").
//
// Bound by memory: 1 byte read per 2.7 to 16 bytes written.  Every wave decodes a stretch of one shard by itself:
//  - its codes come in as 16-byte loads and pass through a piece of LDS that is the wave's own, so that a lane can
//    pick up the codes of its outputs wherever they begin (loading them from memory lane by lane takes two 4-byte
//    loads per lane and 8 weights);
//  - the codebook is rounded to the output type once and kept in LDS, a copy per wave: no barrier;
//  - a lane decodes runs of 16 output bytes that lie on 16-byte boundaries of the output, whatever a shard's
//    length is, and consecutive lanes take consecutive runs: a store instruction writes one contiguous KiB.
// 2 runs per lane, stored nontemporal, loads temporal (streams that the 256 MB cache holds stay there).  Measured
// against two unaligned 4-byte nontemporal loads per 8 weights and one lane per 8 weights in every output type:
// 12 x 589824 weights float32 12.4 -> 6.1 us, binary16 5.3 -> 4.8; 1500 x 589824 (2 to 6 bits) binary16 451 -> 346
// (6.4 TB/s), float32 with raw shards 1530 -> 746; 60 x 300001 float32 48 -> 15.  4 runs per lane: 376 and 835 us,
// 1 run: 527 and 1003; a workgroup's codes staged together behind one barrier: 391 for binary16.
#include <type_traits>
#include "sti_internal.hpp"
#include "weight_loader.hpp"

namespace sti {
namespace {

// pointers that come out of a shard table: without the address space they would be loaded through flat
// instructions, whose waits also cover the LDS
#define STI_GLOBAL __attribute__((address_space(1)))
#define STI_STORE(v, p) __builtin_nontemporal_store((v), (p))
constexpr int kThreads = 512;
// Dictionaries of outliers: up to this many workgroups and entries per shard, each workgroup looks through its
// shard's whole list for the entries that fall into its stretch; beyond that the searching costs more than the launch
// it saves (binary16, 885 entries in 589824 weights: 864 workgroups 7.5 -> 5.5 us, 2304 10.8 -> 9.9, 10800 41.8 ->
// 43.7) and a kernel of its own goes over the lists.
constexpr uint32_t kScannedOutliers = 4096, kScanningWorkgroups = 4096;
// workgroups per launch: a grid holds fewer than 2^32 work items
constexpr uint32_t kLaunchWorkgroups = 1u << 22;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// ---- output element traits: LUT entries are stored as raw bit patterns ----
__device__ inline uint32_t f32_bits(float v) { return __builtin_bit_cast(uint32_t, v); }

__device__ inline uint16_t to_bf16_bits(float v)
{
    uint32_t u = f32_bits(v);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (uint16_t)((u >> 16) | 0x0040u);
    uint32_t lsb = (u >> 16) & 1u;
    return (uint16_t)((u + 0x7FFFu + lsb) >> 16);
}

struct OutF32 {
    typedef uint32_t bits_t;
    static __device__ inline bits_t cvt(float v) { return f32_bits(v); }
};
struct OutF16 {
    typedef uint16_t bits_t;
    static __device__ inline bits_t cvt(float v) { return to_f16_bits(v); }
};
struct OutBF16 {
    typedef uint16_t bits_t;
    static __device__ inline bits_t cvt(float v) { return to_bf16_bits(v); }
};

template <typename Out> constexpr int kRun = 16 / (int)sizeof(typename Out::bits_t);   // weights per run
constexpr int kItems = 2;                                                              // runs per lane
template <typename Out> constexpr int kWaveWeights = 64 * kItems * kRun<Out>;
template <typename Out> constexpr int kChunkWeights = kWaveWeights<Out> * (kThreads / 64);   // per workgroup

template <typename Out>
__device__ __forceinline__ void store_run(typename Out::bits_t *p, const uint32_t *v)
{
    u32x4 q;
    if constexpr (sizeof(typename Out::bits_t) == 4) q = u32x4{v[0], v[1], v[2], v[3]};
    else q = u32x4{v[0] | (v[1] << 16), v[2] | (v[3] << 16), v[4] | (v[5] << 16), v[6] | (v[7] << 16)};
    STI_STORE(q, (STI_GLOBAL u32x4 *)p);
}

// K-bit shards: first is the wave's first weight (negative where a shard's first run begins before it).
template <int K, typename Out>
__device__ __forceinline__ void decode_packed(const ShardDesc &sd, int64_t n, int64_t first, uint32_t *codes,
                                              typename Out::bits_t *lut, typename Out::bits_t *out, int lane)
{
    constexpr int RUN = kRun<Out>, ITEMS = kItems, WEIGHTS = kWaveWeights<Out>;
    constexpr int PIECES = (WEIGHTS * K / 128 + 1 + 63) / 64;   // 16-byte pieces per lane
    const STI_GLOBAL uint8_t *data = (const STI_GLOBAL uint8_t *)sd.data;
    const int64_t nbytes = (n * K + 7) >> 3;
    const int64_t begin = (first < 0 ? 0 : first * K >> 3) & ~(int64_t)15;
    const int64_t last = first + WEIGHTS < n ? first + WEIGHTS : n;
    const int pieces = (int)(((last * K + 7) >> 3) - begin + 15) >> 4;
    const STI_GLOBAL u32x4 *from = (const STI_GLOBAL u32x4 *)(data + begin);
    float centroid = 0.f;
    if (lane < (1 << K)) centroid = ((const STI_GLOBAL float *)sd.codebook)[lane];
    u32x4 w[PIECES];
    if (begin + (int64_t)pieces * 16 <= nbytes) {
#pragma unroll
        for (int i = 0; i < PIECES; ++i)
            if (i * 64 < pieces) w[i] = from[min(lane + i * 64, pieces - 1)];
    } else {
#pragma unroll
        for (int i = 0; i < PIECES; ++i) {
            const int at = min(lane + i * 64, pieces - 1);
            w[i] = u32x4{0, 0, 0, 0};
            if (begin + (at + 1) * 16 <= nbytes) {
                w[i] = from[at];
            } else {
                // the stream ends inside the piece: its bytes one by one, all on their way at once
                const int left = (int)(nbytes - begin) - at * 16;
                uint32_t byte[16];
#pragma unroll
                for (int t = 0; t < 16; ++t) byte[t] = data[begin + at * 16 + min(t, left - 1)];
#pragma unroll
                for (int t = 0; t < 16; ++t)
                    if (t < left) w[i][t / 4] |= byte[t] << (8 * (t & 3));
            }
        }
    }
    if (lane < (1 << K)) lut[lane] = Out::cvt(centroid);
#pragma unroll
    for (int i = 0; i < PIECES; ++i)
        if (i * 64 < pieces) ((u32x4 *)codes)[min(lane + i * 64, pieces - 1)] = w[i];
    // (a wave's LDS accesses are served in order; the fence keeps the compiler from moving reads up)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int bit0 = (int)(first * K - begin * 8);
    auto run = [&](int item, auto two, typename Out::bits_t *o) {
        const int bit = bit0 + item * (RUN * K);
        const uint32_t *q = codes + (bit >> 5);
        uint64_t x = (((uint64_t)q[1] << 32) | q[0]) >> (bit & 31);
        if (!decltype(two)::value && (bit & 31)) x |= (uint64_t)q[2] << (64 - (bit & 31));
        uint32_t v[RUN];
#pragma unroll
        for (int j = 0; j < RUN; ++j) v[j] = lut[(uint32_t)(x >> (j * K)) & ((1u << K) - 1u)];
        store_run<Out>(o, v);
    };
    if (first >= 0 && first + WEIGHTS <= n) {
        typename Out::bits_t *o = out + first + lane * RUN;
        auto all = [&](auto two) {
#pragma unroll
            for (int r = 0; r < ITEMS; ++r) run(r * 64 + lane, two, o + r * (64 * RUN));
        };
        // runs of up to 33 bits span two dwords wherever they begin; those of 40 and 48 bits, if the first
        // begins with a byte and a 16-bit word
        if (RUN * K <= 33 || (bit0 & (RUN * K > 40 ? 15 : 7)) == 0) all(std::true_type{});
        else all(std::false_type{});
        return;
    }
#pragma unroll 1
    for (int r = 0; r < ITEMS; ++r) {
        const int item = r * 64 + lane;
        const int64_t e = first + item * RUN;
        if (e >= 0 && e + RUN <= n) {
            run(item, std::false_type{}, out + e);
        } else {
#pragma unroll 1
            for (int j = 0; j < RUN; ++j) {
                if (e + j < 0 || e + j >= n) continue;
                const int bit = bit0 + (item * RUN + j) * K;
                const uint64_t x = (((uint64_t)codes[(bit >> 5) + 1] << 32) | codes[bit >> 5]) >> (bit & 31);
                out[e + j] = (typename Out::bits_t)lut[(uint32_t)x & ((1u << K) - 1u)];
            }
        }
    }
}

template <typename Out>
__device__ __forceinline__ void decode_raw(const float *data, int64_t n, int64_t first, typename Out::bits_t *out, int lane)
{
    constexpr int RUN = kRun<Out>, ITEMS = kItems, WEIGHTS = kWaveWeights<Out>;
    typedef float f32x4_v __attribute__((ext_vector_type(4)));
    typedef STI_GLOBAL f32x4_v f32x4_any __attribute__((aligned(4)));
    auto run = [&](int64_t e) {
        f32x4_v x[RUN / 4];
#pragma unroll
        for (int h = 0; h < RUN / 4; ++h) x[h] = *((const f32x4_any *)(data + e) + h);
        uint32_t v[RUN];
#pragma unroll
        for (int j = 0; j < RUN; ++j) v[j] = Out::cvt(x[j / 4][j % 4]);
        store_run<Out>(out + e, v);
    };
    if (first >= 0 && first + WEIGHTS <= n) {
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) run(first + (r * 64 + lane) * RUN);
        return;
    }
#pragma unroll 1
    for (int r = 0; r < ITEMS; ++r) {
        const int64_t e = first + (int64_t)(r * 64 + lane) * RUN;
        if (e + RUN <= 0 || e >= n) continue;
        if (e >= 0 && e + RUN <= n) {
            run(e);
        } else {
#pragma unroll 1
            for (int j = 0; j < RUN; ++j)
                if (e + j >= 0 && e + j < n) out[e + j] = (typename Out::bits_t)Out::cvt(data[e + j]);
        }
    }
}

template <typename Out, typename Table>
__global__ __launch_bounds__(kThreads) void decode_kernel(uint64_t n, uint32_t chunks_per_shard, uint32_t chunks_recip, uint32_t first_chunk,
                                                          int patch, typename Out::bits_t *out, Table table)
{
    __shared__ alignas(16) uint32_t wave_codes[kThreads / 64][kWaveWeights<Out> * 6 / 32 + 12];
    __shared__ typename Out::bits_t wave_lut[kThreads / 64][64];
    const uint32_t block = first_chunk + blockIdx.x;
    const uint32_t s = quotient((int)block, (int)chunks_per_shard, chunks_recip);   // (both below 2^31)
    const uint32_t c = block - s * chunks_per_shard;
    const ShardDesc sd = table.get(s);
    const uint64_t at = (uint64_t)s * n;
    typename Out::bits_t *o = out + at;
    // runs lie on 16-byte boundaries of the output
    const int64_t chunk = (int64_t)c * kChunkWeights<Out> - (int64_t)(at % kRun<Out>);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t first = chunk + wave * kWaveWeights<Out>;
    uint32_t *codes = wave_codes[wave];
    typename Out::bits_t *lut = wave_lut[wave];
    if (first < (int64_t)n) {
        switch (sd.bits) {
            case 2: decode_packed<2, Out>(sd, n, first, codes, lut, o, lane); break;
            case 3: decode_packed<3, Out>(sd, n, first, codes, lut, o, lane); break;
            case 4: decode_packed<4, Out>(sd, n, first, codes, lut, o, lane); break;
            case 5: decode_packed<5, Out>(sd, n, first, codes, lut, o, lane); break;
            case 6: decode_packed<6, Out>(sd, n, first, codes, lut, o, lane); break;
            case 32: decode_raw<Out>((const float *)sd.data, n, first, o, lane); break;
            default: break;
        }
    }
    if (sd.n_outliers == 0 || !patch) return;
    __syncthreads();   // the workgroup's outputs are written
    for (uint32_t t = threadIdx.x; t < sd.n_outliers; t += kThreads) {
        const uint32_t pos = ((const STI_GLOBAL uint32_t *)sd.outlier_pos)[t];
        const int64_t rel = (int64_t)pos - chunk;
        if (rel >= 0 && rel < kChunkWeights<Out> && pos < n) o[pos] = Out::cvt(sd.outlier_val[t]);
    }
}

}  // namespace

// ---------------------------------------------------------------------------
// Working buffer for the matrix-core path (Section "Submodel execution": a buffer
// holding one layer of decompressed weights, shared by all layers) -- here binary16
// and fragment-tiled, so that the GEMM loads every weight fragment as one
// contiguous 1 KiB read.  One wave decodes one 32 x 64 cell with the same per-lane
// loader the fused GEMM uses.
// ---------------------------------------------------------------------------
namespace {

template <typename Table>
__global__ __launch_bounds__(256) void decode_tiled_kernel(uint8_t *out, int total_cells, int d, int dh, int f, int per_shard,
                                                           uint32_t recip_shard, uint32_t recip_d, uint32_t recip_dh, uint32_t recip_f,
                                                           Table tab)
{
    __shared__ uint16_t lut[4][kLutEntries];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int cell = blockIdx.x * 4 + wave;
    if (cell >= total_cells) return;   // whole wave; no workgroup barrier is used
    decode_tiled_cell(tab, cell, CellMap{d, dh, f, per_shard, recip_shard, recip_d, recip_dh, recip_f}, out, lut[wave], lane);
}

}  // namespace

// ---------------------------------------------------------------------------
// Outlier dictionary (Section "quantization per shard": the few weights that do not follow
// the Gaussian are preserved as-is; Section "Implementation": they keep a k-bit placeholder
// in the index matrix and their original weights and offsets are bookkept).  After the
// substitution pass the original weights are scattered back.  grid = shards x chunks, flattened
// (the shard count may pass the limit of the second grid dimension).
// ---------------------------------------------------------------------------
namespace {

template <typename Out, typename Table>
__global__ __launch_bounds__(256) void patch_outliers_kernel(Table table, uint64_t n, uint32_t chunks,
                                                             typename Out::bits_t *out)
{
    const uint32_t shard = blockIdx.x / chunks, chunk = blockIdx.x - shard * chunks;
    const ShardDesc sd = table.get(shard);
    typename Out::bits_t *o = out + (uint64_t)shard * n;
    for (uint32_t t = chunk * 256 + threadIdx.x; t < sd.n_outliers; t += chunks * 256) {
        const uint32_t pos = sd.outlier_pos[t];
        if (pos < n) o[pos] = Out::cvt(sd.outlier_val[t]);
    }
}

template <typename Out>
hipError_t patch_typed(const ShardDesc *table, const InlineShardTable *inline_table, int n_shards,
                       uint32_t max_outliers, uint64_t n, void *out, hipStream_t stream)
{
    uint32_t chunks = (max_outliers + 255) / 256;
    if (chunks > 1024) chunks = 1024;
    while ((uint64_t)chunks * (uint64_t)n_shards > 0x7FFFFFFFull) chunks = (chunks + 1) / 2;
    dim3 grid(chunks * (uint32_t)n_shards);
    typedef typename Out::bits_t bits_t;
    auto go = [&](auto t) {
        patch_outliers_kernel<Out, decltype(t)><<<grid, 256, 0, stream>>>(t, n, chunks, (bits_t *)out);
        return hipGetLastError();
    };
    return table ? go(TablePtr{table}) : with_inline_table(*inline_table, n_shards, go);
}

template <typename Out>
hipError_t launch_typed(const ShardDesc *table, const InlineShardTable *inline_table, int n_shards,
                        uint32_t max_outliers, uint64_t n, void *out, hipStream_t stream)
{
    const uint64_t reach = n + (n % kRun<Out> ? kRun<Out> - 1 : 0);   // first run of a shard may begin before it
    const uint64_t chunks = (reach + kChunkWeights<Out> - 1) / kChunkWeights<Out>;
    const uint64_t blocks = chunks * (uint64_t)n_shards;
    if (blocks == 0) return hipSuccess;
    if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
    const bool patch = max_outliers > 0 && max_outliers <= kScannedOutliers && blocks <= kScanningWorkgroups;
    typedef typename Out::bits_t bits_t;
    for (uint64_t b = 0; b < blocks; b += kLaunchWorkgroups) {
        const dim3 grid((uint32_t)(blocks - b < kLaunchWorkgroups ? blocks - b : kLaunchWorkgroups));
        auto go = [&](auto t) {
            launch((decode_kernel<Out, decltype(t)>), grid, dim3(kThreads), 0, stream, n, (uint32_t)chunks, reciprocal((uint32_t)chunks),
                   (uint32_t)b, (int)patch, (bits_t *)out, t);
        };
        if (table) go(TablePtr{table});
        else with_inline_table(*inline_table, n_shards, go);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || patch || max_outliers == 0) return e;
    return patch_typed<Out>(table, inline_table, n_shards, max_outliers, n, out, stream);
}

template <typename Table>
__global__ __launch_bounds__(256) void patch_outliers_tiled_kernel(int d, int dh, int f, uint8_t *out, Table tab)
{
    const ShardDesc sd = tab.get(blockIdx.y);
    const int64_t wsh = (int64_t)d * (4 * dh + 2 * f);
    uint8_t *o = out + (int64_t)blockIdx.y * wsh * 2;
    for (uint32_t t = blockIdx.x * 256 + threadIdx.x; t < sd.n_outliers; t += gridDim.x * 256) {
        const uint32_t pos = sd.outlier_pos[t];
        if (pos < wsh) *(uint16_t *)(o + tiled_byte_offset(pos, d, dh, f)) = to_f16_bits(sd.outlier_val[t]);
    }
}

}  // namespace

// A shard table on its way to the device: tens of KiB, so what counts is the latency.  A kernel that reads the
// pinned slot, with the slot's event as the completion signal of that one dispatch, takes 2.3 us where a
// copy command and a recorded event behind it took 4 us more for 100 descriptors and 20 us more for 1500.
__global__ __launch_bounds__(256) void fetch_table_kernel(const u32x4 *from, u32x4 *to, uint32_t n)
{
    const uint32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) to[i] = from[i];
}

hipError_t launch_fetch_table(const ShardDesc *pinned, ShardDesc *table, size_t count, hipStream_t stream, hipEvent_t done)
{
    static_assert(sizeof(ShardDesc) % 16 == 0, "descriptors travel as 16-byte pieces");
    const uint64_t n = count * (sizeof(ShardDesc) / 16);
    if (n == 0 || n > 0x7FFFFFFFull) return hipErrorInvalidValue;
    hipExtLaunchKernelGGL(fetch_table_kernel, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, stream, nullptr, done, 0,
                          (const u32x4 *)pinned, (u32x4 *)table, (uint32_t)n);
    return hipGetLastError();
}

hipError_t launch_decode(const ShardDesc *table, const InlineShardTable *inline_table, int n_shards,
                         uint32_t max_outliers, uint64_t n, void *out, sti_dtype out_dtype, hipStream_t stream)
{
    switch (out_dtype) {
        case STI_F32: return launch_typed<OutF32>(table, inline_table, n_shards, max_outliers, n, out, stream);
        case STI_F16: return launch_typed<OutF16>(table, inline_table, n_shards, max_outliers, n, out, stream);
        case STI_BF16: return launch_typed<OutBF16>(table, inline_table, n_shards, max_outliers, n, out, stream);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_patch_outliers_tiled(const InlineShardTable &table, int n_shards,
                                       uint32_t max_outliers, int d, int dh, int f, void *out,
                                       hipStream_t stream)
{
    if (n_shards <= 0 || max_outliers == 0) return hipSuccess;
    uint32_t chunks = (max_outliers + 255) / 256;
    if (chunks > 1024) chunks = 1024;
    with_inline_table(table, n_shards, [&](auto t) {
        patch_outliers_tiled_kernel<<<dim3(chunks, n_shards), 256, 0, stream>>>(d, dh, f, (uint8_t *)out, t);
    });
    return hipGetLastError();
}

hipError_t launch_decode_tiled(const InlineShardTable &table, int n_shards, int d, int dh, int f,
                               void *out, hipStream_t stream)
{
    const int64_t wsh = (int64_t)d * (4 * dh + 2 * f);
    const int64_t cells = wsh / 2048 * n_shards;
    if (cells == 0) return hipSuccess;
    if (d % 64 || dh % 64 || f % 64 || cells > 0x7FFFFFF0) return hipErrorInvalidValue;
    const CellMap m = cell_map(d, dh, f);
    with_inline_table(table, n_shards, [&](auto t) {
        launch((decode_tiled_kernel<decltype(t)>), dim3((uint32_t)((cells + 3) / 4)), dim3(256), 0, stream, (uint8_t *)out, (int)cells,
               d, dh, f, m.per_shard, m.recip_shard, m.recip_d, m.recip_dh, m.recip_f, t);
    });
    return hipGetLastError();
}

hipError_t launch_decode_tiled_table(const ShardDesc *device_table, int n_shards, int d, int dh, int f,
                                     void *out, hipStream_t stream)
{
    const int64_t wsh = (int64_t)d * (4 * dh + 2 * f);
    const int64_t cells = wsh / 2048 * n_shards;
    if (cells == 0) return hipSuccess;
    if (d % 64 || dh % 64 || f % 64 || cells > 0x7FFFFFF0) return hipErrorInvalidValue;
    const CellMap m = cell_map(d, dh, f);
    launch((decode_tiled_kernel<TablePtr>), dim3((uint32_t)((cells + 3) / 4)), dim3(256), 0, stream, (uint8_t *)out, (int)cells,
           d, dh, f, m.per_shard, m.recip_shard, m.recip_d, m.recip_dh, m.recip_f, TablePtr{device_table});
    return hipGetLastError();
}

}  // namespace sti
