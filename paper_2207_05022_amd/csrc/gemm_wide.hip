// Projections of the layer on the matrix cores for many tokens (Section "A primer on
// transformer": the Q/K/V, output and two FFN linear layers), with the weights taken from
// the per-layer fragment-tiled binary16 working buffer (Section "Submodel execution": a
// layer's shards are decompressed into a working buffer before the layer runs).
//
//   C[T x N] = A[T x K] * W^T,  float32 accumulation in v_mfma_f32_32x32x16_f16.
//
// One workgroup of NW waves owns a (RA*32) x (NW*32) tile and is sized so that a compute
// unit holds all its waves at once (12 wave slots at this register budget): all waves of a
// unit then move through the K loop in step, share one copy of the A tile and finish together.  Launches of
// many tiles go to the kernel with larger ones (gemm_large.hip); the choice is made here, for both.
//   - the A tile [BM x 64] goes global -> LDS directly (global_load_lds_dwordx4, no
//     registers, no LDS store instructions), three stages; its 16-byte chunks are XOR-swizzled
//     by row pair so that the unpadded rows read without bank conflicts;
//   - the K loop runs in rounds of three K tiles (one per stage) whose loads all exist, without a branch; 128 x 384 outputs
//     of 12 K tiles 22350 -> 20800 clocks;
//   - a wave's weight fragments are contiguous 1 KiB loads from the working buffer, two K
//     tiles ahead, straight into registers; both kinds of load address memory as a scalar
//     base plus a 32-bit lane offset (measured 1.5 % faster end to end than 64-bit lane
//     addresses);
//   - the A fragments of k-step s+1 are read from LDS while the MFMAs of step s run;
//   - the weight fragment is the first MFMA operand, so a lane's accumulators are runs of
//     output columns of one token row; v_permlane32_swap merges them into 16-byte pieces,
//     which get bias / GELU / residual in registers and leave through an LDS copy of the
//     whole tile, so that every global store instruction writes whole rows of the tile.
//
// Sequences of exactly 128 tokens (the padded length the paper profiles with): a 128-row tile is
// one whole sequence, so the Q/K/V projection is cut into 128 x 384 tiles = Q | K | V of two
// heads, and the workgroup that has multiplied such a tile keeps it in LDS and computes those
// heads' attention itself (kind GEMM_QKV_ATTN): no Q/K/V buffer in memory and no attention launch.
#include <algorithm>
#include <math.h>
#include <type_traits>
#include "sti_internal.hpp"
#include "weight_loader.hpp"
#include "gemm_tile.hpp"
#include "attention_core.hpp"

// STI_PHASE_STAMPS (the phase-budget build libsti_phases.so only, never the product library): wave 0
// of every workgroup reads the shader clock counter at six points (kernel entry, prologue loads
// requested, first K tile landed, K loop done, epilogue arithmetic done, last store acknowledged)
// plus the 100 MHz wall clock at both ends, keeps the values in scalar registers (a store inside the
// K loop would count against its hand-written waits) and writes them once, at its exit.
#ifdef STI_PHASE_STAMPS
namespace {
constexpr int kStampKinds = 5, kStampSlots = 512, kStampWords = 8;
__device__ unsigned long long sti_phase_stamps[kStampKinds * kStampSlots * kStampWords];
}
// out: [kind][slot][8] = six clock stamps, wall clock at entry, wall clock at exit (0 = slot unused)
extern "C" int sti_phase_stamps_read(unsigned long long *out, int clear)
{
    hipError_t e = hipMemcpyFromSymbol(out, HIP_SYMBOL(sti_phase_stamps), sizeof(sti_phase_stamps));
    if (e == hipSuccess && clear) {
        void *dev = nullptr;
        e = hipGetSymbolAddress(&dev, HIP_SYMBOL(sti_phase_stamps));
        if (e == hipSuccess) e = hipMemset(dev, 0, sizeof(sti_phase_stamps));
    }
    return (int)e;
}
#define STI_STAMP(i) (stamp[i] = __builtin_amdgcn_s_memtime())
#define STI_STAMPS_OUT()                                                                               \
    do {                                                                                               \
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                                               \
        STI_STAMP(5);                                                                                  \
        const unsigned slot = blockIdx.y * gridDim.x + blockIdx.x;                                     \
        if (threadIdx.x == 0 && slot < (unsigned)kStampSlots) {                                        \
            unsigned long long *o = sti_phase_stamps + ((size_t)KIND * kStampSlots + slot) * kStampWords; \
            for (int i_ = 0; i_ < 6; ++i_) o[i_] = stamp[i_];                                          \
            o[6] = wall0;                                                                              \
            o[7] = wall_clock64();                                                                     \
        }                                                                                              \
    } while (0)
#else
#define STI_STAMP(i) ((void)0)
#define STI_STAMPS_OUT() ((void)0)
#endif

namespace sti {
namespace {

constexpr int BK = 64;   // K positions per LDS stage

// At most N of the loads of this wave still on their way
template <int N>
__device__ inline void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory"); }

typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) const void global_cptr;
typedef __attribute__((address_space(3))) void lds_ptr;

// LDS of the attention that follows the Q/K/V tile (GEMM_QKV_ATTN): per head Q and K row-major
// with padded rows and V transposed, for 128 positions of 64 features
constexpr int ATT_L = 128, ATT_DH = 64, ATT_KPAD = ATT_DH + 8, ATT_VTS = ATT_L + 8;
constexpr int ATT_HEAD_HALVES = 2 * ATT_L * ATT_KPAD + ATT_DH * ATT_VTS;
constexpr size_t kAttentionLdsBytes = (size_t)2 * ATT_HEAD_HALVES * 2;

template <int RA, int NW, int KS>
constexpr size_t wide_lds_bytes()
{
    constexpr size_t stages = (size_t)KS * 3 * (RA * 32) * BK * 2;
    constexpr size_t tile = (size_t)(RA * 32) * (NW * 32 + 8) * 2;
    constexpr size_t partial = (size_t)(KS - 1) * (RA * 32) * (NW * 32) * 4;
    constexpr size_t m = stages > tile ? stages : tile;
    return m > partial ? m : partial;
}

// Workgroups of a Q/K/V launch beyond those of its tiles.  With 128-token sequences the launch has one
// 128 x 384 tile per sequence and pair of heads (192 for 32 sequences of BERT-base), with a few hundred
// tokens a few dozen tiles: fewer than the chip has compute units, so these land on units the tiles
// leave idle.  They decompress the next layer's shards into its working buffer (Section "Submodel
// execution": the next layer is made ready while the current one computes) - work that is bound by
// memory latency and bandwidth, beside a projection that is bound by the matrix cores.
// All waves of the workgroup come here.  LDS: the binary16 codebooks, bitwidths and data pointers of all
// shards, so that a cell costs one round trip to memory; a wave asks for three cells at a time, the first
// three together with the codebooks (a short projection must not end up waiting for these workgroups).
constexpr size_t kNextDecodeLdsBytes = (size_t)kMaxShardsPerLayer * (kLutEntries * 2 + 4 + 8);

template <int NWAVES>
__device__ inline void decode_next_layer(const GemmProblem &p, int d, unsigned char *smem, int worker)
{
    uint16_t *luts = (uint16_t *)smem;                                                    // [shards][64]
    int32_t *bits_of = (int32_t *)(smem + (size_t)kMaxShardsPerLayer * kLutEntries * 2);  // [shards]
    uint64_t *data_of = (uint64_t *)(smem + (size_t)kMaxShardsPerLayer * (kLutEntries * 2 + 4));
    // (pointers that come out of memory are taken as global-memory pointers by hand: the compiler would
    //  address through them with the slower flat instructions)
    auto as_global = [](uint64_t a) { return (const void *)(global_cptr *)a; };
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // round trip 1: the descriptors; round trip 2: the codebooks together with the first cells
    constexpr int SPW = (kMaxShardsPerLayer + NWAVES - 1) / NWAVES;   // shards a wave stages
    float centroid[SPW];
    int staged_bits[SPW];
#pragma unroll
    for (int j = 0; j < SPW; ++j) {
        const int s = wave + j * NWAVES;
        centroid[j] = 0.f;
        staged_bits[j] = 0;
        if (s < p.next_shards) {
            const ShardDesc sd = p.next_table[s];
            staged_bits[j] = sd.bits;
            if (lane == 0) {
                bits_of[s] = sd.bits;
                data_of[s] = (uint64_t)sd.data;
            }
            if (sd.bits <= 6 && lane < (1 << sd.bits)) centroid[j] = ((const float *)as_global((uint64_t)sd.codebook))[lane];
        }
    }
    __syncthreads();
    const int dh = p.d_head, f = p.next_ffn_per_shard;
    const int total = (int)((int64_t)d * (4 * dh + 2 * f) / 2048) * p.next_shards;
    const int stride = p.next_workgroups * NWAVES;
    constexpr int CH = 3;   // cells a wave asks for at a time
    TiledCell t[CH];
    int bits[CH];
    Raw raw[CH];
    auto request = [&](int first) {
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int cell = first + c * stride;
            bits[c] = 0;   // (no cell)
            if (cell < total) {
                t[c] = locate_tiled_cell(cell, p.next_cells);
                bits[c] = bits_of[t[c].shard];
                raw[c] = load_tiled_cell_raw(t[c], bits[c], as_global(data_of[t[c].shard]), lane);
            }
        }
    };
    int first = worker * NWAVES + wave;
    request(first);
#pragma unroll
    for (int j = 0; j < SPW; ++j) {
        const int s = wave + j * NWAVES;
        if (s < p.next_shards && staged_bits[j] <= 6 && lane < (1 << staged_bits[j]))
            luts[s * kLutEntries + lane] = (uint16_t)f16_bits(centroid[j]);
    }
    __syncthreads();
    while (first < total) {
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            if (bits[c] != 0) {
                half8 fr[4];
                decode_raw_any(bits[c], raw[c], luts + t[c].shard * kLutEntries, fr);
                store_tiled_cell(t[c], d, dh, f, fr, (uint8_t *)p.next_out, lane);
            }
        }
        first += CH * stride;
        if (first < total) request(first);
    }
}

// Workgroups of an O or FFN2 projection (gemm_wide_out_carries) beyond those of its tiles: the outlier dictionaries of the layer that this
// layer's Q/K/V launch has decompressed.  One entry per thread, chunks workgroups per shard: three round trips
// (descriptor, entry, store) beside the projection, where a launch of its own is on the chain of launches.
// 1023 tokens, 10 shards of BERT-base with about 900 entries each: 61.8 -> 58.6 us per layer.
template <int NT>
__device__ inline void patch_next_layer(const GemmProblem &p, int d, int dh, int worker)
{
    const int chunks = (p.next_outliers + NT - 1) / NT, f = p.next_ffn_per_shard;
    const int s = worker / chunks;
    const uint32_t t = (uint32_t)(worker - s * chunks) * NT + threadIdx.x;
    const ShardDesc sd = p.next_table[s];
    const int64_t wsh = (int64_t)d * (4 * dh + 2 * f);
    if (t < sd.n_outliers) {
        const uint32_t pos = ((const uint32_t *)(global_cptr *)sd.outlier_pos)[t];
        const float val = ((const float *)(global_cptr *)sd.outlier_val)[t];
        if (pos < wsh) *(uint16_t *)((uint8_t *)p.next_out + s * wsh * 2 + tiled_byte_offset(pos, d, dh, f)) = to_f16_bits(val);
    }
}

// KS = 2 (outputs as narrow as d_model, long K): the workgroup has two groups of NW waves that
// each take one half of K for the same tile, with A stages of their own; at the end each
// hands half of its accumulators over through LDS and ends the other half of the tile.  Twice the waves per compute unit for
// a tile count that is fixed by the output size.
// SUMS (O and FFN2, gemm_wide_sum_planes): raw float32 sums in hot_k_splits planes, for launch_layernorm to add bias and residual in float32.
template <int KIND, int RA, int NW, int KS, bool SUMS>
__global__ __launch_bounds__(NW * KS * 64, 3) void gemm_wide_kernel(
    // what the first loads of a workgroup depend on, as leading scalar arguments: these arrive
    // preloaded in scalar registers (the build asks for kernel-argument preloading), so that the
    // first A fetches and weight loads are not behind a round trip to the argument buffer
    // (14 dwords fit: block_shape = block_rows | block_cols << 16, blocks_splits = n_blocks | k_splits << 16; reciprocals of the
    // tiles of a band of the tile order and of a weight block's 32-row strips (N split) or K tiles: divisions in their place,
    // one of them in every step of the K loop of O and FFN2, made 24 layers of d_model 1024, 24 x 384 tokens 0.9 to 1.8 % slower,
    // from box to box)
    const void *hot_A, const void *hot_w0, const void *hot_resid, const float *hot_bias0, int32_t hot_w_stride,
    int32_t hot_T, uint32_t hot_band_recip, uint32_t hot_block_recip, uint32_t hot_block_shape, uint32_t hot_blocks_splits,
    GemmProblem p, ShardIds shard_of)   // (of p, only the fields that are not among the leading arguments are read)
{
    const int hot_block_rows = hot_block_shape & 0xffff, hot_block_cols = hot_block_shape >> 16;
    const int hot_n_blocks = hot_blocks_splits & 0xffff, hot_k_splits = hot_blocks_splits >> 16;
#ifdef STI_PHASE_STAMPS
    unsigned long long stamp[6] = {0, 0, 0, 0, 0, 0};
    const unsigned long long wall0 = wall_clock64();
    STI_STAMP(0);
#endif
    constexpr int BM = RA * 32, BN = NW * 32, NT = NW * KS * 64, NTH = NW * 64, STAGES = 3;
    constexpr bool n_split = (KIND == GEMM_QKV || KIND == GEMM_FFN_UP || KIND == GEMM_QKV_ATTN);
    constexpr bool qkv = (KIND == GEMM_QKV || KIND == GEMM_QKV_ATTN);
    static_assert(KIND != GEMM_QKV_ATTN || (RA == 4 && NW == 12 && KS == 1), "two heads of one 128-token sequence per tile");
    constexpr int STAGE = BM * BK;              // halves per A stage
    constexpr int FETCHES = BM / 8;             // fetch instructions per A stage: 8 rows (1 KiB) each
    constexpr int FPW = (FETCHES + NW - 1) / NW;   // per wave: wave w issues fetches w, w + NW, ...
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];

    const int N = n_split ? hot_n_blocks * hot_block_rows : hot_block_rows;
    const int K = n_split ? hot_block_cols : hot_n_blocks * hot_block_cols;
    // K is split over the KS wave groups of the workgroup and, for few tiles, over
    // gridDim.y workgroups per tile as well, with a plane of sums each
    static_assert(!SUMS || !n_split, "sums: O and FFN2");
    const int splits = SUMS ? hot_k_splits : 1;
    const int hot_lda = K, hot_ldr = hot_block_rows;   // (rows of A and of the residual follow each other)
    const int nkt_all = splits > 1 ? K / BK / splits : K / BK;   // K tiles of the workgroup; of this wave's group: nkt, from kt0 on
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = wave_all / NW, wave = wave_all - half * NW;   // K group, column strip
    const int nkt = KS == 1 ? nkt_all : (nkt_all + 1 - half) >> 1;
    const int kt0 = (int)blockIdx.y * nkt_all + (KS == 1 ? 0 : half * ((nkt_all + 1) >> 1));
    const int g = lane >> 5, lr = lane & 31;
    const int n_tiles = (N + BN - 1) / BN;
    const int m_tiles = (hot_T + BM - 1) / BM;
    const int total_tiles = n_tiles * m_tiles;
    const int per_xcd = (total_tiles + 7) / 8;
    const int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if constexpr (qkv) {
        if ((int)(blockIdx.x >> 3) >= per_xcd) {   // behind the tiles' workgroups: the next layer's decompression
            if (p.next_workgroups > 0) decode_next_layer<NW * KS>(p, hot_block_cols, smem_raw, (int)blockIdx.x - 8 * per_xcd);
            return;
        }
    }
    if constexpr (KIND == GEMM_OUT || KIND == GEMM_FFN_DOWN) {
        if ((int)(blockIdx.x >> 3) >= per_xcd) {   // behind the tiles' workgroups: the next layer's outlier dictionaries
            if (p.next_outliers > 0 && blockIdx.y == 0)
                patch_next_layer<NT>(p, hot_block_rows, p.d_head, (int)blockIdx.x - 8 * per_xcd);
            return;
        }
    }
    if ((int)(blockIdx.x >> 3) >= per_xcd || tile >= total_tiles) return;
    int tile_m, tile_n;
    locate_tile(tile, n_tiles, m_tiles, hot_band_recip, tile_m, tile_n);
    const int m0 = tile_m * BM;
    // N and the block widths are multiples of 64, so a wave's columns are all inside or all
    // outside the matrix and inside one block; a wave outside recomputes the first columns and its results are
    // dropped by the column mask of the stores
    const int nw_real = tile_n * BN + wave * 32;
    const int nw = nw_real < N ? nw_real : 0;
    int nblk = 0, nrow0 = nw;
    if (n_split) {
        nblk = quotient(nw >> 5, hot_block_rows >> 5, hot_block_recip);
        nrow0 = nw - nblk * hot_block_rows;
    }
    const int tiles_per_kblock = n_split ? nkt : hot_block_cols / BK;

    float16v acc[RA];
#pragma unroll
    for (int i = 0; i < RA; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;

    // ---- A tile: lane l of a fetch instruction fills LDS slot (row l/8, chunk l%8) of its 8
    //      rows with the chunk (l%8) ^ ((row/2)%8) of that row, so that the 16 rows that one
    //      quarter of a fragment read touches (128-byte rows, two per 64-bank line) fall on
    //      16 different bank groups; rows past T repeat row T-1 ----
    const _Float16 *A = (const _Float16 *)hot_A + (int64_t)m0 * hot_lda;   // first row of the tile
    uint32_t src[FPW];   // byte offset of this lane's chunk from the tile's first row and K tile
#pragma unroll
    for (int j = 0; j < FPW; ++j) {
        const int row = (wave + NW * j) * 8 + (lane >> 3);   // row inside the tile
        const int r = m0 + row < hot_T ? row : hot_T - 1 - m0;
        src[j] = (uint32_t)((r * hot_lda + (((lane & 7) ^ ((row >> 1) & 7)) * 8)) * 2);   // < 2^24 * 2
    }
    // The loads of the K loop are written as instructions rather than through the compiler:
    // its own bookkeeping would wait for every outstanding fetch into LDS before the next LDS
    // read, which is exactly the overlap this loop is built for.  The waits are in k_loop().
    const uint32_t lds_base = (uint32_t)(size_t)(lds_ptr *)smem_raw;
    auto fetch_a = [&](int kt, int buf, auto fetches) {   // (fetches: those of this wave)
#pragma unroll
        for (int j = 0; j < decltype(fetches)::value; ++j) {
            const _Float16 *gp = A + (kt0 + kt) * BK;   // scalar base, per-lane 32-bit offset
            const uint32_t at = src[j];
            const uint32_t dst = lds_base + (uint32_t)(((half * STAGES + buf) * STAGE + (wave + NW * j) * 8 * BK) * 2);
            asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                         :: "v"(at), "s"(gp), "s"(dst) : "memory", "m0");
        }
    };
    // byte offset of this lane's fragment of k-step s inside row block 0 of a stage
    int frag_off[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) frag_off[s] = lr * (BK * 2) + (((g * 4 + s) ^ ((lr >> 1) & 7)) * 16);

    const uint32_t lane16 = lane * 16;
    auto frag_ptr = [&](int kt) -> const uint8_t * {
        int blk, ktb, row;
        kt += kt0;
        if (n_split) {
            blk = nblk; ktb = kt; row = nrow0;
        } else {
            blk = quotient(kt, tiles_per_kblock, hot_block_recip); ktb = kt - blk * tiles_per_kblock; row = nw;
        }
        // (the blocks of a working buffer lie at a constant distance: no look-up in the block table)
        const uint8_t *base = (const uint8_t *)hot_w0 + (int64_t)blk * hot_w_stride;   // (stride < 2^31)
        return base + tiled_cell_offset(row >> 5, ktb, hot_block_cols);   // wave-uniform
    };

    // Three A stages and three sets of weight fragment registers: the loads of K tile t+2 are
    // issued while tile t is multiplied (A fetches first, then the 4 fragment loads; with K
    // unsplit behind the MFMAs of the first k-step, so that those start right after the
    // barrier: measured 2 % faster end to end than issuing at the top, while the split-K
    // shapes are faster with the issue at the top).  The wait in front of the barrier is
    // written by hand: it lets the loads of tile t+1, the last ones issued, stay in flight.
    u32x4 bw[STAGES][4];
    auto fetch_w = [&](int kt, u32x4 (&dst)[4]) {
        const uint8_t *q = frag_ptr(kt);
        asm volatile("global_load_dwordx4 %0, %4, %5\n\t"
                     "global_load_dwordx4 %1, %4, %5 offset:1024\n\t"
                     "global_load_dwordx4 %2, %4, %5 offset:2048\n\t"
                     "global_load_dwordx4 %3, %4, %5 offset:3072"
                     : "=&v"(dst[0]), "=&v"(dst[1]), "=&v"(dst[2]), "=&v"(dst[3]) : "v"(lane16), "s"(q) : "memory");
    };
    // EARLY (O and FFN2 that end rows): what
    // the epilogue adds (bias and residual rows) is asked for before the K loop: asked for in
    // the epilogue, these loads cost a whole round trip (3-4 thousand clocks of a 20-50 thousand
    // clock kernel).  They are the oldest loads in flight, so the first wait of the K loop
    // covers them.
    constexpr bool EARLY = !n_split && !SUMS;
    static_assert(n_split || RA <= 2, "registers for the residual rows through the K loop");
    const _Float16 *R = (const _Float16 *)hot_resid;
    static_assert(KS == 1 || KS == 2, "two groups, each of which ends half of the tile's pieces");
    constexpr int PIECES_OWN = RA * 2 / KS, BIASES = PIECES_OWN < 2 ? 1 : 2;   // pieces of 32 rows x 16 columns per wave
    const int first_piece = KS == 1 ? 0 : half * PIECES_OWN;                    // (piece n: rows 32 (n / 2), columns 16 (n % 2))
    f32x4 bias[2][2];
    u32x4 resv[EARLY ? PIECES_OWN : 1];
    auto load_epilogue_operands = [&]() {
#pragma unroll
        for (int q = 0; q < BIASES; ++q) {
            const int c = 16 * (BIASES == 1 ? first_piece : q) + 8 * g;    // first column of the piece inside the wave's columns
            const float *bp;
            if constexpr (qkv) {
                const int nrow = nrow0 + c;
                const int which = nrow / ATT_DH, e0 = nrow - which * ATT_DH;
                bp = (which == 0 ? hot_bias0 : (which == 1 ? p.bias1 : p.bias2)) + shard_of.id(nblk) * ATT_DH + e0;
            } else if constexpr (KIND == GEMM_FFN_UP) {
                bp = hot_bias0 + shard_of.id(nblk) * hot_block_rows + nrow0 + c;
            } else {
                bp = hot_bias0 + nw + c;
            }
            bias[q][0] = *(const f32x4_any *)bp;
            bias[q][1] = *(const f32x4_any *)(bp + 4);
        }
        if constexpr (EARLY) {
#pragma unroll
            for (int j = 0; j < PIECES_OWN; ++j) {
                const int m = min(m0 + ((first_piece + j) >> 1) * 32 + lr, hot_T - 1);   // (rows past T: row T-1 again, never stored)
                resv[j] = *(const u32x4 *)(R + (int64_t)m * hot_ldr + nw + 16 * ((first_piece + j) & 1) + 8 * g);
            }
        }
    };
    // fetches: A fetches this wave issues per stage.  Rounds of three K tiles whose loads all exist run without a branch: every taken
    // one holds up all waves of the workgroup behind the same barrier, and with a condition around each load and wait there were about
    // ten per K tile.  Clocks of a K loop before and now: 128 x 384 tiles, 12 K tiles, 22350 / 20800; 64 x 192, 12 K tiles, 10370 / 8370;
    // K shared by two groups, 24 K tiles each, 34000 / 30600.  Power takes part of it back (1.88 -> 1.81 GHz): 4096 tokens, 12 layers
    // 1155 -> 1133 us, 12 x 384 tokens of d_model 1024, 6 layers, 1140 -> 1112.
    auto k_loop = [&](auto fetches) {
        constexpr int PER_TILE = decltype(fetches)::value + 4;   // loads of a K tile
        auto issue = [&](int kt, int buf, u32x4 (&dst)[4]) {
            fetch_a(kt, buf, fetches);
            fetch_w(kt, dst);
        };
        auto step = [&](int kt, int buf, u32x4 (&bcur)[4], u32x4 (&bnew)[4], auto whole) {
            constexpr bool WHOLE = decltype(whole)::value;
            const bool more = WHOLE || kt + STAGES - 1 < nkt;
            const int next = buf == 0 ? STAGES - 1 : buf - 1;
            // the weight fragments and the A stage of tile kt have landed (the barrier below is a
            // scheduling boundary: no MFMA of this step is placed above the wait) ...
            if (WHOLE || kt + 1 < nkt) wait_loads<PER_TILE>();
            else wait_loads<0>();
            // ... for every wave, and every wave is done reading the stage that is refilled next
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
#ifdef STI_PHASE_STAMPS
            if (kt == 0) STI_STAMP(2);
#endif
            if (KS == 2 && more) issue(kt + STAGES - 1, next, bnew);
            const unsigned char *stage = smem_raw + (half * STAGES + buf) * (STAGE * 2);
            half8 a_cur[RA], a_nxt[RA];
#pragma unroll
            for (int i = 0; i < RA; ++i) a_cur[i] = *(const half8 *)(stage + i * (32 * BK * 2) + frag_off[0]);
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                if (s < 3) {
#pragma unroll
                    for (int i = 0; i < RA; ++i)
                        a_nxt[i] = *(const half8 *)(stage + i * (32 * BK * 2) + frag_off[s + 1]);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < RA; ++i)
                    acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, bcur[s]), a_cur[i], acc[i], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (KS == 1 && s == 0 && more) issue(kt + STAGES - 1, next, bnew);
                __builtin_amdgcn_sched_barrier(0);
                if (s < 3) {
#pragma unroll
                    for (int i = 0; i < RA; ++i) a_cur[i] = a_nxt[i];
                }
            }
        };
        if (nkt > 0) issue(0, 0, bw[0]);
        if (nkt > 1) issue(1, 1, bw[1]);
        STI_STAMP(1);
        int kt = 0;
        for (; kt + 4 < nkt; kt += 3) {
            step(kt, 0, bw[0], bw[2], std::true_type{});
            step(kt + 1, 1, bw[1], bw[0], std::true_type{});
            step(kt + 2, 2, bw[2], bw[1], std::true_type{});
        }
        for (; kt < nkt; kt += 3) {
            step(kt, 0, bw[0], bw[2], std::false_type{});
            if (kt + 1 < nkt) step(kt + 1, 1, bw[1], bw[0], std::false_type{});
            if (kt + 2 < nkt) step(kt + 2, 2, bw[2], bw[1], std::false_type{});
        }
    };
    static_assert(FPW <= 8, "loads of two K tiles in the counter of the waits");
    if (EARLY) load_epilogue_operands();
    if (FETCHES % NW == 0 || wave < FETCHES % NW) k_loop(std::integral_constant<int, FPW>{});
    else k_loop(std::integral_constant<int, FPW - 1>{});
    // (a group with a K tile less than the first one: that one's last barrier)
    if (KS == 2 && nkt * 2 < nkt_all) __builtin_amdgcn_s_barrier();
    STI_STAMP(3);

    // ---- epilogue ----
    // Lane l holds token row lr and output columns (v/4)*8 + g*4 + v%4 of each 32 x 32 block.
    // Swapping the column groups 2q and 2q+1 between lanes l and l+32 leaves the lane with the
    // 8 consecutive columns 16q + 8g .. +8 of its row: one 16-byte piece of the output row.
    constexpr int LDT = BN + 8;   // padded row of the staged tile (halves): conflict-free 16-byte writes
    _Float16 *tile_out = (_Float16 *)smem_raw;
    if (n_split) load_epilogue_operands();
    __syncthreads();   // every wave is done with the A stages
    if constexpr (KIND == GEMM_QKV_ATTN) {
        // ---- the tile is Q | K | V of heads 2 tile_n and 2 tile_n + 1 for the 128 positions of
        //      sequence tile_m: leave them in LDS (binary16, bias added: the values the unfused
        //      route stores) and run the two heads' attention (Section "A primer on transformer":
        //      per-head attention scores) with eight of the twelve waves, 32 queries each ----
        _Float16 *hb = (_Float16 *)smem_raw + (wave / 6) * ATT_HEAD_HALVES;   // this wave's head
        const int part = (wave % 6) >> 1;      // 0 Q, 1 K, 2 V (wave-uniform)
        const int ch = (wave & 1) * 32;        // first feature of the wave's 32 columns
        int Lk = ATT_L;                        // keys that take part
        if (p.key_lengths) Lk = min(max(p.key_lengths[tile_m], 1), ATT_L);
#pragma unroll
        for (int i = 0; i < RA; ++i) {
            const int row = i * 32 + lr;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                half8 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float lo = acc[i][(2 * q) * 4 + e], hi = acc[i][(2 * q + 1) * 4 + e];
                    const auto sw = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, lo),
                                                                     __builtin_bit_cast(uint32_t, hi), false, false);
                    const uint32_t s0 = sw[0], s1 = sw[1];
                    o[e] = (_Float16)(__builtin_bit_cast(float, s0) + bias[q][0][e]);
                    o[4 + e] = (_Float16)(__builtin_bit_cast(float, s1) + bias[q][1][e]);
                }
                const int c = ch + 16 * q + 8 * g;
                if (part < 2) {
                    *(half8 *)(hb + part * (ATT_L * ATT_KPAD) + row * ATT_KPAD + c) = o;
                } else {
                    // (a masked key has weight zero, but 0 times an infinity or NaN in its value would not be)
                    if (row >= Lk) o = half8{};
                    _Float16 *vt = hb + 2 * (ATT_L * ATT_KPAD);
#pragma unroll
                    for (int e = 0; e < 8; ++e) vt[(c + e) * ATT_VTS + row] = o[e];
                }
            }
        }
        __syncthreads();
        STI_STAMP(4);   // (here: Q, K, V of the tile are in LDS; what follows is the attention)
        const int head = tile_n * 2 + (wave >> 2);          // present-head index of waves 0..7
        if (wave >= 8 || head >= hot_n_blocks) return;
        hb = (_Float16 *)smem_raw + (wave >> 2) * ATT_HEAD_HALVES;
        const _Float16 *Qs = hb, *Ks = hb + ATT_L * ATT_KPAD, *Vt = hb + 2 * (ATT_L * ATT_KPAD);
        const int qrow = (wave & 3) * 32 + lr;
        half8 qf[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) qf[s] = *(const half8 *)(Qs + qrow * ATT_KPAD + s * 16 + g * 8);
        float16v ov[2];
        const float run_sum = attention_scores_in_registers<4>(qf, Ks, ATT_KPAD, Vt, ATT_VTS, Lk, lane, ov);
        const float inv = 1.0f / run_sum;
        _Float16 *out = (_Float16 *)p.C + (int64_t)(m0 + qrow) * p.ldc + head * ATT_DH;
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
                half4 h;
#pragma unroll
                for (int i = 0; i < 4; ++i) h[i] = (_Float16)(ov[e][v4 * 4 + i] * inv);
                *(half4 *)(out + e * 32 + v4 * 8 + g * 4) = h;
            }
        STI_STAMPS_OUT();
        return;
    }
    // Two K groups: each ends half of the tile's pieces, adds to them what the other has of them (through LDS, from the same lane and
    // registers) and asked for their bias and residual rows alone.  With all of it left to the first group (the same bits) 12 layers of BERT-base took,
    // us: 1023 tokens with dictionaries 586, now 575, 1116 tokens 622 / 614, 2048 808 / 801, 4096 1086 / 1079; d_model 1024, 1200 tokens 941 / 931.
    auto end_pieces = [&](auto group) {
        constexpr int G = decltype(group)::value, FIRST = G * PIECES_OWN;
        if constexpr (KS == 2) {
            f32x4 *part = (f32x4 *)smem_raw;
            const int th = tid - G * NTH;
#pragma unroll
            for (int j = 0; j < PIECES_OWN; ++j)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int n = (1 - G) * PIECES_OWN + j, v = (n & 1) * 8 + h * 4;
                    part[((G * PIECES_OWN + j) * 2 + h) * NTH + th] = f32x4{acc[n >> 1][v], acc[n >> 1][v + 1], acc[n >> 1][v + 2], acc[n >> 1][v + 3]};
                }
            __syncthreads();
#pragma unroll
            for (int j = 0; j < PIECES_OWN; ++j)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const f32x4 other = part[(((1 - G) * PIECES_OWN + j) * 2 + h) * NTH + th];
                    const int n = FIRST + j, v = (n & 1) * 8 + h * 4;
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[n >> 1][v + e] += other[e];
                }
            __syncthreads();   // the sums are in registers: the buffer can take the staged tile
        }
#pragma unroll
        for (int j = 0; j < PIECES_OWN; ++j) {
            const int i = (FIRST + j) >> 1, q = (FIRST + j) & 1;
            const int row = i * 32 + lr, m = m0 + row;   // row inside the tile, token
            float x[8];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                // (element values first: a bit cast applied to a vector element itself reads element 0)
                const float lo = acc[i][(2 * q) * 4 + e], hi = acc[i][(2 * q + 1) * 4 + e];
                const auto sw = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, lo),
                                                                 __builtin_bit_cast(uint32_t, hi), false, false);
                const uint32_t s0 = sw[0], s1 = sw[1];
                x[e] = __builtin_bit_cast(float, s0);
                x[4 + e] = __builtin_bit_cast(float, s1);
            }
            if constexpr (SUMS) {   // 32 bytes per lane and piece
                if (nw_real < N && m < hot_T) {
                    float *dst = (float *)p.C + (int64_t)blockIdx.y * p.partial_stride + (int64_t)m * p.ldc + nw + 16 * q + 8 * g;
                    *(f32x4 *)dst = f32x4{x[0], x[1], x[2], x[3]};
                    *(f32x4 *)(dst + 4) = f32x4{x[4], x[5], x[6], x[7]};
                }
                continue;
            }
            half8 res = {}, o;
            if constexpr (EARLY) res = __builtin_bit_cast(half8, resv[j]);
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] += bias[BIASES == 1 ? 0 : q][e >> 2][e & 3];
            if constexpr (KIND == GEMM_FFN_UP) {
                const float none = zero_of(x);
#pragma unroll
                for (int e = 0; e < 8; ++e) x[e] = gelu_wide(x[e], none);
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                if constexpr (!n_split) x[e] += (float)res[e];
                o[e] = (_Float16)x[e];
            }
            *(half8 *)(tile_out + row * LDT + wave * 32 + 16 * q + 8 * g) = o;
        }
    };
    if (KS == 1 || half == 0) end_pieces(std::integral_constant<int, 0>{});
    else end_pieces(std::integral_constant<int, KS - 1>{});
    if constexpr (SUMS) {
        STI_STAMP(4);
        STI_STAMPS_OUT();
        return;
    }
    __syncthreads();
    STI_STAMP(4);
    // BN/8 lanes per tile row: every store instruction writes whole rows of the tile
    _Float16 *C = (_Float16 *)p.C;
    constexpr int PIECES_PER_ROW = BN / 8;
    constexpr int PASSES = BM * PIECES_PER_ROW / NT;
    static_assert(PASSES * NT == BM * PIECES_PER_ROW, "whole passes");
    u32x4 piece[PASSES];
#pragma unroll
    for (int j = 0; j < PASSES; ++j) {
        const int pc = tid + NT * j;
        piece[j] = *(const u32x4 *)(tile_out + (pc / PIECES_PER_ROW) * LDT + (pc % PIECES_PER_ROW) * 8);
    }
#pragma unroll
    for (int j = 0; j < PASSES; ++j) {
        const int pc = tid + NT * j;
        const int m = m0 + pc / PIECES_PER_ROW, n = tile_n * BN + (pc % PIECES_PER_ROW) * 8;
        if (m < hot_T && n < N) *(u32x4 *)(C + (int64_t)m * p.ldc + n) = piece[j];
    }
    STI_STAMPS_OUT();
}

template <int KIND, int RA, int NW, int KS, bool SUMS>
hipError_t launch_variant(const GemmProblem &p, const GemmBlocks &blocks, int N, hipStream_t stream);

template <int KIND, int RA, int NW, int KS>
hipError_t launch_shape(const GemmProblem &p, const GemmBlocks &blocks, int N, hipStream_t stream)
{
    // (tiles of choose() for sums: 32 x 96, 64 x 64 and, O with dictionaries beside it, 64 x 192)
    constexpr bool sums = KS == 2 && (RA == 1 || NW == 2 || (NW == 6 && KIND == GEMM_OUT));
    if (p.k_splits > 0) {
        if constexpr (sums) return launch_variant<KIND, RA, NW, KS, true>(p, blocks, N, stream);
        return hipErrorInvalidValue;
    }
    return launch_variant<KIND, RA, NW, KS, false>(p, blocks, N, stream);
}

template <int KIND, int RA, int NW, int KS, bool SUMS>
hipError_t launch_variant(const GemmProblem &p, const GemmBlocks &blocks, int N, hipStream_t stream)
{
    constexpr int BM = RA * 32, BN = NW * 32;
    constexpr size_t lds = (KIND == GEMM_QKV_ATTN && kAttentionLdsBytes > wide_lds_bytes<RA, NW, KS>())
                               ? kAttentionLdsBytes : wide_lds_bytes<RA, NW, KS>();
    // once per instantiation, and safe when several host threads make their first call together
    static const hipError_t attr_status =
        hipFuncSetAttribute((const void *)gemm_wide_kernel<KIND, RA, NW, KS, SUMS>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (attr_status != hipSuccess) return attr_status;
    const int total = ((N + BN - 1) / BN) * ((p.T + BM - 1) / BM);
    const bool n_split = (KIND == GEMM_QKV || KIND == GEMM_FFN_UP || KIND == GEMM_QKV_ATTN);
    dim3 grid(((total + 7) / 8) * 8, SUMS ? p.k_splits : 1);
    if ((KIND == GEMM_QKV_ATTN || KIND == GEMM_QKV) && p.next_workgroups > 0) {
        static_assert((KIND != GEMM_QKV_ATTN && KIND != GEMM_QKV) || kNextDecodeLdsBytes <= lds, "the decompressing workgroups' tables fit");
        if (!p.next_table || !p.next_out || p.next_shards <= 0 || p.next_shards > kMaxShardsPerLayer ||
            p.next_ffn_per_shard <= 0 || p.next_ffn_per_shard % 64 || p.block_cols % 64 ||
            (int)grid.x + p.next_workgroups > kComputeUnits)
            return hipErrorInvalidValue;
        grid.x += p.next_workgroups;
    }
    if ((KIND == GEMM_OUT || KIND == GEMM_FFN_DOWN) && p.next_outliers > 0) {
        constexpr int NT = NW * KS * 64;
        if (!p.next_table || !p.next_out || p.next_shards <= 0 || p.next_ffn_per_shard <= 0 || p.d_head <= 0) return hipErrorInvalidValue;
        grid.x += p.next_shards * ((p.next_outliers + NT - 1) / NT);
    }
    GemmProblem q = p;
    if (p.next_workgroups > 0) q.next_cells = cell_map(p.block_cols, p.d_head, p.next_ffn_per_shard);
    const int64_t w_stride = p.n_blocks > 1 ? (const uint8_t *)blocks.b[1].w - (const uint8_t *)blocks.b[0].w : 0;
    const ShardIds shard_of = shard_ids(blocks);
    const int n_tiles = (N + BN - 1) / BN;
    const uint32_t band_recip = band_reciprocal(n_tiles);
    const uint32_t block_recip = reciprocal(n_split ? p.block_rows / 32 : p.block_cols / BK);
    launch((gemm_wide_kernel<KIND, RA, NW, KS, SUMS>), grid, dim3(NW * KS * 64), lds, stream, p.A, blocks.b[0].w,
           p.resid, p.bias0, (int32_t)w_stride, p.T, band_recip, block_recip, (uint32_t)p.block_rows | (uint32_t)p.block_cols << 16,
           (uint32_t)p.n_blocks | (uint32_t)(SUMS ? p.k_splits : 1) << 16, q, shard_of);
    return hipGetLastError();
}

template <int RA, int NW>
hipError_t launch_kind(const GemmProblem &p, const GemmBlocks &blocks, int N, hipStream_t stream)
{
    switch (p.kind) {
    case GEMM_QKV: return launch_shape<GEMM_QKV, RA, NW, 1>(p, blocks, N, stream);
    case GEMM_FFN_UP: return launch_shape<GEMM_FFN_UP, RA, NW, 1>(p, blocks, N, stream);
    case GEMM_OUT: return launch_shape<GEMM_OUT, RA, NW, 1>(p, blocks, N, stream);
    case GEMM_FFN_DOWN: return launch_shape<GEMM_FFN_DOWN, RA, NW, 1>(p, blocks, N, stream);
    case GEMM_QKV_ATTN: break;   // one shape only, launched by launch_gemm_wide itself
    }
    return hipErrorInvalidValue;
}

template <int RA, int NW>   // K shared by two groups of waves
hipError_t launch_groups(const GemmProblem &p, const GemmBlocks &blocks, int N, hipStream_t stream)
{
    return p.kind == GEMM_OUT ? launch_shape<GEMM_OUT, RA, NW, 2>(p, blocks, N, stream) : launch_shape<GEMM_FFN_DOWN, RA, NW, 2>(p, blocks, N, stream);
}

// Tile shapes, rows x columns, and the time of a launch: start_us + rounds * (K tiles * (tile_us + full_us * fill) + round_us (+ gelu_us for
// FFN1, resid_us for O and FFN2)), rounds = tiles on the busiest compute unit (shared: several workgroups on a unit, half way between that and
// the average), fill = average / busiest: a chip with idle units clocks higher.  The shapes of 12000 values and more: fitted
// to 256 launches of 64 layer shapes with the K loops of then, 0.95 of that today; the smaller ones to 936 launches of 234 layer shapes (350 to
// 9216 tokens, d_model 256 .. 1024, 2 to 16 shards), off by 6 % (root mean square).  The shape so chosen costs 0.8 % (Q/K/V, FFN1) and 1.6 % (O,
// FFN2) more than the fastest of all over those 936.
// What a small tile is for: a unit takes in about 48 bytes a clock whatever runs on it, rows + columns of a tile per K position, so that
// with few tokens the launch ends sooner the smaller and squarer the tiles are, as long as every one has a unit of its own; and four or six
// waves start sooner than twelve.  Without 64 x 128 and the shapes of fewer than 12000 values Q/K/V and FFN1 cost 6 %, O and FFN2 22 % more than the
// fastest.  FFN2 of 1116 tokens, BERT-base, us: 64 x 192 with twelve waves 19.4, 32 x 192 16.3; 12 layers of it: 64 x 192 782, 64 x 96 702, 64 x 64
// 664 (with four groups of waves 683, six 711); 1023 tokens, 10 shards: 32 x 96 584, 64 x 64 602, 64 x 96 633.  More than 256 of these tiles
// lose to the next larger shape (1792 tokens: 64 x 96 781, 64 x 64 862), and more groups than two to two.
// large: gemm_large.hip.
struct Shape {
    int rows, cols, groups;   // groups of waves that share K: O and FFN2, a workgroup to a unit
    bool shared, large;
    float start_us, tile_us, full_us, round_us, gelu_us, resid_us;
};
enum ShapeId { W128x384, W128x288, W64x384, W64x192, W64x128, G64x192, G64x96, G64x64, G32x96, L128x256, L192x256, L256x256, kShapeCount };
constexpr Shape kShapes[kShapeCount] = {{128, 384, 1, false, false, 1.064f, 0.693f, 0.597f, 4.341f, 3.173f, 1.482f},   // Q/K/V and FFN1
                                        {128, 288, 1, false, false, 0.541f, 0.659f, 0.404f, 4.712f, 2.926f, 1.254f},   // Q/K/V beside a decompression
                                        {64, 384, 1, false, false, 0.142f, 0.451f, 0.32f, 3.524f, 1.662f, 1.596f},
                                        {64, 192, 1, true, false, 1.396f, 0.402f, 0.085f, 1.159f, 0.798f, 1.425f},
                                        {64, 128, 1, true, false, 3.13f, 0.264f, 0.007f, 0.34f, 0.22f, 0.12f},
                                        {64, 192, 2, false, false, 2.821f, 0.279f, 0.126f, 0.f, 0.f, 1.415f},
                                        {64, 96, 2, false, false, 3.84f, 0.197f, 0.034f, 0.f, 0.f, 0.f},
                                        {64, 64, 2, false, false, 3.63f, 0.144f, 0.032f, 0.f, 0.f, 0.f},
                                        {32, 96, 2, false, false, 3.18f, 0.097f, 0.091f, 0.f, 0.f, 0.f},
                                        {128, 256, 1, false, true, 1.311f, 0.558f, 0.419f, 2.137f, 1.976f, 1.092f},
                                        {192, 256, 1, false, true, 2.014f, 0.734f, 0.559f, 2.099f, 3.087f, 1.89f},
                                        {256, 256, 1, false, true, 2.727f, 0.869f, 0.734f, 2.812f, 4.151f, 2.318f}};

// Workgroups beside `tiles` that still find a compute unit of their own in the first round; fewer than an eighth of the
// chip are not used.
inline int spare_units(long tiles)
{
    const long spare = kComputeUnits - (tiles + 7) / 8 * 8;
    return spare >= kComputeUnits / 8 ? (int)spare : 0;
}

// Time of a layer's decompression beside the tiles of a Q/K/V launch, by `spare` workgroups of nw waves, and of one that
// stands in the chain by itself (grouped: several full layers in one launch).  Fitted to 98 layer shapes (512 x 8, 768 x 6
// to 12, 1024 x 12 and 16 shards, 704 to 6144 tokens) with every tile shape, each with and without the decompression beside
// it.  What a Q/K/V shape costs is therefore not its own time alone: 768 x 10 shards at 3584 tokens took
// 789 us per 8 layers where 32 workgroups of four waves were left to the decompression (now 706), 768 at 4096 tokens where
// none were (now 741).
// (In the chain: 13.8 us for four layers of 12 shards of BERT-base, 6.8 for one.  With 1.3 us less, 1824 tokens took launches of their own: 2.5 % slower.)
inline float beside_us(float cells, int spare, int nw) { return (1.0f + 0.035f * nw) * cells / (spare * nw) + 4.f + 0.5f * nw; }
inline float in_chain_us(float cells, bool grouped) { return cells * 2048.f * 0.4e-6f + (grouped ? 0.7f : 4.f); }

// 2048-weight cells of the layer that p.next_shards and p.next_ffn_per_shard describe
inline float next_cells(const GemmProblem &p)
{
    return (float)p.next_shards * p.block_cols * (4 * (p.block_rows / 3) + 2 * p.next_ffn_per_shard) / 2048.f;
}

}  // namespace

bool gemm_wide_supported(const GemmProblem &p, const GemmBlocks &blocks)
{
    if (p.n_blocks <= 0 || p.T <= 0) return false;
    for (int b = 0; b < p.n_blocks; ++b)
        if (blocks.b[b].bits != kTiledBits) return false;
    // the kernel addresses block b as block 0 + b * (distance of the first two)
    const int64_t stride = p.n_blocks > 1 ? (const uint8_t *)blocks.b[1].w - (const uint8_t *)blocks.b[0].w : 0;
    for (int b = 2; b < p.n_blocks; ++b)
        if ((const uint8_t *)blocks.b[b].w - (const uint8_t *)blocks.b[0].w != stride * b) return false;
    // ... and takes the stride and the block shape and count as 32- and 16-bit kernel arguments
    if (stride < 0 || stride > INT32_MAX || p.n_blocks > 0xffff || p.block_rows > 0xffff || p.block_cols > 0xffff ||
        p.k_splits > 0xffff)
        return false;
    return true;
}

namespace {

// Whether O and FFN2 leave their sums in float32, with bias and residual added by LayerNorm, instead of rows in binary16: few tokens and
// K tiles in fours, from 12 on, with which K can be split over workgroups (gemm_wide_sum_planes), and then whether it is or not.  What a call of
// so many tokens keeps by it: 12 layers of BERT-base, error against float64 with these rows in binary16 and with sums, 2-norm, 707 tokens 6.9e-4 /
// 5.5e-4, 1024 tokens 6.6e-4 / 5.2e-4; what it costs: 557 / 567, 605 / 612 us.
inline bool leaves_sums(int64_t T, int N, int k_tiles) { return T <= gemm_wide_most_tokens(2, N) && k_tiles >= 12 && k_tiles % 4 == 0; }

struct Choice {
    int shape;       // index into kShapes
    long tiles;
    int nkt_total;
    float us;        // estimated; infinite: no shape has workgroups to spare
};

// The shape with the least estimated time; with next_workgroups, of those that have workgroups to spare; with next_outliers, of those that
// add in the order of the shape without: the bits of a call do not depend on where its dictionaries go in.
Choice choose(const GemmProblem &p, int N)
{
    int groups = 0;   // (0: any)
    if (p.next_outliers > 0) {
        GemmProblem alone = p;
        alone.next_outliers = 0;
        groups = kShapes[choose(alone, N).shape].groups;
    }
    const bool n_split = (p.kind == GEMM_QKV || p.kind == GEMM_FFN_UP || p.kind == GEMM_QKV_ATTN);
    const int nkt = (n_split ? p.block_cols : p.n_blocks * p.block_cols) / BK;
    const bool sums = !n_split && leaves_sums(p.T, N, nkt);
    const bool beside = p.kind == GEMM_QKV && p.next_workgroups > 0;
    Choice best = {};
    best.us = INFINITY;
    for (int c = 0; c < kShapeCount; ++c) {
        const Shape &sh = kShapes[c];
        if ((c == W128x288 && !beside) || (!n_split && sh.rows >= 128 && !sh.large) || (sh.groups > 1 && (n_split || nkt < 4))) continue;
        // (the large tiles have no workgroups for the next layer's shards or dictionaries, whole strips of 64 columns, two K tiles at least,
        // no sums, and 256 rows only without residual)
        if (sh.large && (beside || sums || p.next_outliers > 0 || N % 64 || nkt < 2 || (!n_split && sh.rows > 192))) continue;
        const long tiles = (long)((N + sh.cols - 1) / sh.cols) * ((p.T + sh.rows - 1) / sh.rows);
        const float avg = (float)tiles / kComputeUnits;
        const long per_cu = (tiles + kComputeUnits - 1) / kComputeUnits;   // workgroups on the busiest unit
        // (64 x 128 tiles, three and more to a unit: twelve shapes of 1300 to 6500 tokens 1 % faster to 6 % slower than the next larger shape)
        if ((sh.groups > 1 && per_cu > 1) || (c == W64x128 && per_cu > 2) || (groups && sh.groups != groups)) continue;
        // (sums, 12 K tiles and more on at most 192 units in tiles of 64 x 64: one group of waves, or 64 x 96 tiles, are slower by this table)
        if (sums && (sh.groups == 1 || c == G64x96)) continue;
        // (an output projection with dictionaries beside it: tiles with units to spare, or FFN2 takes them, see gemm_wide_out_carries)
        if (p.kind == GEMM_OUT && p.next_outliers > 0 && (c == W64x128 || sh.cols < 192)) continue;
        const float rounds = sh.shared ? std::max(1.f, (avg + per_cu) / 2) : (float)per_cu;
        float us = sh.start_us + rounds * (nkt * (sh.tile_us + sh.full_us * avg / per_cu) + sh.round_us + (p.kind == GEMM_FFN_UP ? sh.gelu_us : 0.f) +
                                           (n_split ? 0.f : sh.resid_us));
        if (beside) {
            const int spare = spare_units(tiles);
            if (spare == 0) continue;
            us = std::max(us, beside_us(next_cells(p), spare, sh.cols / 32));
        }
        if (us < best.us) {
            best.us = us;
            best.shape = c;
            best.tiles = tiles;
            best.nkt_total = nkt;
        }
    }
    return best;
}

}  // namespace

// Planes of float32 sums that O or FFN2 leaves, 0: rows in binary16.  With the fewest tiles (narrow models, more than 256 neurons per
// shard) a workgroup would walk a long K range alone while most compute units idle: K is then split over 2 or 4 workgroups per tile as
// well, each with at least 3 K tiles per wave group, while they fill at most half the chip (8 splits, or splitting up to the whole
// chip, cost more in the LayerNorm that adds the planes than they save here).
int gemm_wide_sum_planes(const GemmProblem &p)
{
    if (p.kind == GEMM_QKV || p.kind == GEMM_FFN_UP || p.kind == GEMM_QKV_ATTN || p.n_blocks <= 0 || p.T <= 0) return 0;
    if (!leaves_sums(p.T, p.block_rows, p.n_blocks * p.block_cols / BK)) return 0;
    GemmProblem alone = p;   // (the same number of planes with dictionaries beside it, in whatever tiles: the same bits)
    alone.next_outliers = 0;
    const Choice ch = choose(alone, p.block_rows);
    if (kShapes[ch.shape].groups == 1) return 1;
    for (int s = 4; s >= 2; s >>= 1)
        if (ch.tiles * s <= kComputeUnits / 2 && ch.nkt_total % (2 * s) == 0 && ch.nkt_total / (2 * s) >= 3) return s;
    return 1;
}

// Which of a layer's two d_model-wide projections loses less when the next layer's dictionaries go out beside it: neither may be in large
// tiles then, and O not in those of fewer than 192 columns, 64 x 128 among them.  FFN2 therefore carries wherever it has no large tiles and O
// has small ones; O elsewhere.  Where O has small tiles it is one as the other: ten shapes of 1023 to 3400 tokens, 200 to 900 entries
// per shard, six layers, beside FFN2 against beside O in its own tile 0.15 % slower to 1.0 % faster, 0.25 % faster on
// average (1023 tokens, 10 shards of BERT-base 295.0 / 294.6 us, d_model 1024, 1200 tokens 468.3 / 470.6, 512 x 8 shards, 3000 tokens
// 294.4 / 295.5).
bool gemm_wide_out_carries(GemmProblem out, GemmProblem down, int entries)
{
    auto lost = [&](GemmProblem &p) {
        p.next_outliers = 0;
        const float alone = choose(p, p.block_rows).us;
        p.next_outliers = entries;
        return choose(p, p.block_rows).us - alone;
    };
    return lost(out) <= lost(down);
}

int gemm_wide_max_sum_planes(int64_t T, int N)
{
    for (int s = 4; s >= 2; s >>= 1)
        if (T <= gemm_wide_most_tokens(s, N)) return s;
    return 1;
}

int64_t gemm_wide_most_tokens(int splits, int N)   // (64 x 192 tiles)
{
    return (int64_t)64 * (kComputeUnits / 2 / splits / ((N + 191) / 192));
}

// The fused form pays once its 128 x 384 tiles (one per sequence and pair of heads) fill at least
// half of the compute units; below that the separate Q/K/V projection spreads over more of them.
bool gemm_wide_fuses_attention(int B, int L, int m, int dh)
{
    return L == ATT_L && dh == ATT_DH && m > 0 && (int64_t)B * ((m + 1) / 2) >= kComputeUnits / 2;
}

// Every workgroup of the launch, tiles and decompression, finds a compute unit in the first round.
int gemm_wide_spare_workgroups(const GemmProblem &p, bool grouped)
{
    if (p.n_blocks <= 0 || p.T <= 0) return 0;
    if (p.kind == GEMM_QKV_ATTN) return spare_units((long)(p.T / ATT_L) * ((p.n_blocks + 1) / 2));
    if (p.kind != GEMM_QKV) return 0;
    const int N = p.n_blocks * p.block_rows;
    GemmProblem q = p;
    q.next_workgroups = 0;
    const Choice alone = choose(q, N);
    if (p.next_shards <= 0) return spare_units(alone.tiles);
    q.next_workgroups = 1;
    const Choice beside = choose(q, N);
    return beside.us <= alone.us + in_chain_us(next_cells(p), grouped) ? spare_units(beside.tiles) : 0;
}

hipError_t launch_gemm_wide(const GemmProblem &p, const GemmBlocks &blocks, hipStream_t stream)
{
    const bool n_split = (p.kind == GEMM_QKV || p.kind == GEMM_FFN_UP || p.kind == GEMM_QKV_ATTN);
    const int N = n_split ? p.n_blocks * p.block_rows : p.block_rows;
    if (p.T <= 0 || N <= 0) return hipSuccess;
    if (!gemm_wide_supported(p, blocks)) return hipErrorInvalidValue;
    if (N % 32 || p.block_rows % 32 || p.block_cols % BK || p.ldc % 8) return hipErrorInvalidValue;
    // (the kernel takes these distances from the products' shapes)
    if (p.lda != (n_split ? p.block_cols : p.n_blocks * p.block_cols) || (!n_split && p.ldr != p.block_rows) ||
        ((p.kind == GEMM_QKV || p.kind == GEMM_QKV_ATTN) && p.d_head != ATT_DH))
        return hipErrorInvalidValue;
    if (p.kind == GEMM_QKV_ATTN) {
        if (p.T % ATT_L || p.block_rows != 3 * ATT_DH || p.d_head != ATT_DH || p.ldc < p.n_blocks * ATT_DH)
            return hipErrorInvalidValue;
        return launch_shape<GEMM_QKV_ATTN, 4, 12, 1>(p, blocks, N, stream);
    }
    const Choice ch = choose(p, N);
    if (!(ch.us < INFINITY)) return hipErrorInvalidValue;
    if (!n_split && p.k_splits != gemm_wide_sum_planes(p)) return hipErrorInvalidValue;
    switch (ch.shape) {
    case W128x384: return p.kind == GEMM_QKV ? launch_shape<GEMM_QKV, 4, 12, 1>(p, blocks, N, stream) : launch_shape<GEMM_FFN_UP, 4, 12, 1>(p, blocks, N, stream);
    case W128x288: return launch_shape<GEMM_QKV, 4, 9, 1>(p, blocks, N, stream);
    case W64x384: return launch_kind<2, 12>(p, blocks, N, stream);
    case W64x192: return launch_kind<2, 6>(p, blocks, N, stream);
    case W64x128: return launch_kind<2, 4>(p, blocks, N, stream);
    case G64x192: return launch_groups<2, 6>(p, blocks, N, stream);
    case G64x96: return launch_groups<2, 3>(p, blocks, N, stream);
    case G64x64: return launch_groups<2, 2>(p, blocks, N, stream);
    case G32x96: return launch_groups<1, 3>(p, blocks, N, stream);
    default: return launch_gemm_large(p, blocks, N, kShapes[ch.shape].rows / 64, stream);
    }
}

}  // namespace sti

// The tile that a projection takes in a launch of its own, for the tests of its kernels (no device is touched): rows, columns, groups of
// waves that share K, and whether it is one of gemm_large.hip.  outliers: entries per dictionary of a next layer put in beside it.
extern "C" void sti_internal_projection_tile(int kind, int T, int n_blocks, int block_rows, int block_cols, int outliers, int *tile)
{
    sti::GemmProblem p = {};
    p.kind = (sti::GemmKind)kind;
    p.T = T; p.n_blocks = n_blocks; p.block_rows = block_rows; p.block_cols = block_cols; p.next_outliers = outliers;
    const bool n_split = kind == sti::GEMM_QKV || kind == sti::GEMM_FFN_UP;
    const sti::Choice ch = sti::choose(p, n_split ? n_blocks * block_rows : block_rows);
    const sti::Shape &sh = sti::kShapes[ch.shape];
    tile[0] = sh.rows; tile[1] = sh.cols; tile[2] = sh.groups; tile[3] = sh.large;
}

// The planes of float32 sums that it leaves (gemm_wide_sum_planes); likewise.
extern "C" int sti_internal_sum_planes(int kind, int T, int n_blocks, int block_rows, int block_cols, int outliers)
{
    sti::GemmProblem p = {};
    p.kind = (sti::GemmKind)kind;
    p.T = T; p.n_blocks = n_blocks; p.block_rows = block_rows; p.block_cols = block_cols; p.next_outliers = outliers;
    return sti::gemm_wide_sum_planes(p);
}

// Whether O (or else FFN2) takes the next layer's dictionaries along, of at most `outliers` entries each; likewise for the tests.
extern "C" int sti_internal_out_carries(int T, int n_shards, int d_model, int ffn_per_shard, int outliers)
{
    sti::GemmProblem out = {};
    out.kind = sti::GEMM_OUT;
    out.T = T; out.n_blocks = n_shards; out.block_rows = d_model; out.block_cols = 64;
    sti::GemmProblem down = out;
    down.kind = sti::GEMM_FFN_DOWN;
    down.block_cols = ffn_per_shard;
    return sti::gemm_wide_out_carries(out, down, outliers);
}
