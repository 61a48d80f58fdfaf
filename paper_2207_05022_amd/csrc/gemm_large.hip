// Projections of thousands of tokens: the same product, operands and epilogues as the wide-tile kernel (gemm_wide.hip),
//
//   C[T x N] = A[T x K] * W^T,  float32 accumulation in v_mfma_f32_32x32x16_f16,
//
// in tiles of 64 RA rows x 256 columns (RA = 2, 3 or 4), one workgroup of eight waves per compute unit that goes from tile to tile.
//
// What bounds it: the matrix cores at the rate that the chip's power leaves them, and the epilogue, beside which they are idle.  9216 tokens,
// 12 shards of d_model 1024, clocks of wave 0 (libsti_phases.so): FFN1, 256 x 256 tiles, 2370 per K tile of 64, 2048 of them products, at
// 1.66 GHz; Q/K/V, 192 x 256, 1850 and 1536; O and FFN2 on 192 of the 256 units 2220 and 1930 and 1536, at 1.8 GHz (with a branch around every
// request 2530, 2030, 2450 and 2160, at 1.8 and 2.0: the denser the products the lower the clock).  An epilogue takes
// 9830 with GELU, 3600 for Q/K/V, 5000 to 5200 with residual rows.  160-row tiles, which put O and FFN2 on 232 units, gave 0 to 0.6 %.  What costs power or leaves the matrix cores idle:
//   - bytes: both operands go through LDS (an A row is read by four waves, a weight by two), so that a unit asks for 64 KiB per K tile
//     and 256 x 256 outputs - the kernel with weights straight into registers (gemm_wide.hip) asks for 96;
//   - requests in a burst: 64 KiB keep the unit's address path busy for 1024 clocks, and a wave whose request has to wait does not issue
//     its products either.  Requests for A go out among the products of a K tile's last step, those for weights among the first
//     step's of the next one (all in the last step: a tenth more clocks per K tile), LDS reads one by one among the products, too (with all
//     of a step's reads in front of them a fifth more);
//   - start and end of a tile: a workgroup asks for the next tile's first two stages during the last two K tiles of this one.  The
//     epilogue is each wave's own (4 KiB of LDS, no barrier), the residual rows asked for in front of the last K tile.
// Launches, us, this kernel with those branches against gemm_wide.hip before it, which held 128 x 256 tiles of four waves: 9216 tokens, d_model
// 1024, 12 shards Q/K/V 192 x 256 47 / 52, FFN1 256 x 256 66 / 69, O 192 x 256 21.6 / 23.5, FFN2 192 x 256 59 / 66; 5000 tokens, d_model 768
// Q/K/V 22.5 / 27.2; 3000 tokens, 10 shards Q/K/V 128 x 256 14.5 / 17.3.
#include <algorithm>
#include <type_traits>
#include "sti_internal.hpp"
#include "weight_loader.hpp"
#include "gemm_tile.hpp"

// STI_PHASE_STAMPS (libsti_phases.so only, as in gemm_wide.hip): clocks of wave 0 of every workgroup, summed over its tiles, kept in scalar
// registers and written once at its exit.
#ifdef STI_PHASE_STAMPS
namespace {
constexpr int kStampKinds = 4, kStampHeights = 3, kStampSlots = 256, kStampWords = 8;
__device__ unsigned long long sti_large_phase_stamps[kStampKinds * kStampHeights * kStampSlots * kStampWords];
}
// out: [kind][64-row blocks - 2][workgroup][8] = clocks from entry to exit, to the first stage, in K loops, in epilogues; tiles; K tiles of a
// tile; wall clock (100 MHz) at entry and exit (0 = slot unused)
extern "C" int sti_phase_stamps_read_large(unsigned long long *out)
{
    return (int)hipMemcpyFromSymbol(out, HIP_SYMBOL(sti_large_phase_stamps), sizeof(sti_large_phase_stamps));
}
#define STI_CLOCK(name) const unsigned long long name = __builtin_amdgcn_s_memtime()
#define STI_STAMPED(...) __VA_ARGS__
#else
#define STI_CLOCK(name)
#define STI_STAMPED(...)
#endif

namespace sti {
namespace {

constexpr int BK = 64, BN = 256, kWaves = 8;

typedef __attribute__((address_space(3))) void lds_ptr;

template <int RA>
constexpr size_t large_lds_bytes() { return (size_t)2 * (64 * RA + BN) * BK * 2 + kWaves * 4096; }

template <int KIND, int RA>
__global__ __launch_bounds__(kWaves * 64, 2) void gemm_large_kernel(
    // (14 dwords that arrive preloaded; see gemm_wide.hip)
    const void *hot_A, const void *hot_w0, const void *hot_resid, const float *hot_bias0, int32_t hot_w_stride, int32_t hot_T,
    uint32_t hot_band_recip, uint32_t hot_block_recip, uint32_t hot_block_shape, uint32_t hot_n_blocks,
    void *C_out, int32_t ldc, const float *bias1, const float *bias2, ShardIds shard_of)
{
    STI_CLOCK(entry);
    STI_STAMPED(const unsigned long long wall_entry = wall_clock64(); unsigned long long in_loops = 0, in_epilogues = 0; int tiles_done = 0);
    constexpr bool n_split = (KIND == GEMM_QKV || KIND == GEMM_FFN_UP);
    constexpr int BM = 64 * RA, WM = 32 * RA;
    constexpr int A_BYTES = BM * BK * 2, STAGE = A_BYTES + BN * BK * 2;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];

    const int block_rows = hot_block_shape & 0xffff, block_cols = hot_block_shape >> 16, n_blocks = hot_n_blocks;
    const int N = n_split ? n_blocks * block_rows : block_rows;
    const int K = n_split ? block_cols : n_blocks * block_cols;
    const int nkt = K / BK;   // (at least 2)
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 2, wn = wave & 3;
    const int g = lane >> 5, lr = lane & 31;
    const int n_tiles = (N + BN - 1) / BN, m_tiles = (hot_T + BM - 1) / BM;
    const int total = n_tiles * m_tiles, per_xcd = (total + 7) / 8;
    // this workgroup's tiles: first, first + step, ... of its XCD's range
    const int step_tiles = gridDim.x >> 3;
    const int tile_end = min(((int)(blockIdx.x & 7) + 1) * per_xcd, total);
    int tile = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if (tile >= tile_end) return;

    // ---- what this wave brings into LDS per K tile: RA pieces of 8 rows of A (chunks XOR-swizzled by row pair) and the 4 KiB
    //      cell of weight strip `wave` (strips past the last column: the first one again) ----
    int f_tile = tile, f_kt = 0;
    const _Float16 *f_A;
    uint32_t f_src[RA];
    const uint8_t *f_w;
    auto enter_tile = [&]() {
        int tm, tn;
        locate_tile(f_tile, n_tiles, m_tiles, hot_band_recip, tm, tn);
        const int m0 = tm * BM, n0 = tn * BN;
        f_A = (const _Float16 *)hot_A + (int64_t)m0 * K;
#pragma unroll
        for (int j = 0; j < RA; ++j) {
            const int row = (wave + kWaves * j) * 8 + (lane >> 3);
            const int r = m0 + row < hot_T ? row : hot_T - 1 - m0;   // rows past T: row T - 1
            f_src[j] = (uint32_t)((r * K + (((lane & 7) ^ ((row >> 1) & 7)) * 8)) * 2);
        }
        const int col = n0 + wave * 32 < N ? n0 + wave * 32 : 0;   // (N a multiple of 64)
        if constexpr (n_split) {
            const int blk = quotient(col >> 5, block_rows >> 5, hot_block_recip);
            f_w = (const uint8_t *)hot_w0 + (int64_t)blk * hot_w_stride + tiled_cell_offset((col - blk * block_rows) >> 5, 0, block_cols);
        } else {
            f_w = (const uint8_t *)hot_w0 + tiled_cell_offset(col >> 5, 0, block_cols);
        }
    };
    const int tiles_per_kblock = block_cols / BK;
    const uint32_t lane16 = lane * 16;
    const uint32_t lds_base = (uint32_t)(size_t)(lds_ptr *)smem_raw;
    // (written as instructions: the compiler would wait for all outstanding fetches into LDS before the next LDS read)
    auto to_lds = [&](const void *base, uint32_t offset, uint32_t dst) {
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" :: "v"(offset), "s"(base), "s"(dst) : "memory", "m0");
    };
    auto fetch_a = [&](int buf, int j) { to_lds(f_A + f_kt * BK, f_src[j], lds_base + (uint32_t)(buf * STAGE + (wave + kWaves * j) * 1024)); };
    auto fetch_w = [&](int buf, int q, const uint8_t *cell) {
        to_lds(cell + q * 1024, lane16, lds_base + (uint32_t)(buf * STAGE + A_BYTES + wave * 4096 + q * 1024));
    };
    auto w_cell = [&]() -> const uint8_t * {
        if constexpr (n_split) return f_w + (int64_t)f_kt * 4096;
        const int blk = quotient(f_kt, tiles_per_kblock, hot_block_recip);
        return f_w + (int64_t)blk * hot_w_stride + (int64_t)(f_kt - blk * tiles_per_kblock) * 4096;
    };
    auto next_fetch = [&]() {   // the K tile after the one just asked for: of this tile, or the first of the next one
        if (++f_kt < nkt) return;
        f_kt = 0;
        f_tile += step_tiles;
        if (f_tile < tile_end) enter_tile();
    };
    int frag_off[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) frag_off[s] = (wm * WM + lr) * (BK * 2) + (((g * 4 + s) ^ ((lr >> 1) & 7)) * 16);
    // fragment n of a k-step: the two weight strips, then the row blocks
    auto read_fragment = [&](int buf, int s, int n, half8 (&a)[RA], half8 (&b)[2]) {
        const unsigned char *stage = smem_raw + buf * STAGE;
        if (n < 2) b[n] = *(const half8 *)(stage + A_BYTES + (wn * 2 + n) * 4096 + s * 1024 + lane16);
        else if (n < 2 + RA) a[n - 2] = *(const half8 *)(stage + (n - 2) * (32 * BK * 2) + frag_off[s]);
    };
    auto read_fragments = [&](int buf, int s, half8 (&a)[RA], half8 (&b)[2]) {
#pragma unroll
        for (int n = 0; n < 2 + RA; ++n) read_fragment(buf, s, n, a, b);
    };
    float16v acc[RA][2];
    auto multiply = [&](int n, const half8 (&a)[RA], const half8 (&b)[2]) {   // product n of a k-step
        acc[n >> 1][n & 1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(b[n & 1], a[n >> 1], acc[n >> 1][n & 1], 0, 0, 0);
    };
#define STI_FENCE() __builtin_amdgcn_sched_barrier(0)
    half8 a[2][RA], b[2][2];
    int buf = 0;
    // One K tile: fragments of step s + 1 are read while step s is multiplied.  In front of the last step the wave has all of
    // this stage in registers: the next stage has landed (wait, barrier), its first fragments are read and this stage is
    // refilled while the last step's products run.
    bool refill = false;                 // whether the other stage is being filled
    const uint8_t *cell = nullptr;
    // whole: the requests of this step are for later K tiles of the same tile, so that it has no branch.  With a condition around
    // every request (a dozen per K tile, all waves behind one barrier) a K tile took, of 9216 tokens, d_model 1024, 16 shards, Q/K/V
    // 256 x 256 tiles 2500 clocks, now 2320, FFN1 192 x 256 2170, now 2040, FFN2 2200, now 1970: 7200 -> 7040 us for 24 layers.
    auto tile_step = [&](bool later, auto whole) {
        constexpr bool WHOLE = decltype(whole)::value;
        const bool more = WHOLE || later;
#pragma unroll
        for (int s = 0; s < 3; ++s) {
#pragma unroll
            for (int n = 0; n < 2 * RA; ++n) {
                multiply(n, a[s & 1], b[s & 1]);
                STI_FENCE();
                read_fragment(buf, s + 1, n, a[(s + 1) & 1], b[(s + 1) & 1]);
                STI_FENCE();
                if (s == 0 && (WHOLE || refill) && (n & 1) && (n >> 1) < 4) fetch_w(buf ^ 1, n >> 1, cell);
                STI_FENCE();
            }
#pragma unroll
            for (int n = 2 * RA; n < 2 + RA; ++n) read_fragment(buf, s + 1, n, a[(s + 1) & 1], b[(s + 1) & 1]);
            if (s == 0 && (WHOLE || refill)) {
#pragma unroll
                for (int q = RA; q < 4; ++q) fetch_w(buf ^ 1, q, cell);
                if constexpr (WHOLE) ++f_kt;
                else next_fetch();
            }
            STI_FENCE();
        }
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        STI_FENCE();
        if constexpr (!WHOLE) refill = f_tile < tile_end;
        cell = w_cell();
#pragma unroll
        for (int n = 0; n < 2 * RA; ++n) {
            multiply(n, a[1], b[1]);
            STI_FENCE();
            if (more) read_fragment(buf ^ 1, 0, n, a[0], b[0]);
            STI_FENCE();
            if ((WHOLE || refill) && (n & 1)) fetch_a(buf, n >> 1);
            STI_FENCE();
        }
        buf ^= 1;
    };
    static_assert(RA <= 4 && (n_split || RA < 4), "registers for the residual rows");
    auto fetch_stage = [&](int to) {
        const uint8_t *cell = w_cell();
#pragma unroll
        for (int j = 0; j < RA; ++j) fetch_a(to, j);
#pragma unroll
        for (int q = 0; q < 4; ++q) fetch_w(to, q, cell);
        next_fetch();
    };
    enter_tile();
    fetch_stage(0);
    fetch_stage(1);
    if constexpr (RA == 4) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    else if constexpr (RA == 3) asm volatile("s_waitcnt vmcnt(7)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(6)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    STI_FENCE();

    STI_CLOCK(first_stage);
    unsigned char *mine = smem_raw + 2 * STAGE + wave * 4096;   // 32 x 64 outputs on their way to whole rows
    _Float16 *C = (_Float16 *)C_out;
    const _Float16 *R = (const _Float16 *)hot_resid;
    for (; tile < tile_end; tile += step_tiles) {
#pragma unroll
        for (int i = 0; i < RA; ++i)
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][r][v] = 0.f;
        STI_CLOCK(loop_begin);
        read_fragments(buf, 0, a[0], b[0]);
        tile_step(true, std::false_type{});
        int kt = 1;
        for (; kt + 2 < nkt; ++kt) tile_step(true, std::true_type{});
        for (; kt < nkt - 1; ++kt) tile_step(true, std::false_type{});
        int tile_m, tile_n;
        locate_tile(tile, n_tiles, m_tiles, hot_band_recip, tile_m, tile_n);
        const int m0 = tile_m * BM + wm * WM, nw_real = tile_n * BN + wn * 64;
        const int nw = nw_real < N ? nw_real : 0;   // (results of a wave outside are dropped)
        // Residual rows, whole rows of the wave's 64 columns per request (they reach their lanes through LDS), in front of the last K tile
        u32x4 resv[n_split ? 1 : RA][4];
        if constexpr (!n_split) {
#pragma unroll
            for (int i = 0; i < RA; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int m = min(m0 + i * 32 + 8 * j + (lane >> 3), hot_T - 1);   // (rows past T: row T - 1 again, never stored)
                    resv[i][j] = *(const u32x4 *)(R + (int64_t)m * block_rows + nw + (lane & 7) * 8);
                }
            STI_FENCE();
        }
        tile_step(false, std::false_type{});
        STI_CLOCK(loop_end);

        // ---- epilogue, wave by wave: the first two stages of the next tile are on their way ----
        f32x4 bias[2][2][2];
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const float *bp;   // of the strip
            const int col = nw + r * 32;
            if constexpr (n_split) {
                const int blk = quotient(col >> 5, block_rows >> 5, hot_block_recip), row = col - blk * block_rows;
                if constexpr (KIND == GEMM_QKV) {
                    const int which = row >> 6;   // heads of 64 features; a strip lies inside one of Q, K, V
                    bp = (which == 0 ? hot_bias0 : which == 1 ? bias1 : bias2) + shard_of.id(blk) * 64 + (row & 63);
                } else {
                    bp = hot_bias0 + shard_of.id(blk) * block_rows + row;
                }
            } else {
                bp = hot_bias0 + col;
            }
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                bias[r][q][0] = *(const f32x4_any *)(bp + 16 * q + 8 * g);
                bias[r][q][1] = *(const f32x4_any *)(bp + 16 * q + 8 * g + 4);
            }
        }
#pragma unroll
        for (int i = 0; i < RA; ++i) {
            if constexpr (!n_split) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int row = 8 * j + (lane >> 3);
                    *(u32x4 *)(mine + row * 128 + (((lane & 7) ^ (row & 7)) * 16)) = resv[i][j];
                }
                wave_lds_fence();
            }
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {
                const int r = rq >> 1, q = rq & 1;
                // v_permlane32_swap leaves the lane with 8 consecutive columns of its row
                float x[8];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float lo = acc[i][r][(2 * q) * 4 + e], hi = acc[i][r][(2 * q + 1) * 4 + e];
                    const auto sw = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi), false, false);
                    const uint32_t s0 = sw[0], s1 = sw[1];
                    x[e] = __builtin_bit_cast(float, s0);
                    x[4 + e] = __builtin_bit_cast(float, s1);
                }
                half8 *slot = (half8 *)(mine + lr * 128 + (((2 * rq + g) ^ (lr & 7)) * 16));
                half8 o, res;
                if constexpr (!n_split) res = *slot;
#pragma unroll
                for (int e = 0; e < 8; ++e) x[e] += bias[r][q][e >> 2][e & 3];
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
                *slot = o;
            }
            wave_lds_fence();
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int row = 8 * j + (lane >> 3), m = m0 + i * 32 + row;
                const u32x4 piece = *(const u32x4 *)(mine + row * 128 + (((lane & 7) ^ (row & 7)) * 16));
                if (m < hot_T && nw_real < N) *(u32x4 *)(C + (int64_t)m * ldc + nw + (lane & 7) * 8) = piece;
            }
            wave_lds_fence();
        }
        STI_CLOCK(tile_done);
        STI_STAMPED(in_loops += loop_end - loop_begin; in_epilogues += tile_done - loop_end; ++tiles_done);
    }
#ifdef STI_PHASE_STAMPS
    const unsigned long long leaving = __builtin_amdgcn_s_memtime();
    if (tid == 0 && blockIdx.x < (unsigned)kStampSlots) {
        unsigned long long *o = sti_large_phase_stamps + (((size_t)KIND * kStampHeights + RA - 2) * kStampSlots + blockIdx.x) * kStampWords;
        o[0] = leaving - entry; o[1] = first_stage - entry; o[2] = in_loops; o[3] = in_epilogues;
        o[4] = tiles_done; o[5] = nkt; o[6] = wall_entry; o[7] = wall_clock64();
    }
#endif
}

template <int KIND, int RA>
hipError_t launch_variant(const GemmProblem &p, const GemmBlocks &blocks, int N, hipStream_t stream)
{
    constexpr bool n_split = (KIND == GEMM_QKV || KIND == GEMM_FFN_UP);
    constexpr size_t lds = large_lds_bytes<RA>();
    static const hipError_t attr_status =   // once per instantiation, safe from several threads
        hipFuncSetAttribute((const void *)gemm_large_kernel<KIND, RA>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (attr_status != hipSuccess) return attr_status;
    const int n_tiles = (N + BN - 1) / BN, total = n_tiles * ((p.T + 64 * RA - 1) / (64 * RA));
    const int64_t w_stride = p.n_blocks > 1 ? (const uint8_t *)blocks.b[1].w - (const uint8_t *)blocks.b[0].w : 0;
    const uint32_t band_recip = band_reciprocal(n_tiles);
    const uint32_t block_recip = reciprocal(n_split ? p.block_rows / 32 : p.block_cols / BK);
    launch((gemm_large_kernel<KIND, RA>), dim3(std::min((total + 7) / 8 * 8, kComputeUnits)), dim3(kWaves * 64), lds, stream, p.A, blocks.b[0].w, p.resid, p.bias0,
           (int32_t)w_stride, p.T, band_recip, block_recip, (uint32_t)p.block_rows | (uint32_t)p.block_cols << 16, (uint32_t)p.n_blocks,
           p.C, p.ldc, p.bias1, p.bias2, shard_ids(blocks));
    return hipGetLastError();
}

template <int RA>
hipError_t launch_kind(const GemmProblem &p, const GemmBlocks &blocks, int N, hipStream_t stream)
{
    switch (p.kind) {
    case GEMM_QKV: return launch_variant<GEMM_QKV, RA>(p, blocks, N, stream);
    case GEMM_FFN_UP: return launch_variant<GEMM_FFN_UP, RA>(p, blocks, N, stream);
    default: break;
    }
    if constexpr (RA < 4) {
        if (p.kind == GEMM_OUT) return launch_variant<GEMM_OUT, RA>(p, blocks, N, stream);
        if (p.kind == GEMM_FFN_DOWN) return launch_variant<GEMM_FFN_DOWN, RA>(p, blocks, N, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_gemm_large(const GemmProblem &p, const GemmBlocks &blocks, int N, int row_blocks, hipStream_t stream)
{
    // (a wave stores whole strips of 64 columns; a workgroup starts with two stages of its first tile; no partial sums, no work beside the tiles)
    const int K = p.kind == GEMM_QKV || p.kind == GEMM_FFN_UP ? p.block_cols : p.n_blocks * p.block_cols;
    if (N % 64 || K < 2 * BK || p.k_splits > 0 || p.next_workgroups > 0 || p.next_outliers > 0) return hipErrorInvalidValue;
    switch (row_blocks) {
    case 2: return launch_kind<2>(p, blocks, N, stream);
    case 3: return launch_kind<3>(p, blocks, N, stream);
    case 4: return launch_kind<4>(p, blocks, N, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace sti
