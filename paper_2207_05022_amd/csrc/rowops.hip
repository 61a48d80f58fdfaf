// Row-wise and elementwise helpers of the layer: LayerNorm over d features
// (biased variance, Section "A primer on transformer" runs stock BERT layers)
// and activation type conversion.
#include <type_traits>
#include "sti_internal.hpp"
#include "lane_ops.hpp"
#include "split_planes.hpp"
#include "split_decode.hpp"

namespace sti {
namespace {

__device__ inline uint16_t f32_to_bf16_bits(float v)
{
    uint32_t u = __builtin_bit_cast(uint32_t, v);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (uint16_t)((u >> 16) | 0x0040u);
    return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}
__device__ inline float bf16_bits_to_f32(uint16_t b)
{
    return __builtin_bit_cast(float, (uint32_t)b << 16);
}

template <int DT> struct Elem;
template <> struct Elem<STI_F32> {
    typedef float type;
    static __device__ inline float load(const float *p) { return *p; }
    static __device__ inline void store(float *p, float v) { *p = v; }
};
template <> struct Elem<STI_F16> {
    typedef _Float16 type;
    static __device__ inline float load(const _Float16 *p) { return (float)*p; }
    static __device__ inline void store(_Float16 *p, float v) { *p = (_Float16)v; }
};
template <> struct Elem<STI_BF16> {
    typedef uint16_t type;
    static __device__ inline float load(const uint16_t *p) { return bf16_bits_to_f32(*p); }
    static __device__ inline void store(uint16_t *p, float v) { *p = f32_to_bf16_bits(v); }
};

// element offset of columns c .. of a row (runs of 8 columns are contiguous in both layouts)
__device__ inline int64_t act_offset(int layout, int row, int c, int d)
{
    return layout == LAYOUT_TILED ? tiled_offset(row, c, d >> 6) : (int64_t)row * d + c;
}

// v[t][:] = pre[t][:] (+ bias[:]) (+ resid[t][:]);  y[t][:] = LayerNorm(v) * g + b.
// One wave per row; two-pass mean / variance in float32.  General sizes.
template <int DT, typename RT>   // RT: type of the residual rows
__global__ __launch_bounds__(256) void layernorm_kernel(const float *pre, int n_partials,
                                                        int64_t partial_stride, const float *bias,
                                                        const RT *resid, int resid_layout, int y_layout,
                                                        typename Elem<DT>::type *y, const float *g,
                                                        const float *b, int T, int d, float eps)
{
    const int row = blockIdx.x * 4 + threadIdx.x / 64;
    const int lane = threadIdx.x % 64;
    if (row >= T) return;
    const float *r = pre + (int64_t)row * d;
    auto value = [&](int c) {
        float v = n_partials > 0 ? r[c] : 0.f;
        for (int s = 1; s < n_partials; ++s) v += r[(int64_t)s * partial_stride + c];
        if (bias) v += bias[c];
        if (resid) v += (float)resid[act_offset(resid_layout, row, c, d)];
        return v;
    };
    float s = 0.f;
    for (int c = lane; c < d; c += 64) s += value(c);
    const float mean = lane_sum<64>(s) / (float)d;
    float q = 0.f;
    for (int c = lane; c < d; c += 64) {
        float t = value(c) - mean;
        q = fmaf(t, t, q);
    }
    const float var = lane_sum<64>(q) / (float)d;
    const float inv = 1.0f / sqrtf(var + eps);
    for (int c = lane; c < d; c += 64)
        Elem<DT>::store(y + act_offset(y_layout, row, c, d), (value(c) - mean) * inv * g[c] + b[c]);
}

// Same, for d a multiple of 4 and at most 2048: the row is read once with 16-byte loads
// and kept in registers.
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));

// sum / d as a division rounds it, in a third of the dependent instructions: inv_d is 1 / d in float64, and the quotient of a float32 by an
// integer of d's size is never as close to a rounding boundary as that product is off.  (A product with a float32 1 / d is: the mean of equal
// values came out beside them at d_model 448, 832, 896 and 960, far enough for an eps of 1e-12.)  24 layers of d_model 1024, 256
// tokens, us: 991, divisions 999.
__device__ inline float row_quotient(float sum, double inv_d) { return (float)((double)sum * inv_d); }

// LPR lanes share one row.  TILED: one of the layouts is; MAXC = 16-byte chunks per lane: d <= 4 * LPR * MAXC; PLANES: partial sums
// requested together; ROWS: rows per workgroup.
// Few rows: bound by latency (the launch, one round trip, two sums over the row).  The leading 14 dwords of the arguments arrive preloaded
// in scalar registers: everything the requests of a row depend on, but for the distance of the second and later planes of partial sums.
// shape: n_partials | resid_layout << 8 | y_layout << 16.
// (A function that the kernels inline, not a kernel's own body: that was compiled with a wait for everything behind each of a tiled row's first
// three bias requests, three round trips ahead of the sums'.  256 tokens of d_model 1024, us per launch: one plane 4.3, now 3.3, several planes
// 4.7 / 4.0; 24 layers 988 / 948.)
template <int DT, typename RT, bool TILED, int LPR, int MAXC, int PLANES, int ROWS>
__device__ __forceinline__ void layernorm_rows(const float *pre, const float *bias, const RT *resid, const float *g,
                                                            const float *b, int T, int d, int shape, float eps, int64_t partial_stride,
                                                            typename Elem<DT>::type *y, uint16_t *planes, double inv_d)
{
    const int n_partials = shape & 0xff, resid_layout = shape >> 8 & 0xff, y_layout = shape >> 16;
    const int sub = threadIdx.x % LPR;
    int row = blockIdx.x * ROWS + threadIdx.x / LPR;
    // A cache line of a tiled matrix holds 16 bytes of each of eight rows: such rows go to workgroups of one XCD (workgroups are handed
    // to the eight XCDs in turn), where they meet in its L2.  12 layers, us: BERT-base 512 tokens 525 -> 501, d_model 1024 384 tokens
    // 618 -> 604; 128 tokens and fewer: the same.
    if constexpr (TILED && ROWS == 1) row = ((blockIdx.x >> 6) * 8 + (blockIdx.x & 7)) * 8 + (blockIdx.x >> 3 & 7);
    if (row >= T) return;   // whole row groups leave together; shuffles stay inside a group
    const int nchunk = d >> 2;
    // Every load of this row is independent of the others: they are issued in groups (bias and
    // residual first, then the partial sums PLANES planes at a time) and only then added, in the
    // fixed order plane 0, 1, ..., bias, residual.  (Written as load-then-use per chunk, each of
    // up to 8 planes x 8 chunks cost a round trip to memory of its own.)  Lanes past the end of
    // the row load its last chunk and drop the value.
    const int last = nchunk - 1;
    int cj[MAXC];
#pragma unroll
    for (int j = 0; j < MAXC; ++j) cj[j] = min(sub + LPR * j, last);
    typedef RT resid4 __attribute__((ext_vector_type(4)));
    f32x4 bs[MAXC];
    resid4 rs4[MAXC];
#pragma unroll
    for (int j = 0; j < MAXC; ++j) {
        bs[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        rs4[j] = resid4{(RT)0.f, (RT)0.f, (RT)0.f, (RT)0.f};
        if (bias) bs[j] = ((const f32x4 *)bias)[cj[j]];
        if (resid) rs4[j] = *(const resid4 *)(resid + act_offset(TILED ? resid_layout : LAYOUT_ROWS, row, 4 * cj[j], d));
    }
    f32x4 gg[MAXC], bb[MAXC];
#pragma unroll
    for (int j = 0; j < MAXC; ++j) {
        gg[j] = ((const f32x4 *)g)[cj[j]];
        bb[j] = ((const f32x4 *)b)[cj[j]];
    }
    f32x4 v[MAXC];
#pragma unroll
    for (int j = 0; j < MAXC; ++j) v[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const float *rp = pre + (int64_t)row * d;
    for (int sp = 0; sp < n_partials; sp += PLANES) {
        f32x4 t[PLANES][MAXC];
#pragma unroll
        for (int k = 0; k < PLANES; ++k) {   // (planes past the last one: that one again, not added)
            const int64_t plane = (int64_t)(PLANES > 1 ? min(sp + k, n_partials - 1) : sp) * partial_stride;
#pragma unroll
            for (int j = 0; j < MAXC; ++j) t[k][j] = *(const f32x4 *)(rp + plane + 4 * cj[j]);
        }
#pragma unroll
        for (int k = 0; k < PLANES; ++k) {
            if (sp + k < n_partials) {       // uniform
#pragma unroll
                for (int j = 0; j < MAXC; ++j) v[j] = sp + k == 0 ? t[k][j] : v[j] + t[k][j];
            }
        }
    }
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < MAXC; ++j) {
        f32x4 x = v[j];
        if (bias) x += bs[j];
        if (resid) x += f32x4{(float)rs4[j].x, (float)rs4[j].y, (float)rs4[j].z, (float)rs4[j].w};
        if (sub + LPR * j >= nchunk) x = f32x4{0.f, 0.f, 0.f, 0.f};
        v[j] = x;
        s += (x.x + x.y) + (x.z + x.w);
    }
    const float mean = row_quotient(lane_sum<LPR>(s), inv_d);
    float q = 0.f;
#pragma unroll
    for (int j = 0; j < MAXC; ++j) {
        if (sub + LPR * j < nchunk) {
            f32x4 t = v[j] - mean;
            q += (t.x * t.x + t.y * t.y) + (t.z * t.z + t.w * t.w);
        }
    }
    const float var = row_quotient(lane_sum<LPR>(q), inv_d);
    const float inv = 1.0f / sqrtf(var + eps);
#pragma unroll
    for (int j = 0; j < MAXC; ++j) {
        const int c = sub + LPR * j;
        typename Elem<DT>::type *o = y + act_offset(TILED ? y_layout : LAYOUT_ROWS, row, 4 * c, d);
        if (c < nchunk) {
            const f32x4 t = (v[j] - mean) * inv * gg[j] + bb[j];
            if constexpr (DT == STI_F32) {
                *(f32x4 *)o = t;
                if constexpr (std::is_same<RT, float>::value) {
                    if (planes) store_planes4(planes, row, 4 * c, d >> 6, t);
                }
            } else if constexpr (DT == STI_F16) {
                *(half4 *)o = half4{(_Float16)t.x, (_Float16)t.y, (_Float16)t.z, (_Float16)t.w};
            } else {
                Elem<DT>::store(o, t.x); Elem<DT>::store(o + 1, t.y);
                Elem<DT>::store(o + 2, t.z); Elem<DT>::store(o + 3, t.w);
            }
        }
    }
}
template <int DT, typename RT, bool TILED, int LPR, int MAXC, int PLANES, int ROWS>
__global__ __launch_bounds__(LPR * ROWS) void layernorm_vec_kernel(const float *pre, const float *bias, const RT *resid, const float *g,
                                                            const float *b, int T, int d, int shape, float eps, int64_t partial_stride,
                                                            typename Elem<DT>::type *y, uint16_t *planes, double inv_d)
{
    layernorm_rows<DT, RT, TILED, LPR, MAXC, PLANES, ROWS>(pre, bias, resid, g, b, T, d, shape, eps, partial_stride, y, planes, inv_d);
}

// The same with planes (float32 layers on the bfloat16 matrix cores) and, in the workgroups behind those of the rows, the decompression of
// the weights that the launches to come multiply with: FFN1 and FFN2 beside the first LayerNorm of a layer, the next layer's Q, K, V and O beside
// the second.  LayerNorm waits for its rows while the decompression writes.  8 x 128 tokens of BERT-base, 12 layers: 1723 -> 1627 us, 4 x 128
// tokens 1262 -> 1172.
template <int MAXC, int PLANES, typename Table>
__global__ __launch_bounds__(256) void layernorm_decode_kernel(const float *pre, const float *bias, const float *resid, const float *g, const float *b, int T, int d,
                                                              int shape, float eps, int64_t partial_stride, float *y, uint16_t *planes, double inv_d,
                                                              SplitDecodeJob job, Table tab)
{
    __shared__ u32x2 lut[4][kLutEntries];
    const int ahead = (T + 3) / 4;
    if ((int)blockIdx.x < ahead) layernorm_rows<STI_F32, float, false, 64, MAXC, PLANES, 4>(pre, bias, resid, g, b, T, d, shape, eps, partial_stride, y, planes, inv_d);
    else decode_split_block(job, tab, (int)blockIdx.x - ahead, lut);
}


// LayerNorm of rows that already hold sum + bias + residual in binary16 (written by the
// matrix-core GEMM); d a multiple of 8 and at most 8 * LPR * MAXC; LPR lanes per row.  All
// loads (the row, gains, shifts) are issued before the first use: one round trip to memory.
// Lanes past the end of the row load its last chunk and drop the value.
template <int DT, int LPR, int MAXC>
__global__ __launch_bounds__(256) void layernorm_f16in_kernel(const _Float16 *pre,
                                                              typename Elem<DT>::type *y,
                                                              const float *g, const float *b, int T,
                                                              int d, float eps, double inv_d)
{
    typedef _Float16 half8 __attribute__((ext_vector_type(8)));
    constexpr int ROWS = 256 / LPR;
    const int sub = threadIdx.x % LPR;
    const int row = blockIdx.x * ROWS + threadIdx.x / LPR;
    if (row >= T) return;   // whole row groups leave together; shuffles stay inside a group
    const int nchunk = d >> 3, last = nchunk - 1;
    const half8 *r = (const half8 *)(pre + (int64_t)row * d);
    half8 h[MAXC];
    f32x4 g0[MAXC], g1[MAXC], b0[MAXC], b1[MAXC];
#pragma unroll
    for (int j = 0; j < MAXC; ++j) h[j] = r[min(sub + LPR * j, last)];
#pragma unroll
    for (int j = 0; j < MAXC; ++j) {
        const int c = min(sub + LPR * j, last);
        g0[j] = ((const f32x4 *)g)[2 * c]; g1[j] = ((const f32x4 *)g)[2 * c + 1];
        b0[j] = ((const f32x4 *)b)[2 * c]; b1[j] = ((const f32x4 *)b)[2 * c + 1];
    }
    float v[MAXC][8];
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < MAXC; ++j) {
        const bool in = sub + LPR * j < nchunk;
#pragma unroll
        for (int e = 0; e < 8; ++e) { v[j][e] = in ? (float)h[j][e] : 0.f; s += v[j][e]; }
    }
    const float mean = row_quotient(lane_sum<LPR>(s), inv_d);
    float q = 0.f;
#pragma unroll
    for (int j = 0; j < MAXC; ++j)
        if (sub + LPR * j < nchunk) {
#pragma unroll
            for (int e = 0; e < 8; ++e) { const float t = v[j][e] - mean; q = fmaf(t, t, q); }
        }
    const float var = row_quotient(lane_sum<LPR>(q), inv_d);
    const float inv = 1.0f / sqrtf(var + eps);
    typename Elem<DT>::type *o = y + (int64_t)row * d;
#pragma unroll
    for (int j = 0; j < MAXC; ++j) {
        const int c = sub + LPR * j;
        if (c < nchunk) {
            const float gg[8] = {g0[j].x, g0[j].y, g0[j].z, g0[j].w, g1[j].x, g1[j].y, g1[j].z, g1[j].w};
            const float bb[8] = {b0[j].x, b0[j].y, b0[j].z, b0[j].w, b1[j].x, b1[j].y, b1[j].z, b1[j].w};
            float t[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) t[e] = (v[j][e] - mean) * inv * gg[e] + bb[e];
            if constexpr (DT == STI_F16) {
                half8 o8;
#pragma unroll
                for (int e = 0; e < 8; ++e) o8[e] = (_Float16)t[e];
                ((half8 *)o)[c] = o8;
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) Elem<DT>::store(o + 8 * c + e, t[e]);
            }
        }
    }
}

// Same for rows of any length (d a multiple of 8): the row is read three times (mean, variance,
// output) instead of being kept in registers.
template <int DT>
__global__ __launch_bounds__(256) void layernorm_f16in_long_kernel(const _Float16 *pre,
                                                                   typename Elem<DT>::type *y,
                                                                   const float *g, const float *b, int T,
                                                                   int d, float eps)
{
    typedef _Float16 half8 __attribute__((ext_vector_type(8)));
    const int lane = threadIdx.x % 64;
    const int row = blockIdx.x * 4 + threadIdx.x / 64;
    if (row >= T) return;
    const int nchunk = d >> 3;
    const half8 *r = (const half8 *)(pre + (int64_t)row * d);
    float s = 0.f;
    for (int c = lane; c < nchunk; c += 64) {
        const half8 h = r[c];
#pragma unroll
        for (int e = 0; e < 8; ++e) s += (float)h[e];
    }
    const float mean = lane_sum<64>(s) / (float)d;
    float q = 0.f;
    for (int c = lane; c < nchunk; c += 64) {
        const half8 h = r[c];
#pragma unroll
        for (int e = 0; e < 8; ++e) { const float t = (float)h[e] - mean; q = fmaf(t, t, q); }
    }
    const float inv = 1.0f / sqrtf(lane_sum<64>(q) / (float)d + eps);
    typename Elem<DT>::type *o = y + (int64_t)row * d;
    for (int c = lane; c < nchunk; c += 64) {
        const half8 h = r[c];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            Elem<DT>::store(o + 8 * c + e, ((float)h[e] - mean) * inv * g[8 * c + e] + b[8 * c + e]);
    }
}

template <int SRC, int DST>
__global__ __launch_bounds__(256) void convert_kernel(const typename Elem<SRC>::type *src,
                                                      typename Elem<DST>::type *dst, uint64_t n)
{
    uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    const uint64_t stride = (uint64_t)gridDim.x * 256;
    for (; i < n; i += stride) Elem<DST>::store(dst + i, Elem<SRC>::load(src + i));
}

template <int SRC>
hipError_t convert_from(const void *src, void *dst, sti_dtype dst_dtype, uint64_t n, dim3 grid,
                        hipStream_t stream)
{
    typedef typename Elem<SRC>::type S;
    switch (dst_dtype) {
        case STI_F32:
            launch((convert_kernel<SRC, STI_F32>), grid, dim3(256), 0, stream, (const S *)src, (float *)dst, n);
            break;
        case STI_F16:
            launch((convert_kernel<SRC, STI_F16>), grid, dim3(256), 0, stream, (const S *)src, (_Float16 *)dst, n);
            break;
        case STI_BF16:
            launch((convert_kernel<SRC, STI_BF16>), grid, dim3(256), 0, stream, (const S *)src, (uint16_t *)dst, n);
            break;
    }
    return hipGetLastError();
}

}  // namespace

template <int DT, typename RT, bool TILED>
void launch_ln_typed(const float *pre, int n_partials, int64_t partial_stride, const float *bias,
                     const void *resid, ActLayout resid_layout, ActLayout y_layout, void *y, const float *g, const float *b,
                     int T, int d, float eps, bool vec, hipStream_t stream, uint16_t *planes, const SplitRide *ride)
{
    typedef typename Elem<DT>::type O;
#define STI_LN_PLANES(LPR, MAXC, PLANES, ROWS) \
    launch((layernorm_vec_kernel<DT, RT, TILED, LPR, MAXC, PLANES, ROWS>), dim3(TILED && ROWS == 1 ? (T + 63) / 64 * 64 : (T + ROWS - 1) / ROWS), dim3(LPR * ROWS), 0, stream, pre, \
           bias, (const RT *)resid, g, b, T, d, n_partials | (int)resid_layout << 8 | (int)y_layout << 16, eps, partial_stride, (O *)y, planes, 1.0 / d)
#define STI_LN_VEC(LPR, MAXC, ROWS)                                       \
    do {                                                                  \
        if (n_partials <= 1) STI_LN_PLANES(LPR, MAXC, 1, ROWS);           \
        else if (n_partials == 2) STI_LN_PLANES(LPR, MAXC, 2, ROWS);      \
        else STI_LN_PLANES(LPR, MAXC, 4, ROWS);                           \
    } while (0)
    // many rows: 32 lanes per row (8 rows per workgroup); few rows: a wave and a workgroup per row, so that the rows spread
    // over as many compute units as there are; chunks per lane sized to the row, so that the registers hold no more
    // loads in flight than it has
    if (!TILED && vec && !planes && T >= 2048 && d <= 1024) {   // (tiled: at most kFewMaxTokens rows)
        if constexpr (!TILED) {
            if (d <= 768) STI_LN_VEC(32, 6, 8);
            else STI_LN_VEC(32, 8, 8);
        }
    } else if (vec && planes) {
        if constexpr (DT == STI_F32 && std::is_same<RT, float>::value) {
            SplitDecodeJob job;
            if (ride && split_decode_job(ride->n_shards, d, ride->d_head, ride->ffn_per_shard, ride->ffn, ride->out, &job)) {
                with_inline_table(*ride->table, ride->n_shards, [&](auto t) {
#define STI_LN_RIDE(MAXC, PLANES) \
    launch((layernorm_decode_kernel<MAXC, PLANES, decltype(t)>), dim3((uint32_t)((T + 3) / 4 + (job.cells + 3) / 4)), dim3(256), 0, stream, pre, bias, (const float *)resid, g, b, \
           T, d, n_partials | (int)resid_layout << 8 | (int)y_layout << 16, eps, partial_stride, (float *)y, planes, 1.0 / d, job, t)
#define STI_LN_RIDES(MAXC)                              \
    do {                                                \
        if (n_partials <= 1) STI_LN_RIDE(MAXC, 1);      \
        else if (n_partials == 2) STI_LN_RIDE(MAXC, 2); \
        else STI_LN_RIDE(MAXC, 4);                      \
    } while (0)
                    if (d <= 768) STI_LN_RIDES(3);
                    else STI_LN_RIDES(4);
#undef STI_LN_RIDES
#undef STI_LN_RIDE
                });
                return;
            }
            if (d <= 768) STI_LN_VEC(64, 3, 4);
            else if (d <= 1024) STI_LN_VEC(64, 4, 4);
            else STI_LN_VEC(64, 8, 4);
        }
    } else if (vec) {
        if (d <= 768) STI_LN_VEC(64, 3, 1);
        else if (d <= 1024) STI_LN_VEC(64, 4, 1);
        else STI_LN_VEC(64, 8, 1);
    } else {
        launch((layernorm_kernel<DT, RT>), dim3((T + 3) / 4), dim3(256), 0, stream, pre, n_partials, partial_stride, bias, (const RT *)resid, (int)resid_layout, (int)y_layout, (O *)y, g, b, T, d, eps);
    }
#undef STI_LN_VEC
#undef STI_LN_PLANES
}

bool layernorm_reads_wide(const float *pre, int64_t partial_stride, const float *bias, const void *resid, const void *y, const float *g, const float *b, int d)
{
    auto al16 = [](const void *p) { return ((uintptr_t)p & 15) == 0; };
    return d % 4 == 0 && d <= 2048 && partial_stride % 4 == 0 && al16(pre) && al16(g) && al16(b) && al16(y) && (!bias || al16(bias)) &&
           (!resid || al16(resid));
}

hipError_t launch_layernorm(const float *pre, int n_partials, int64_t partial_stride,
                            const float *bias, const void *resid, bool resid_f32, ActLayout resid_layout, void *y,
                            sti_dtype out_dtype, ActLayout y_layout,
                            const float *g, const float *b, int T, int d, float eps,
                            hipStream_t stream, void *planes, const SplitRide *ride)
{
    if (T <= 0 || d <= 0) return hipSuccess;
    const bool vec = layernorm_reads_wide(pre, partial_stride, bias, resid, y, g, b, d);
    if (planes && (!vec || d % 64 || !resid_f32 || out_dtype != STI_F32)) return hipErrorInvalidValue;
    SplitDecodeJob job;
    if (ride && (!planes || d > kRideFeatures || !split_decode_job(ride->n_shards, d, ride->d_head, ride->ffn_per_shard, ride->ffn, ride->out, &job))) return hipErrorInvalidValue;
    if (n_partials < 0 || n_partials > 255 || (n_partials > 0 && !pre)) return hipErrorInvalidValue;
    if ((resid_layout == LAYOUT_TILED || y_layout == LAYOUT_TILED) && (d % 64 || (resid_f32 && (resid_layout == LAYOUT_TILED || out_dtype != STI_F16))))
        return hipErrorInvalidValue;
    auto go = [&](auto resid_type, auto tiled) {
        typedef decltype(resid_type) RT;
        constexpr bool TL = decltype(tiled)::value;
        switch (out_dtype) {
            case STI_F32: launch_ln_typed<STI_F32, RT, TL>(pre, n_partials, partial_stride, bias, resid, resid_layout, y_layout, y, g, b, T, d, eps, vec, stream, (uint16_t *)planes, ride); break;
            case STI_F16: launch_ln_typed<STI_F16, RT, TL>(pre, n_partials, partial_stride, bias, resid, resid_layout, y_layout, y, g, b, T, d, eps, vec, stream, (uint16_t *)planes, ride); break;
            case STI_BF16: launch_ln_typed<STI_BF16, RT, TL>(pre, n_partials, partial_stride, bias, resid, resid_layout, y_layout, y, g, b, T, d, eps, vec, stream, (uint16_t *)planes, ride); break;
        }
    };
    if (resid_f32 && y_layout == LAYOUT_TILED)
        launch_ln_typed<STI_F16, float, true>(pre, n_partials, partial_stride, bias, resid, LAYOUT_ROWS, y_layout, y, g, b, T, d, eps, vec, stream, nullptr, nullptr);
    else if (resid_f32) go(float{}, std::false_type{});
    else if (resid_layout == LAYOUT_TILED || y_layout == LAYOUT_TILED) go(_Float16{}, std::true_type{});
    else go(_Float16{}, std::false_type{});
    return hipGetLastError();
}

hipError_t launch_layernorm_f16in(const void *pre_f16, void *y, sti_dtype out_dtype, const float *g,
                                  const float *b, int T, int d, float eps, hipStream_t stream)
{
    if (T <= 0 || d <= 0) return hipSuccess;
    if (d % 8) return hipErrorInvalidValue;
    dim3 grid((T + 3) / 4);
    const _Float16 *p = (const _Float16 *)pre_f16;
    if (d > 2048) {
        switch (out_dtype) {
            case STI_F32: launch((layernorm_f16in_long_kernel<STI_F32>), grid, dim3(256), 0, stream, p, (float *)y, g, b, T, d, eps); break;
            case STI_F16: launch((layernorm_f16in_long_kernel<STI_F16>), grid, dim3(256), 0, stream, p, (_Float16 *)y, g, b, T, d, eps); break;
            case STI_BF16: launch((layernorm_f16in_long_kernel<STI_BF16>), grid, dim3(256), 0, stream, p, (uint16_t *)y, g, b, T, d, eps); break;
        }
        return hipGetLastError();
    }
    // 32 lanes per row while the row fits 3 or 4 chunks of 8 per lane (every lane busy at d_model 768
    // and 1024), a whole wave per row beyond
    auto go = [&](auto dt) {
        constexpr int DT = decltype(dt)::value;
        typedef typename Elem<DT>::type O;
        if (d <= 768)
            launch((layernorm_f16in_kernel<DT, 32, 3>), dim3((T + 7) / 8), dim3(256), 0, stream, p, (O *)y, g, b, T, d, eps, 1.0 / d);
        else if (d <= 1024)
            launch((layernorm_f16in_kernel<DT, 32, 4>), dim3((T + 7) / 8), dim3(256), 0, stream, p, (O *)y, g, b, T, d, eps, 1.0 / d);
        else
            launch((layernorm_f16in_kernel<DT, 64, 4>), dim3((T + 3) / 4), dim3(256), 0, stream, p, (O *)y, g, b, T, d, eps, 1.0 / d);
    };
    switch (out_dtype) {
        case STI_F32: go(std::integral_constant<int, STI_F32>{}); break;
        case STI_F16: go(std::integral_constant<int, STI_F16>{}); break;
        case STI_BF16: go(std::integral_constant<int, STI_BF16>{}); break;
    }
    return hipGetLastError();
}

// Rows to tiled binary16: a thread takes 8 consecutive columns, consecutive threads the rows of a
// 32-row block first, so that a wave's store is one contiguous fragment.
namespace {

template <int SRC>
__global__ __launch_bounds__(256) void tile_rows_kernel(const typename Elem<SRC>::type *src, _Float16 *dst, int T, int d)
{
    typedef _Float16 half8 __attribute__((ext_vector_type(8)));
    const int chunks = d >> 3, i = blockIdx.x * 256 + threadIdx.x;
    const int row = i / (32 * chunks) * 32 + i % 32, c = i / 32 % chunks * 8;
    if (row >= T) return;
    const typename Elem<SRC>::type *p = src + (int64_t)row * d + c;
    half8 h;
#pragma unroll
    for (int e = 0; e < 8; ++e) h[e] = (_Float16)Elem<SRC>::load(p + e);
    *(half8 *)(dst + tiled_offset(row, c, d >> 6)) = h;
}

}  // namespace

hipError_t launch_tile_rows(const void *src, sti_dtype src_dtype, void *dst, int T, int d, hipStream_t stream)
{
    if (T <= 0 || d <= 0) return hipSuccess;
    if (d % 64) return hipErrorInvalidValue;
    const int64_t threads = (int64_t)((T + 31) / 32) * 32 * (d / 8);
    if (threads > 0x7FFFFF00) return hipErrorInvalidValue;
    const dim3 grid((uint32_t)((threads + 255) / 256));
    switch (src_dtype) {
        case STI_F32: launch((tile_rows_kernel<STI_F32>), grid, dim3(256), 0, stream, (const float *)src, (_Float16 *)dst, T, d); break;
        case STI_F16: launch((tile_rows_kernel<STI_F16>), grid, dim3(256), 0, stream, (const _Float16 *)src, (_Float16 *)dst, T, d); break;
        case STI_BF16: launch((tile_rows_kernel<STI_BF16>), grid, dim3(256), 0, stream, (const uint16_t *)src, (_Float16 *)dst, T, d); break;
    }
    return hipGetLastError();
}

hipError_t launch_convert(const void *src, sti_dtype src_dtype, void *dst, sti_dtype dst_dtype,
                          uint64_t n, hipStream_t stream)
{
    if (n == 0) return hipSuccess;
    uint64_t blocks = (n + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    dim3 grid((uint32_t)blocks);
    switch (src_dtype) {
        case STI_F32: return convert_from<STI_F32>(src, dst, dst_dtype, n, grid, stream);
        case STI_F16: return convert_from<STI_F16>(src, dst, dst_dtype, n, grid, stream);
        case STI_BF16: return convert_from<STI_BF16>(src, dst, dst_dtype, n, grid, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace sti
