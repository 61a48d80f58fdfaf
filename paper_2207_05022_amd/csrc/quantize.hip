// Outlier-aware quantization of one layer's shards into a k-bit version (Section
// "quantization per shard"; Section "Implementation", preprocessing): a single Gaussian is
// fitted to all weights of the layer, weights whose log likelihood is below a threshold are
// outliers, the others are cut into 2^k clusters of equal population (by sorted rank), each
// cluster's centroid is the mean of its members, and every weight becomes the k-bit index of
// its cluster; outliers keep a placeholder index and are bookkept with offset and value.
//
// No sort is needed for equal-population clusters: only the 2^k - 1 boundary values are.  Four passes
// stream the layer, each with a workgroup per compute unit and results of its own per workgroup:
//   moments -> histogram of the inliers over 4096 equal bins of their value range, outliers per 512 weights
//   -> (merge) -> ranks -> boundary bins, values of those into one list per bin
//   -> (boundary values: radix selection inside a list) -> cluster indexes: packed streams, outlier
//   dictionaries and sums per cluster -> (centroids).
// The steps in brackets are small kernels in between.  Every result is independent of the order in
// which workgroups and lanes run: counts are integers, the moments are added in a fixed order in float64, and the
// sums of a workgroup are 64-bit integers (weights scaled by a power of two) that hold every weight exactly.
//
// Infinite and NaN weights (the moments are NaN then, so that nothing is an outlier) take the general ways through
// the same kernels: one bin for all weights, clusters by comparison of keys, sums beside the integers.
//
// What bounds it: seven dependent launches, and in the streaming passes the LDS (a look-up and an atomic per weight, 3.4 units of 512
// weights per wave) behind what each works out before its first weight: 6500 clocks of the histogram pass (the Gaussian), 3800 of the
// collecting pass.  More units on their way at once change nothing.  BERT-base at 4 bits: 48 us, 54 with the boundary bins looked up by one
// wave, the atomics behind the weights and up to three rounds for a boundary value; d_model 384, 3 bits 36.9 -> 30.5.
#include "api_internal.hpp"
#include "lane_ops.hpp"

namespace sti {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kUnit = 512;          // weights a wave takes at a time
constexpr int kThreads = 1024;      // workgroups of the streaming passes
constexpr int kWaves = kThreads / 64;
constexpr int kMaxClusters = 64;
constexpr int kBins = 4096;
constexpr int kGroups = 256;        // workgroups of a streaming pass, as long as ...
constexpr int kGroupUnits = 112;    // ... each sees at most this many units (57344 weights: 16-bit counters)
constexpr int kMomentGroups = 512;
constexpr uint64_t kGranule = 1024; // weights per shard are a multiple of this

// What a layer's kernels pass on.
struct QuantState {
    double mu, var;
    float xlo, xhi;                 // inliers are the weights in [xlo, xhi]
    float bin_scale, bin_shift;     // bin of x: (int)(x * scale + shift), clamped to 0 .. kBins - 1
    int sum_exp;                    // |inlier| < 2^sum_exp
    uint32_t non_finite;            // some weight is infinite or NaN
    unsigned long long n_inliers;
    uint32_t error;                 // 1: no inliers
    uint32_t slot_fill[kMaxClusters];            // list entries taken so far
    // boundary c = 1 .. C-1 at [c-1]: the lowest member of cluster c
    unsigned long long edge_begin[kMaxClusters];                 // its bin's list
    uint32_t edge_count[kMaxClusters], edge_rank[kMaxClusters];  // ... and the rank inside it
    unsigned long long edge_before[kMaxClusters];                // inliers in lower bins
    uint32_t edge_key[kMaxClusters];
    unsigned long long edge_below[kMaxClusters];                 // inliers below the boundary value
};

struct QuantLayout {
    size_t state, partials, unit_count, unit_off, shard_count, hist_part, hist, table, lists, csum, total;
    int groups;
};

int stream_groups(uint64_t n)
{
    const uint64_t units = n / kUnit;
    uint64_t g = (units + kWaves - 1) / kWaves;
    if (g > kGroups) g = kGroups;
    const uint64_t least = (units + kGroupUnits - 1) / kGroupUnits;
    return (int)(g < least ? least : g);
}

QuantLayout quant_layout(uint64_t n)
{
    QuantLayout L;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t at = off; off = align_up(off + bytes, 256); return at; };
    L.groups = stream_groups(n);
    L.state = take(sizeof(QuantState));
    L.partials = take((size_t)kMomentGroups * 3 * sizeof(double));
    L.unit_count = take((size_t)(n / kUnit) * 4);
    L.unit_off = take((size_t)(n / kUnit) * 4);
    L.shard_count = take((size_t)kMaxShardsPerLayer * 4);
    L.hist_part = take((size_t)L.groups * kBins * 2);
    L.hist = take((size_t)kBins * 4);
    L.table = take((size_t)kBins * 2);
    L.lists = take((size_t)n * 4);
    L.csum = take((size_t)L.groups * kMaxClusters * sizeof(double));
    L.total = off;
    return L;
}

// order-preserving image of a float (-0.0 counted as +0.0)
__device__ inline uint32_t order_key(float x)
{
    const uint32_t u = __builtin_bit_cast(uint32_t, x + 0.0f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ inline float key_value(uint32_t k)
{
    const uint32_t u = (k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k;
    return __builtin_bit_cast(float, u);
}

// monotone in x: a product-sum with a non-negative factor, rounded once, clamped and truncated
__device__ inline int bin_of(float x, float scale, float shift)
{
    return (int)__builtin_amdgcn_fmed3f(fmaf(x, scale, shift), 0.0f, (float)(kBins - 1));
}

__device__ inline double wave_sum_f64(double v)   // (in lane 0)
{
    return lane_tree(v, [](double a, double b) { return a + b; });
}
__device__ inline double wave_max_f64(double v)   // (in lane 0; of values that are not negative, or NaN)
{
    return lane_tree(v, [](double a, double b) { return fmax(a, b); });
}

// per workgroup: sum, sum of squares (float64, fixed order), largest magnitude
__global__ __launch_bounds__(256) void moments_kernel(const float *w, uint64_t n, double *partials)
{
    __shared__ double lds[4][3];
    double s0 = 0.0, s1 = 0.0, q0 = 0.0, q1 = 0.0;
    float mx = 0.0f;
    const uint64_t n4 = n / 4, step = (uint64_t)gridDim.x * 256;
    uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    auto add = [&](f32x4 v) {
        const double a = v[0], b = v[1], c = v[2], d = v[3];
        s0 += a; s1 += b; q0 += a * a; q1 += b * b;
        s0 += c; s1 += d; q0 += c * c; q1 += d * d;
        mx = fmaxf(fmaxf(mx, fmaxf(fabsf(v[0]), fabsf(v[1]))), fmaxf(fabsf(v[2]), fabsf(v[3])));
    };
    for (; i + 3 * step < n4; i += 4 * step) {
        const f32x4 a = ((const f32x4 *)w)[i], b = ((const f32x4 *)w)[i + step], c = ((const f32x4 *)w)[i + 2 * step],
                    d = ((const f32x4 *)w)[i + 3 * step];
        add(a); add(b); add(c); add(d);
    }
    for (; i < n4; i += step) add(((const f32x4 *)w)[i]);
    const double s = wave_sum_f64(s0 + s1), q = wave_sum_f64(q0 + q1);
    mx = (float)wave_max_f64((double)mx);
    if ((threadIdx.x & 63) == 0) {
        lds[threadIdx.x >> 6][0] = s;
        lds[threadIdx.x >> 6][1] = q;
        lds[threadIdx.x >> 6][2] = mx;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        partials[3 * blockIdx.x] = lds[0][0] + lds[1][0] + lds[2][0] + lds[3][0];
        partials[3 * blockIdx.x + 1] = lds[0][1] + lds[1][1] + lds[2][1] + lds[3][1];
        partials[3 * blockIdx.x + 2] = fmax(fmax(lds[0][2], lds[1][2]), fmax(lds[2][2], lds[3][2]));
    }
}

// What every workgroup of the histogram pass works out for itself from the partial moments (all get the same).
struct Fit {
    double mu, var;
    float xlo, xhi, bin_scale, bin_shift;
    int sum_exp;
    uint32_t non_finite;
};

// (NaN weights, whose Gaussian has a NaN mean and no bounds, are inliers)
__device__ inline bool is_inlier(float x, float xlo, float xhi) { return !(x < xlo || x > xhi); }

__device__ inline Fit fit_gaussian(double ts, double tss, float largest, uint64_t n, double threshold, double reg_covar)
{
    Fit f;
    f.mu = ts / (double)n;
    f.var = tss / (double)n - f.mu * f.mu + reg_covar;
    // log N(x; mu, var) < threshold  <=>  (x - mu)^2 > 2 var (-threshold - log sqrt(2 pi var)); the squared distance,
    // rounded, grows with |x - mu|, so the inliers are the floats of one interval, whose ends are found
    // from the rounded ones in a few steps
    const double r2 = 2.0 * f.var * (-threshold - 0.5 * log(2.0 * 3.14159265358979323846 * f.var));
    auto outlier = [&](float x) { const double d = (double)x - f.mu; return d * d > r2; };
    const double r = sqrt(r2);
    if (r2 < 0.0) {
        f.xlo = INFINITY; f.xhi = -INFINITY;
    } else if (!(f.mu + r < 3.0e38 && f.mu - r > -3.0e38)) {   // (no bound that a float reaches, or none at all)
        f.xlo = -INFINITY; f.xhi = INFINITY;
    } else {
        uint32_t hi = order_key((float)(f.mu + r)), lo = order_key((float)(f.mu - r));
        for (int i = 0; i < 8 && outlier(key_value(hi)); ++i) --hi;
        for (int i = 0; i < 8 && !outlier(key_value(hi + 1)); ++i) ++hi;
        for (int i = 0; i < 8 && outlier(key_value(lo)); ++i) ++lo;
        for (int i = 0; i < 8 && !outlier(key_value(lo - 1)); ++i) --lo;
        f.xhi = key_value(hi);
        f.xlo = key_value(lo);
        if (outlier(f.xhi) || outlier(f.xlo)) { f.xlo = INFINITY; f.xhi = -INFINITY; }   // (no float lies inside)
    }
    const float lo = fmaxf(f.xlo, -largest), hi = fminf(f.xhi, largest);
    f.bin_scale = 0.0f;   // (every weight in bin 0)
    f.bin_shift = 0.0f;
    f.non_finite = !(fabs(ts) < INFINITY);
    if (hi > lo && !f.non_finite) {
        const float scale = (float)kBins / (hi - lo);
        if (scale < 1.0e30f && fabsf(lo * scale) < 1.0e30f) { f.bin_scale = scale; f.bin_shift = -lo * scale; }
    }
    int e = 0;
    (void)frexp((double)fmaxf(fabsf(lo), fabsf(hi)), &e);      // largest inlier magnitude < 2^e
    f.sum_exp = f.non_finite ? 128 : hi >= lo ? e : 0;
    return f;
}

// Histogram of the inliers (counters of the workgroup in LDS, written as 16-bit values) and outliers per unit.
__global__ __launch_bounds__(kThreads) void histogram_kernel(const float *w, uint64_t n, const double *partials, int n_partials,
                                                             double threshold, double reg_covar, QuantState *st,
                                                             uint32_t *unit_count, uint32_t *hist_part)
{
    __shared__ uint32_t hist[kBins + 1];     // (the last one takes the outliers)
    __shared__ double red[kWaves][3];
    __shared__ Fit fit;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t n_units = n / kUnit, stride = (uint64_t)gridDim.x * kWaves;
    uint64_t u = (uint64_t)blockIdx.x * kWaves + wave;
    f32x4 next[2] = {};
    auto request = [&](uint64_t unit) {
#pragma unroll
        for (int h = 0; h < 2; ++h) next[h] = ((const f32x4 *)(w + unit * kUnit))[h * 64 + lane];
    };
    if (u < n_units) request(u);
    double s = 0.0, q = 0.0, mx = 0.0;
    if ((int)threadIdx.x < n_partials) {
        s = partials[3 * threadIdx.x];
        q = partials[3 * threadIdx.x + 1];
        mx = partials[3 * threadIdx.x + 2];
    }
    for (int i = threadIdx.x; i < kBins; i += kThreads) hist[i] = 0;
    s = wave_sum_f64(s);
    q = wave_sum_f64(q);
    mx = wave_max_f64(mx);
    if (lane == 0) { red[wave][0] = s; red[wave][1] = q; red[wave][2] = mx; }
    __syncthreads();
    if (threadIdx.x == 0) {
        double ts = 0.0, tq = 0.0, tm = 0.0;
        for (int i = 0; i < kWaves; ++i) { ts += red[i][0]; tq += red[i][1]; tm = fmax(tm, red[i][2]); }
        fit = fit_gaussian(ts, tq, (float)tm, n, threshold, reg_covar);
        if (blockIdx.x == 0) {
            st->mu = fit.mu; st->var = fit.var; st->xlo = fit.xlo; st->xhi = fit.xhi;
            st->bin_scale = fit.bin_scale; st->bin_shift = fit.bin_shift;
            st->sum_exp = fit.sum_exp; st->non_finite = fit.non_finite;
        }
    }
    __syncthreads();
    const float xlo = fit.xlo, xhi = fit.xhi, scale = fit.bin_scale, shift = fit.bin_shift;
    while (u < n_units) {
        const f32x4 v[2] = {next[0], next[1]};
        const uint64_t here = u;
        u += stride;
        if (u < n_units) request(u);
        uint32_t outliers = 0;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float x = v[h][e];
                const bool in = is_inlier(x, xlo, xhi);
                outliers += __popcll(__ballot(!in));
                atomicAdd(&hist[in ? bin_of(x, scale, shift) : kBins], 1u);
            }
        if (lane == 0) unit_count[here] = outliers;
    }
    __syncthreads();
    uint32_t *out = hist_part + (size_t)blockIdx.x * (kBins / 2);
    for (int i = threadIdx.x; i < kBins / 2; i += kThreads) out[i] = hist[2 * i] | (hist[2 * i + 1] << 16);
}

// Workgroups 0 .. kMergeGroups-1: add the workgroups' histograms, 64 bins each.  The others: outlier list
// offsets of one shard (exclusive scan of its units' counts) and its number of outliers.
constexpr int kMergeGroups = kBins / 64;

__global__ __launch_bounds__(256) void merge_kernel(const uint32_t *hist_part, int groups, uint32_t *hist,
                                                    const uint32_t *unit_count, uint32_t *unit_off, int units_per_shard,
                                                    uint32_t *shard_count, uint32_t *outlier_count, QuantState *st)
{
    __shared__ uint32_t red[8][64];
    __shared__ uint32_t wave_total[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (blockIdx.x == 0 && tid < kMaxClusters) st->slot_fill[tid] = 0;   // (collect_kernel counts here)
    if (blockIdx.x < kMergeGroups) {
        const int pair = tid & 31, row = tid >> 5;
        uint32_t a = 0, b = 0;
#pragma unroll 8
        for (int g = row; g < groups; g += 8) {
            const uint32_t x = hist_part[(size_t)g * (kBins / 2) + blockIdx.x * 32 + pair];
            a += x & 0xFFFFu;
            b += x >> 16;
        }
        red[row][2 * pair] = a;
        red[row][2 * pair + 1] = b;
        __syncthreads();
        if (tid < 64) {
            uint32_t s = 0;
#pragma unroll
            for (int r = 0; r < 8; ++r) s += red[r][tid];
            hist[blockIdx.x * 64 + tid] = s;
        }
        return;
    }
    const int shard = blockIdx.x - kMergeGroups;
    const uint32_t *cnt = unit_count + (size_t)shard * units_per_shard;
    uint32_t *off = unit_off + (size_t)shard * units_per_shard;
    uint32_t carry = 0;
    for (int base = 0; base < units_per_shard; base += 256 * 8) {
        const int first = base + tid * 8;
        uint32_t v[8], mine = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            v[j] = first + j < units_per_shard ? cnt[first + j] : 0;
            mine += v[j];
        }
        const uint32_t inc = lane_scan(mine);
        __syncthreads();
        if (lane == 63) wave_total[wave] = inc;
        __syncthreads();
        uint32_t p = carry + inc - mine;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (i < wave) p += wave_total[i];
            carry += wave_total[i];
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (first + j < units_per_shard) off[first + j] = p;
            p += v[j];
        }
    }
    if (tid == 0) {
        shard_count[shard] = carry;
        outlier_count[shard] = carry;
    }
}

// For every boundary the bin that holds its rank; the bins that hold one become slots with a
// list each.  table[bin] = (boundaries in lower bins) | (slot + 1, or 0) << 8 | kSeveral where there are two or more.
// Every workgroup of the collecting pass works this out for itself while its first weights are on their way; the first one leaves it in
// memory for those behind.  Two sums over the bins and one search of six steps per thread (1.7 us; 4.3 with the boundaries looked
// up among the bins by one wave, a launch of one workgroup 4.6 and the way from one launch to the next).
constexpr uint32_t kSeveral = 0x8000;

struct BoundaryScratch {
    uint64_t rank[kMaxClusters];         // of boundary c = 1 .. C-1 at [c-1]; behind the last: more than there are inliers
    uint64_t wave_sum[16], wave_slots[16];
};

// Of the workgroup (LDS): the table, where each slot's list begins, its bin, the number of slots.  The state and table_out
// are written where `keep`.
__device__ inline void boundary_bins(BoundaryScratch &sc, QuantState *st, const uint32_t *hist, uint16_t *table, uint16_t *table_out,
                                     uint64_t *slot_begin, uint32_t *slot_bin, uint32_t *n_slots, bool keep, uint64_t n,
                                     const uint32_t *shard_count, int n_shards, int n_clusters)
{
    constexpr int kSlotShift = 56;       // a sum of list lengths and, above it, of slots
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint4 h4 = ((const uint4 *)hist)[tid];
    const uint32_t h[4] = {h4.x, h4.y, h4.z, h4.w};
    const uint32_t outl = lane < n_shards ? shard_count[lane] : 0;   // (kMaxShardsPerLayer lanes)
    const uint64_t out_scan = lane_scan((uint64_t)outl);
    const uint64_t n_out = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(out_scan >> 32), 63) << 32 | (uint32_t)__builtin_amdgcn_readlane((int)out_scan, 63);
    const uint64_t n_in = n - n_out;
    const uint64_t own = (uint64_t)h[0] + h[1] + h[2] + h[3], inc = lane_scan(own);
    if (lane == 63) sc.wave_sum[wave] = inc;
    if (tid < kMaxClusters)              // (n_clusters is a power of two)
        sc.rank[tid] = tid < n_clusters - 1 && n_in > 0 ? ((uint64_t)(tid + 1) * n_in) >> __builtin_ctz(n_clusters) : ~0ull;
    __syncthreads();
    uint64_t before[5];                  // inliers below the thread's four bins, and behind them
    before[0] = inc - own;
    for (int i = 0; i < wave; ++i) before[0] += sc.wave_sum[i];
#pragma unroll
    for (int b = 0; b < 4; ++b) before[b + 1] = before[b] + h[b];
    uint32_t lower[5] = {0, 0, 0, 0, 0};   // boundaries whose rank lies below (the last entry of rank[] never does)
#pragma unroll
    for (int step = 32; step > 0; step >>= 1) lower[0] += sc.rank[lower[0] + step - 1] < before[0] ? step : 0;
    uint64_t lists = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        lower[b + 1] = lower[b];
        while (sc.rank[lower[b + 1]] < before[b + 1]) ++lower[b + 1];
        if (lower[b + 1] > lower[b]) lists += (1ull << kSlotShift) + h[b];
    }
    const uint64_t list_scan = lane_scan(lists);
    if (lane == 63) sc.wave_slots[wave] = list_scan;
    __syncthreads();
    uint64_t at = list_scan - lists;
    for (int i = 0; i < wave; ++i) at += sc.wave_slots[i];
    uint32_t packed[2] = {0, 0};
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        uint32_t entry = lower[b];
        if (lower[b + 1] > lower[b]) {
            const uint32_t slot = (uint32_t)(at >> kSlotShift);
            const uint64_t begin = at & ((1ull << kSlotShift) - 1);
            entry |= (slot + 1) << 8;
            if (lower[b + 1] > lower[b] + 1) entry |= kSeveral;
            slot_begin[slot] = begin;
            slot_bin[slot] = 4 * tid + b;
            if (keep) {
                for (uint32_t c = lower[b]; c < lower[b + 1]; ++c) {
                    st->edge_begin[c] = begin;
                    st->edge_count[c] = h[b];
                    st->edge_rank[c] = (uint32_t)(sc.rank[c] - before[b]);
                    st->edge_before[c] = before[b];
                }
            }
            at += (1ull << kSlotShift) + h[b];
        }
        packed[b >> 1] |= entry << (16 * (b & 1));
    }
    if (tid == kThreads - 1) *n_slots = (uint32_t)(at >> kSlotShift);
    if (keep && tid == 0) {
        st->n_inliers = n_in;
        st->error = n_in == 0 ? 1 : 0;
    }
    ((uint2 *)table)[tid] = uint2{packed[0], packed[1]};
    if (keep) ((uint2 *)table_out)[tid] = uint2{packed[0], packed[1]};
}

// The keys of the weights in boundary bins, one list per bin (in no particular order).  A workgroup has the units that it had in the
// histogram pass, so that its own counters of that pass say how many it will find: it takes room for them with one atomic per list
// before it looks at a weight (the answers of 256 workgroups' atomics take 1.6 us), keeps what it finds in LDS and then writes it; if
// that does not fit (a bin holds a large part of the layer), it reads its weights again instead.
constexpr uint32_t kFound = 8192;

__global__ __launch_bounds__(kThreads) void collect_kernel(const float *w, uint64_t n, QuantState *st, const uint32_t *hist,
                                                           const uint32_t *shard_count, int n_shards, int n_clusters,
                                                           uint16_t *table_out, uint32_t *lists, const uint16_t *hist_part)
{
    static_assert(kThreads == 1024 && kBins == 4096, "four bins per thread");
    __shared__ BoundaryScratch scratch;
    __shared__ float found[kFound];
    __shared__ __attribute__((aligned(8))) uint16_t table[kBins + 4];      // (one entry for outliers)
    __shared__ uint32_t n_found, n_slots, count[kMaxClusters], slot_bin[kMaxClusters];
    __shared__ uint64_t at[kMaxClusters], slot_begin[kMaxClusters];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint64_t n_units = n / kUnit, stride = (uint64_t)gridDim.x * kWaves, u0 = (uint64_t)blockIdx.x * kWaves + wave;
    uint64_t u = u0;
    f32x4 next[2] = {};
    auto request = [&](uint64_t unit) {
#pragma unroll
        for (int h = 0; h < 2; ++h) next[h] = ((const f32x4 *)(w + unit * kUnit))[h * 64 + lane];
    };
    if (u < n_units) request(u);
    const float xlo = st->xlo, xhi = st->xhi, scale = st->bin_scale, shift = st->bin_shift;
    if (tid < kMaxClusters) count[tid] = 0;
    if (tid == 0) { n_found = 0; table[kBins] = 0; }
    boundary_bins(scratch, st, hist, table, table_out, slot_begin, slot_bin, &n_slots, blockIdx.x == 0, n, shard_count, n_shards, n_clusters);
    __syncthreads();
    uint64_t my_list = 0;                      // where this workgroup's part of list `tid` begins
    if (tid < (int)n_slots) {
        const uint32_t own = hist_part[(size_t)blockIdx.x * kBins + slot_bin[tid]];
        if (own) my_list = slot_begin[tid] + atomicAdd(&st->slot_fill[tid], own);
    }
    auto slot_of = [&](float x) -> uint32_t {   // slot + 1, or 0
        return (table[is_inlier(x, xlo, xhi) ? bin_of(x, scale, shift) : kBins] & ~kSeveral) >> 8;
    };
    while (u < n_units) {
        const f32x4 v[2] = {next[0], next[1]};
        u += stride;
        if (u < n_units) request(u);
        uint32_t slot[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) slot[e] = slot_of(v[e >> 2][e & 3]);
        uint32_t total = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) total += __popcll(__ballot(slot[e] != 0));
        if (total == 0) continue;
        uint32_t first = 0;
        if (lane == 0) first = atomicAdd(&n_found, total);
        first = __shfl(first, 0, 64);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const uint64_t mask = __ballot(slot[e] != 0);
            if (slot[e]) {
                const uint32_t at_found = first + __popcll(mask & ((1ull << lane) - 1));
                if (at_found < kFound) found[at_found] = v[e >> 2][e & 3];
            }
            first += __popcll(mask);
        }
    }
    if (tid < (int)n_slots) at[tid] = my_list;
    __syncthreads();
    auto put = [&](float x, uint32_t s) { lists[at[s - 1] + atomicAdd(&count[s - 1], 1u)] = order_key(x); };
    if (n_found <= kFound) {
        for (uint32_t i = tid; i < n_found; i += kThreads) put(found[i], slot_of(found[i]));
    } else {
        for (u = u0; u < n_units; u += stride) {
            request(u);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float x = next[e >> 2][e & 3];
                const uint32_t s = slot_of(x);
                if (s) put(x, s);
            }
        }
    }
}

// One workgroup per boundary: the key at its rank in its bin's list, by rounds of radix selection over
// the distance from the list's lowest key, 11 bits at a time from the highest bit that differs (the keys of a bin
// share their upper bits: without that every key would count on the same few counters), and the number of
// inliers below it.  One round leaves a few of a list's thousands of keys: up to 64 of them are settled by one wave that
// compares each with all, in place of one or two more rounds of four barriers.
constexpr int kHeld = 12;   // list entries per thread kept in registers

__global__ __launch_bounds__(1024) void boundary_values_kernel(QuantState *st, const uint32_t *lists)
{
    __shared__ uint32_t hist[2048];
    __shared__ uint32_t wave_lo[16], wave_hi[16];
    __shared__ uint32_t chosen, below, in_digit, n_left, left[64];
    if (st->error) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c = blockIdx.x;
    const uint32_t m = st->edge_count[c];
    const uint32_t *list = lists + st->edge_begin[c];
    uint32_t rank = st->edge_rank[c];
    uint32_t held[kHeld], lo = 0xFFFFFFFFu, hi = 0;
#pragma unroll
    for (int i = 0; i < kHeld; ++i) held[i] = list[min(tid + 1024u * i, m - 1)];
    hist[tid] = 0;
    hist[tid + 1024] = 0;
    if (tid == 0) n_left = 0;
#pragma unroll
    for (int i = 0; i < kHeld; ++i) { lo = min(lo, held[i]); hi = max(hi, held[i]); }
    for (uint32_t i = tid + 1024u * kHeld; i < m; i += 1024) { lo = min(lo, list[i]); hi = max(hi, list[i]); }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) { lo = min(lo, __shfl_xor(lo, o, 64)); hi = max(hi, __shfl_xor(hi, o, 64)); }
    if (lane == 0) { wave_lo[wave] = lo; wave_hi[wave] = hi; }
    __syncthreads();
    lo = wave_lo[lane & 15];
    hi = wave_hi[lane & 15];
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) { lo = min(lo, __shfl_xor(lo, o, 64)); hi = max(hi, __shfl_xor(hi, o, 64)); }
    uint32_t prefix = 0, total_below = 0;   // distance's digits so far
    int top = hi == lo ? 0 : 32 - __builtin_clz(hi - lo);   // bits not settled
    while (top > 0) {                       // at most three rounds
        const int low = max(top - 11, 0), bits = top - low;
        auto count = [&](uint32_t key) {
            const uint32_t d = key - lo;
            if (top == 32 || d >> top == prefix) atomicAdd(&hist[(d >> low) & ((1u << bits) - 1)], 1u);
        };
#pragma unroll
        for (int i = 0; i < kHeld; ++i)
            if (tid + 1024u * i < m) count(held[i]);
        for (uint32_t i = tid + 1024u * kHeld; i < m; i += 1024) count(list[i]);
        __syncthreads();
        const uint32_t a = hist[2 * tid], b = hist[2 * tid + 1];
        const uint32_t inc = lane_scan(a + b);
        if (lane == 63) wave_hi[wave] = inc;
        hist[2 * tid] = 0;
        hist[2 * tid + 1] = 0;
        __syncthreads();
        uint32_t p = inc - a - b;
        for (int i = 0; i < wave; ++i) p += wave_hi[i];
        if (rank >= p && rank < p + a) { chosen = 2 * tid; below = p; in_digit = a; }
        else if (rank >= p + a && rank < p + a + b) { chosen = 2 * tid + 1; below = p + a; in_digit = b; }
        __syncthreads();
        prefix = (top == 32 ? 0 : prefix << bits) | chosen;
        rank -= below;
        total_below += below;
        top = low;
        if (top == 0 || in_digit > 64) continue;
        auto keep = [&](uint32_t key) {
            if ((key - lo) >> top == prefix) left[atomicAdd(&n_left, 1u)] = key;
        };
#pragma unroll
        for (int i = 0; i < kHeld; ++i)
            if (tid + 1024u * i < m) keep(held[i]);
        for (uint32_t i = tid + 1024u * kHeld; i < m; i += 1024) keep(list[i]);
        __syncthreads();
        if (wave == 0) {
            const int n = (int)in_digit;
            const uint32_t key = lane < n ? left[lane] : 0xFFFFFFFFu;
            uint32_t less = 0, before = 0;      // keys below this one; and those of its value in front of it
            for (int i = 0; i < n; ++i) {
                const uint32_t other = (uint32_t)__builtin_amdgcn_readlane((int)key, i);
                less += other < key;
                before += other == key && i < lane;
            }
            if (lane < n && less + before == rank) {
                st->edge_key[c] = key;
                st->edge_below[c] = st->edge_before[c] + total_below + less;
            }
        }
        return;
    }
    if (tid == 0) {
        st->edge_key[c] = lo + prefix;
        st->edge_below[c] = st->edge_before[c] + total_below;
    }
}

// Cluster of every weight -> packed streams and outlier dictionaries (in offset order), and the
// sum of every cluster's inliers in this workgroup.  A wave takes 512 weights, 8 per lane = k bytes.
// The cluster is looked up by bin and settled by one comparison with the next boundary value (more where a
// bin holds several); nothing in the common path branches.
// Sums: 64-bit integers in LDS, weight * 2^(46 - sum_exp), 32 copies by lane so that the atomics of one instruction never
// meet.  A weight down to 2^(sum_exp - 22) is an integer at that scale; the rare smaller ones go to further sums whose
// scales are 22 powers of two apart, so that every weight is held exactly (a float32 has 24 bits, a sum of a workgroup's
// 57344 weights below 2^46 fits 62).
constexpr int kSumBits = 46, kSumStep = 22;
constexpr int kSumScales = (128 + 149 + kSumStep - 1) / kSumStep;   // from 2^128 down to the last subnormal, 2^-149

template <int K>
__global__ __launch_bounds__(kThreads) void pack_kernel(const float *w, uint64_t n, const QuantState *st, const uint16_t *table_in,
                                                        const uint32_t *unit_off, uint32_t units_per_shard, uint8_t *packed,
                                                        uint32_t *outlier_pos, float *outlier_val, uint32_t max_outliers,
                                                        double *csum)
{
    constexpr int C = 1 << K;
    constexpr int COPIES = 32;
    __shared__ uint16_t table[kBins];
    __shared__ unsigned long long sums[C][COPIES];
    __shared__ unsigned long long small_sums[C][kSumScales];
    __shared__ float non_finite_sums[C];
    __shared__ float edges[kMaxClusters];            // boundary values; NaN behind the last: no weight reaches it
    __shared__ uint32_t edge_keys[kMaxClusters];
    __shared__ uint32_t bytes[kWaves][16 * K];      // a wave's 64 k bytes of stream
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint64_t n_units = n / kUnit, stride = (uint64_t)gridDim.x * kWaves;
    uint64_t u = (uint64_t)blockIdx.x * kWaves + wave;
    f32x4 next[2] = {};
    uint32_t next_off = 0;
    auto request = [&](uint64_t unit) {
        const f32x4 *src = (const f32x4 *)(w + unit * kUnit + lane * 8);
        next[0] = src[0];
        next[1] = src[1];
        next_off = unit_off[unit];
    };
    if (u < n_units) request(u);
    ((uint2 *)table)[tid] = ((const uint2 *)table_in)[tid];
    if (tid < kMaxClusters) {
        edge_keys[tid] = (tid < C - 1 && !st->error) ? st->edge_key[tid] : 0xFFFFFFFFu;
        edges[tid] = key_value(edge_keys[tid]);
    }
    for (int i = tid; i < C * COPIES; i += kThreads) (&sums[0][0])[i] = 0;
    for (int i = tid; i < C * kSumScales; i += kThreads) (&small_sums[0][0])[i] = 0;
    if (tid < C) non_finite_sums[tid] = 0.0f;
    const float xlo = st->xlo, xhi = st->xhi, scale = st->bin_scale, shift = st->bin_shift;
    const int sum_exp = st->sum_exp;
    const double sum_scale = ldexp(1.0, kSumBits - sum_exp);
    const float least = st->non_finite ? __builtin_nanf("") : ldexpf(1.0f, sum_exp - kSumStep);
    const double magic = 6755399441055744.0;        // 1.5 * 2^52: x + magic holds round(x) in its low bits
    __syncthreads();
    while (u < n_units) {
        const float x[8] = {next[0][0], next[0][1], next[0][2], next[0][3], next[1][0], next[1][1], next[1][2], next[1][3]};
        const uint64_t here = u;
        const uint32_t first = next_off;
        u += stride;
        if (u < n_units) request(u);
        uint32_t entry[8], cluster[8], flags = 0;
        float edge[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) entry[e] = table[bin_of(x[e], scale, shift)];
#pragma unroll
        for (int e = 0; e < 8; ++e) edge[e] = edges[entry[e] & 0xFFu];
        uint32_t several = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            cluster[e] = (entry[e] & 0xFFu) + (edge[e] <= x[e] ? 1 : 0);
            several |= entry[e];
        }
        if (__ballot(several & kSeveral)) {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                for (cluster[e] = entry[e] & 0xFFu; cluster[e] < C - 1 && edge_keys[cluster[e]] <= order_key(x[e]);) ++cluster[e];
        }
        uint64_t bits = 0;
        uint32_t small = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            bits |= (uint64_t)cluster[e] << (e * K);
            const bool in = is_inlier(x[e], xlo, xhi), regular = fabsf(x[e]) >= least;
            if (!in) flags |= 1u << e;
            if (in && !regular && x[e] != 0.0f) small |= 1u << e;
            const double y = fma((double)(in && regular ? x[e] : 0.0f), sum_scale, magic);
            atomicAdd(&sums[cluster[e]][lane & (COPIES - 1)],
                      __builtin_bit_cast(unsigned long long, y) - __builtin_bit_cast(unsigned long long, magic));
        }
        if (__ballot(small != 0)) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                if (!(small & (1u << e))) continue;
                if (!(fabsf(x[e]) < INFINITY)) {
                    unsafeAtomicAdd(&non_finite_sums[cluster[e]], x[e]);
                    continue;
                }
                int exp;
                (void)frexpf(x[e], &exp);               // |x| < 2^exp
                const int scale = (sum_exp - exp) / kSumStep;
                const double whole = ldexp((double)x[e], kSumBits - sum_exp + scale * kSumStep);
                atomicAdd(&small_sums[cluster[e]][scale], (unsigned long long)(long long)whole);
            }
        }
        uint8_t *dst = packed + here * (kUnit / 8 * K);
        if constexpr (K == 4) {
            ((uint32_t *)dst)[lane] = (uint32_t)bits;
        } else if constexpr (K == 2) {
            ((uint16_t *)dst)[lane] = (uint16_t)bits;
        } else {
            uint8_t *stage = (uint8_t *)bytes[wave] + lane * K;
#pragma unroll
            for (int j = 0; j < K; ++j) stage[j] = (uint8_t)(bits >> (8 * j));
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int j = 0; j < (16 * K + 63) / 64; ++j)
                if (lane + 64 * j < 16 * K) ((uint32_t *)dst)[lane + 64 * j] = bytes[wave][lane + 64 * j];
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        if (__ballot(flags != 0)) {
            const uint32_t mine = __popc(flags);
            const uint32_t inc = lane_scan(mine);
            const uint32_t shard = (uint32_t)(here / units_per_shard);
            uint32_t at = first + inc - mine;
            const uint32_t in_shard = (uint32_t)(here - (uint64_t)shard * units_per_shard) * kUnit + lane * 8;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                if (flags & (1u << e)) {
                    if (at < max_outliers) {
                        outlier_pos[(uint64_t)shard * max_outliers + at] = in_shard + e;
                        outlier_val[(uint64_t)shard * max_outliers + at] = x[e];
                    }
                    ++at;
                }
            }
        }
    }
    __syncthreads();
    if (tid < C) {
        unsigned long long first = small_sums[tid][0];
        for (int i = 0; i < COPIES; ++i) first += sums[tid][(i + tid) & (COPIES - 1)];
        double s = 0.0;
        for (int i = kSumScales - 1; i > 0; --i) s += ldexp((double)(long long)small_sums[tid][i], sum_exp - kSumBits - i * kSumStep);
        csum[(size_t)blockIdx.x * kMaxClusters + tid] = s + ldexp((double)(long long)first, sum_exp - kSumBits) + non_finite_sums[tid];
    }
}

// one wave per cluster: centroid = mean of the cluster (its lower boundary value if it is empty); the
// workgroups' sums are added in a fixed order
__global__ __launch_bounds__(64) void centroids_kernel(const QuantState *st, const double *csum, int groups, int n_clusters,
                                                       uint64_t n_total, float *codebook, sti_quant_stats *stats)
{
    const int lane = threadIdx.x, c = blockIdx.x;
    double s = 0.0;
#pragma unroll 4
    for (int b = lane; b < groups; b += 64) s += csum[(size_t)b * kMaxClusters + c];
    s = wave_sum_f64(s);
    if (lane == 0) {
        const uint64_t begin = c > 0 ? st->edge_below[c - 1] : 0;
        const uint64_t end = c < n_clusters - 1 ? st->edge_below[c] : st->n_inliers;
        float cen;
        if (st->error) cen = 0.0f;
        else if (end > begin) cen = (float)(s / (double)(end - begin));
        else cen = key_value(st->edge_key[c > 0 ? c - 1 : 0]);
        codebook[c] = cen;
        if (c == 0 && stats) {
            stats->mean = st->mu;
            stats->variance = st->var;
            stats->n_outliers = n_total - st->n_inliers;
            stats->status = st->error;
        }
    }
}

}  // namespace
}  // namespace sti

using namespace sti;

extern "C" {

size_t sti_quantize_workspace_bytes(const sti_dims *dims)
{
    if (!dims || dims->d_model <= 0 || dims->d_head <= 0 || dims->ffn_per_shard <= 0 || dims->n_heads <= 0 ||
        dims->n_heads > kMaxShardsPerLayer)
        return 0;
    const uint64_t wsh = (uint64_t)dims->d_model * (4 * (uint64_t)dims->d_head + 2 * (uint64_t)dims->ffn_per_shard);
    if (wsh % kGranule) return 0;
    return quant_layout(wsh * dims->n_heads).total;
}

sti_status sti_quantize_layer(const sti_dims *dims, const float *weights, int bitwidth, double loglik_threshold,
                              double reg_covar, uint8_t *packed, float *codebook, uint32_t *outlier_pos,
                              float *outlier_val, uint32_t max_outliers_per_shard, uint32_t *outlier_count,
                              sti_quant_stats *stats, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    if (!dims || !weights || !packed || !codebook || !outlier_count) return STI_ERR_NULL;
    if (max_outliers_per_shard > 0 && (!outlier_pos || !outlier_val)) return STI_ERR_NULL;
    if (!valid_packed_bits(bitwidth)) return STI_ERR_BITWIDTH;
    if (dims->d_model <= 0 || dims->d_head <= 0 || dims->ffn_per_shard <= 0 || dims->n_heads <= 0 ||
        dims->n_heads > kMaxShardsPerLayer)
        return STI_ERR_DIMS;
    if (!(reg_covar >= 0.0) || !(loglik_threshold == loglik_threshold)) return STI_ERR_DIMS;
    const uint64_t wsh = (uint64_t)dims->d_model * (4 * (uint64_t)dims->d_head + 2 * (uint64_t)dims->ffn_per_shard);
    if (wsh % kGranule) return STI_ERR_UNSUPPORTED;
    const int M = dims->n_heads;
    const uint64_t n = wsh * M;
    if (n / kGranule > 0x7FFFFFFFull) return STI_ERR_DIMS;
    if (!aligned(weights, 16) || !aligned(packed, 16) || !aligned(workspace, 256)) return STI_ERR_ALIGN;
    const QuantLayout L = quant_layout(n);
    if (!workspace || workspace_bytes < L.total) return STI_ERR_WORKSPACE;

    hipStream_t stream = (hipStream_t)hip_stream;
    uint8_t *ws = (uint8_t *)workspace;
    QuantState *st = (QuantState *)(ws + L.state);
    double *partials = (double *)(ws + L.partials), *csum = (double *)(ws + L.csum);
    uint32_t *unit_count = (uint32_t *)(ws + L.unit_count), *unit_off = (uint32_t *)(ws + L.unit_off);
    uint32_t *shard_count = (uint32_t *)(ws + L.shard_count), *hist_part = (uint32_t *)(ws + L.hist_part);
    uint32_t *hist = (uint32_t *)(ws + L.hist), *lists = (uint32_t *)(ws + L.lists);
    uint16_t *table = (uint16_t *)(ws + L.table);
    const int C = 1 << bitwidth;
    const uint32_t units_per_shard = (uint32_t)(wsh / kUnit);
    const uint64_t moment_groups = (n + 4095) / 4096;
    const int nm = (int)(moment_groups < kMomentGroups ? moment_groups : kMomentGroups);
    static_assert(kMomentGroups <= kThreads && kGroupUnits % kWaves == 0 && kGroupUnits * kUnit < 65536,
                  "one partial moment per thread; 16-bit counters");
    const dim3 grid(L.groups), block(kThreads);
    launch(moments_kernel, dim3(nm), dim3(256), 0, stream, weights, n, partials);
    launch(histogram_kernel, grid, block, 0, stream, weights, n, partials, nm, loglik_threshold, reg_covar, st, unit_count, hist_part);
    launch(merge_kernel, dim3(kMergeGroups + M), dim3(256), 0, stream, hist_part, L.groups, hist, unit_count, unit_off, (int)units_per_shard,
           shard_count, outlier_count, st);
    launch(collect_kernel, grid, block, 0, stream, weights, n, st, hist, shard_count, M, C, table, lists, (const uint16_t *)hist_part);
    launch(boundary_values_kernel, dim3(C - 1), dim3(1024), 0, stream, st, lists);
#define STI_PACK(K) \
    launch(pack_kernel<K>, grid, block, 0, stream, weights, n, st, table, unit_off, units_per_shard, packed, outlier_pos, outlier_val, max_outliers_per_shard, csum)
    switch (bitwidth) {
    case 2: STI_PACK(2); break;
    case 3: STI_PACK(3); break;
    case 4: STI_PACK(4); break;
    case 5: STI_PACK(5); break;
    default: STI_PACK(6); break;
    }
#undef STI_PACK
    launch(centroids_kernel, dim3(C), dim3(64), 0, stream, st, csum, L.groups, C, n, codebook, stats);
    STI_TRY(hipGetLastError());
    return STI_OK;
}

}  // extern "C"
