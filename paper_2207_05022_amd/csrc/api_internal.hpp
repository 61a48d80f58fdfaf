// Host-side helpers shared by the entry points in api.hip and pipeline.hip.
#pragma once
#include "sti_internal.hpp"

namespace sti {

inline bool aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }
inline bool valid_packed_bits(int b) { return b >= 2 && b <= 6; }
inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

#define STI_TRY(expr)                                 \
    do {                                              \
        if ((expr) != hipSuccess) return STI_ERR_HIP; \
    } while (0)

constexpr size_t kStaticScratchBytes = (size_t)64 << 20;   // of sti_layer_forward_static

// Offsets of the scratch regions of one layer call inside the caller's workspace.
struct WorkspaceLayout {
    size_t w32 = 0, w16 = 0, act[2] = {0, 0}, qkv = 0, ctx = 0, h = 0, u = 0, table = 0, total = 0;
    size_t pre_out = 0, pre_down = 0;   // sums before LayerNorm of the O and of the FFN2 product (compact: over other buffers)
    int pre_planes = 1;                // planes of partial sums there is room for (buffers of their own only)
    bool few = false;                   // the layers take the few-token kernels
    bool split = false;                 // there is room for float32 layers on the bfloat16 matrix cores (takes_planes)
    // ... whose buffers lie over those of the others: planes of a layer's input, context, first LayerNorm's rows, neurons; Q/K/V and
    // the first LayerNorm's rows in float32; the end of the region that holds all but the last of these
    size_t s_in = 0, s_ctx = 0, s_h = 0, s_u = 0, s_qkv = 0, s_h32 = 0, s_end = 0;
    ActLayout inner = LAYOUT_ROWS;      // how the layers of the call hand activations on
    int w16_layers = 1;   // layers the binary16 working buffer holds at once (a ring: layer l in slot l % w16_layers)
    int decode_group = 1; // layers that one decompression launch of sti_model_forward takes (<= w16_layers)
};
// model_layers > 1 (sti_model_forward with room for it): a ring of binary16 working buffers - as many
// layers as one decompression launch takes (64 MiB worth), at least two, so that a layer can be
// decompressed while the one before it computes - and the device copy of the whole model's shard table.
// compact (binary16 only): activations row by row without padding, sums before LayerNorm over buffers that are read by then.
// few (binary16 only): for the few-token kernels.
WorkspaceLayout workspace_layout(const sti_dims &d, int64_t T, sti_precision prec, bool few, int model_layers = 1, bool compact = false);
// That of one layer at a time on the route that T tokens take with a workspace of `bytes` (its total may be more than that).
WorkspaceLayout layout_within(const sti_dims &d, int64_t T, sti_precision prec, size_t bytes);

sti_status check_dims(const sti_dims *dims, int batch, int seq, sti_precision prec);
sti_status check_decode_shard(const sti_shard &s);   // bitwidth 2..6 or 32, pointers, alignment
sti_status check_params(const sti_layer_params *p);
sti_status check_io(const void *x, void *y, sti_dtype io, int64_t T, int d);

// One layer over shards[M] (bitwidth 0 = absent), arguments already validated.  `in` is
// float32 (F32 precision) or binary16 (MFMA precision); `out` is written as out_dtype.
// What a layer's Q/K/V launch (many-token route) does on the compute units its tiles leave idle:
// decompress the following layer (n_shards shards of the device table into the working buffer `out`,
// dictionaries of outliers not applied) with `workgroups` workgroups.
struct NextLayerDecode {
    const ShardDesc *table;
    int n_shards;
    void *out;
    int workgroups;
    int max_outliers;   // > 0: the layer's O or FFN2 projection puts the outlier dictionaries in
};
// Workgroups such a launch of a layer of m present shards gives to the m_next of the next layer (0: the layer does not go
// through the many-token route, its projection fills the chip, or a decompression launch in the chain - for several
// layers if `grouped` - costs less).
int spare_decode_workgroups(const sti_dims &d, int B, int Lseq, int m, int m_next, bool grouped, sti_precision prec);

// Whether a layer over these shards goes through the bfloat16 matrix cores in three planes per float32 (gemm_f32_split.hip).
bool takes_planes(const sti_dims &d, const sti_shard *shards, int64_t T, const WorkspaceLayout &wl);

// Layers one after another whose weights become planes (takes_planes): the Q, K, V and O of the next one can be decompressed beside a layer's last
// LayerNorm.
struct SplitChain {
    const sti_shard *next;   // shards of the layer behind this one, which takes planes; or null
    bool ready;              // on entry: this layer's are there; on return: the next one's are
};

sti_status run_layer(const sti_dims &d, const sti_shard *shards, const sti_layer_params &prm,
                     const void *in, void *out, sti_dtype out_dtype, int B, int Lseq,
                     sti_precision prec, uint8_t *ws, const WorkspaceLayout &wl, hipStream_t stream,
                     const void *predecoded = nullptr, const int32_t *key_lengths = nullptr,
                     const NextLayerDecode *next = nullptr, ActLayout in_layout = LAYOUT_ROWS,
                     ActLayout out_layout = LAYOUT_ROWS, bool planes_out = false, SplitChain *chain = nullptr);
// The caller's x as the first layer takes it: itself where it already has the type (and, few tokens, row by row),
// otherwise converted into the first activation buffer (in_buffer: whether it is there); few tokens: float32 rows as they are, where the
// Q/K/V projection takes them.  As planes, too, where that layer takes them.
// shards: that layer's.
sti_status bring_in(const sti_dims &d, const sti_shard *shards, const void *x, sti_dtype io_dtype, int64_t T, sti_precision prec, uint8_t *ws,
                    const WorkspaceLayout &wl, hipStream_t stream, const void **in, ActLayout *in_layout, bool *in_buffer);
// `predecoded`: the layer's present shards already sit there in fragment-tiled binary16 order
// (outliers applied); run_layer then decompresses nothing.
// `key_lengths` (device, [B]): real positions per padded sequence; null = every position is real.
// `planes_out`: `out` (float32, in the workspace) is left as planes, too: the layer that follows takes them.
// `next` (only with `predecoded`, and only when spare_decode_workgroups says so for this layer).
// Layouts of `in` and `out`: tiled only where wl.inner is.
sti_status check_key_lengths(const int32_t *key_lengths);   // non-null, 4-byte aligned

}  // namespace sti
