"""Tiles that the projections of a layer take with many tokens, as the library chooses them (no GPU needed to ask)."""
import ctypes as C

QKV, FFN1, O, FFN2 = range(4)


def tile(P, kind, tokens, shards, block_rows, block_cols, outliers=0):
    """(rows, columns, groups of waves that share K, kernel with both operands through LDS)"""
    out = (C.c_int * 4)()
    P.lib.sti_internal_projection_tile(kind, tokens, shards, block_rows, block_cols, outliers, out)
    return out[0], out[1], out[2], bool(out[3])


def sum_planes(P, kind, tokens, shards, block_rows, block_cols, outliers=0):
    """Planes of float32 sums that O or FFN2 leaves, 0: finished rows in binary16"""
    return P.lib.sti_internal_sum_planes(kind, tokens, shards, block_rows, block_cols, outliers)


def out_carries(P, dims, tokens, shards, entries):
    """Whether O, or else FFN2, puts the next layer's dictionaries in."""
    return bool(P.lib.sti_internal_out_carries(tokens, shards, dims.d_model, dims.ffn_per_shard, entries))


def layer_tiles(P, dims, tokens, shards, outliers=0):
    """Per projection "rows x columns", * where K is shared by two groups of waves, L: the kernel with both operands through LDS,
    /: tiles in all, more than 256 of them several to a workgroup of that kernel.  outliers: entries per dictionary beside O."""
    d, dh, f = dims.d_model, dims.d_head, dims.ffn_per_shard
    out = {}
    for name, kind, rows, cols in (("qkv", QKV, 3 * dh, d), ("o", O, d, dh), ("ffn1", FFN1, f, d), ("ffn2", FFN2, d, f)):
        r, c, groups, large = tile(P, kind, tokens, shards, rows, cols, outliers if kind == O else 0)
        n = shards * rows if kind in (QKV, FFN1) else rows
        out[name] = f"{r}x{c}{'*' if groups > 1 else ''}{'L' if large else ''}/{-(-n // c) * -(-tokens // r)}"
    return out
