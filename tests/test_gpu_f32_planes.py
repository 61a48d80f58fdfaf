"""float32 layers on the bfloat16 matrix cores: every tile width, and accuracy that a lost term of a product would spoil.

The general tolerance of the float32 path (1e-5 of the largest value) leaves room for a product without one of its six
terms (2.4e-6 of it, 2-norm).  Here single products decide the output and the 2-norm of the error is bounded: 768 and 3072 products of
random operands summed in float32 leave 3.9e-7 and 8.6e-7, LayerNorm about 1e-7.
"""
import numpy as np
import pytest

import sti_synth as S
from parity import assert_parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    import paper_2207_05022_amd as P
    from paper_2207_05022_amd import device as D
    assert torch.cuda.is_available(), "needs a GPU"
    return torch, P, D


def forward(gpu, wl, want_planes):
    torch, P, D = gpu
    shards, params, x = D.upload_workload(wl)
    y = torch.full_like(x, float("nan"))
    ws = torch.empty(P.sti_workspace_bytes(wl.dims, wl.batch, wl.seq, P.STI_PREC_F32), dtype=torch.uint8, device="cuda")
    P.sti_profile_begin()
    P.sti_layer_forward(wl.dims, shards[0], params[0], x, y, P.STI_PREC_F32, ws)
    torch.cuda.synchronize()
    launches = {k: n for k, (n, _) in P.sti_profile_end().items()}
    assert launches["decode"] == (2 if want_planes else 1)   # planes: attention's weights, then the FFN's
    return y.cpu().numpy()


def norm_error(got, want):
    return float(np.linalg.norm(got.astype(np.float64) - want) / np.linalg.norm(want))


# tile widths (32-column strips) and K splits of Q/K/V, O, FFN1, FFN2 as chosen for these sizes; the last 128 rows and most of
# the last column tiles are cut
@pytest.mark.parametrize("d,M,f,B,L", [
    (768, 12, 256, 7, 143),    # 3, 1, 3, 3 with 4 K splits
    (960, 8, 192, 7, 88),      # 1, 1, 1, 2 with 3
    (576, 15, 64, 5, 181),     # 3, 2 with 3, 1, 2 with 3
    (576, 9, 192, 5, 181),     # 2, 2 with 3, 2, 2 with 3
    (448, 11, 64, 26, 61),     # 4, 1, 2, 1
    (832, 15, 64, 21, 57),     # 4, 4 with 3, 2, 4 with 3
    (128, 11, 192, 34, 98),    # 4, 1 with 2, 4, 1 with 2
    (640, 7, 128, 33, 98),     # 3, 3, 4, 3
    (320, 5, 192, 33, 98),     # 4, 2, 4, 4 with 3
    (320, 8, 64, 33, 98),      # 3, 3 with 2, 2, 3 with 2
    (832, 7, 192, 37, 98),     # 3, 4, 3, 4
])
def test_tile_widths(gpu, oracle_mod, d, M, f, B, L):
    wl = S.small_workload(44000 + d + M, S.Dims(d, M, 64, f, 1e-12), 1, B, L)
    S.make_every_term_matter(wl, M, amp=2.0)
    want = oracle_mod.layer_forward(wl.dims, wl.shards[0], wl.params[0], wl.x)
    got = forward(gpu, wl, True)
    assert_parity(got, want, 1e-5)
    assert norm_error(got, want) <= 2e-6


def pack(index, k):
    bits = (index[:, None] >> np.arange(k)) & 1
    return np.packbits(bits.astype(np.uint8).ravel(), bitorder="little")


def one_product(live, bits, dims, tokens):
    """A layer in which one projection multiplies random weights and the others select or are zero: its product, exact on the way
    in and out but for LayerNorm and GELU, is the output's largest term."""
    rng = np.random.default_rng([44, bits, len(live)])
    d, M, dh, f = dims.d_model, dims.n_heads, dims.d_head, dims.ffn_per_shard
    random = rng.normal(0.0, 0.2, 1 << min(bits, 6)).astype(np.float32)
    random[0], random[1] = 0.0, 1.0

    def dense(rows, cols):
        return rng.normal(0.0, 0.2, (rows, cols)).astype(np.float32) if bits == 32 else rng.integers(2, 64, (rows, cols))

    def zeros(rows, cols):
        return np.zeros((rows, cols), np.float32 if bits == 32 else np.int64)

    def select(rows, cols, row0, col0):     # rows row0 .. of an identity over the concatenated shards
        w = zeros(rows, cols)
        for r in range(rows):
            c = (row0 + r - col0) % (M * dh if cols == dh else max(d, M * f))
            if c < cols:
                w[r, c] = 1
        return w
    shards = []
    for i in range(M):
        v = dense(dh, d) if live == "v" else select(dh, d, i * dh, 0) if live == "o" else zeros(dh, d)
        o = dense(d, dh) if live == "o" else select(d, dh, 0, i * dh) if live == "v" else zeros(d, dh)
        w1 = dense(f, d) if live == "ffn1" else select(f, d, i * f % d, 0) if live == "ffn2" else zeros(f, d)
        w2 = dense(d, f) if live == "ffn2" else select(d, f, 0, i * f) if live in ("ffn1", "gelu") else zeros(d, f)
        flat = np.concatenate([m.ravel() for m in (zeros(dh, d), zeros(dh, d), v, o, w1, w2)])
        shards.append(S.Shard(32, flat.astype(np.float32), None) if bits == 32 else S.Shard(bits, pack(flat, bits), random))
    prm = {n: np.zeros(M * dh if n in ("bq", "bk", "bv") else M * f if n == "b1" else d, np.float32) for n in S.LayerParams.NAMES}
    prm["ln1_g"][:] = prm["ln2_g"][:] = 1.0
    x = rng.normal(0.0, 1.0, (tokens, 1, d)).astype(np.float32)
    return S.Workload(live, dims, tokens, 1, np.full((1, M), bits, np.int8), [shards], [S.LayerParams(**prm)], x)


def two_planes(w):
    """w without the lowest of its three bfloat16 values."""
    def bf16(v):
        u = v.astype(np.float32).view(np.uint32)
        return ((u + 0x7FFF + (u >> 16 & 1)) & 0xFFFF0000).astype(np.uint32).view(np.float32)
    h = bf16(w)
    return h.astype(np.float64) + bf16(w - h)


@pytest.mark.parametrize("bits", [32, 6])
@pytest.mark.parametrize("live,f,bound", [("v", 128, 1e-6), ("o", 128, 1e-6), ("ffn1", 128, 1e-6), ("ffn2", 256, 1.5e-6)])
def test_no_term_of_a_product_is_lost(gpu, oracle_mod, live, f, bound, bits):
    wl = one_product(live, bits, S.Dims(768, 12, 64, f, 1e-12), 856)
    want = oracle_mod.layer_forward(wl.dims, wl.shards[0], wl.params[0], wl.x)
    assert norm_error(forward(gpu, wl, True), want) <= bound
    # what a lost term leaves in the product is beyond that
    rng = np.random.default_rng(5)
    a, w = rng.normal(size=(64, 768)).astype(np.float32), rng.normal(0.0, 0.2, (768, 64)).astype(np.float32)
    exact = a.astype(np.float64) @ w
    assert norm_error(a.astype(np.float64) @ two_planes(w), exact) > 1.5 * bound


@pytest.mark.parametrize("tokens,spread", [(1, 0.05), (1, 0.3), (1, 1.0), (856, 0.05), (856, 1.0)])
def test_gelu_is_as_accurate_as_one_from_erf(gpu, oracle_mod, tokens, spread):
    """The neurons' arguments are the bias, the second LayerNorm sees the GELU alone; mean and scale, which all features
    share, are fitted out.  z / 2 (1 + erf) in float32 has 3.7e-8 to 4.1e-8 (2-norm), the two roundings of LayerNorm 3.5e-8 together: 5.4e-8."""
    dims = S.Dims(768, 12, 64, 128, 1e-12)
    wl = one_product("gelu", 32, dims, tokens)
    prm = wl.params[0]
    prm.ln1_g[:] = 0.0
    z = np.random.default_rng(7).normal(0.0, spread, 768).astype(np.float32)
    prm.b1[:768] = z
    for s in wl.shards[0]:
        s.data *= np.float32(64.0)
    want = oracle_mod.layer_forward(dims, wl.shards[0], prm, wl.x).reshape(tokens, 768)
    got = forward(gpu, wl, tokens > 1).reshape(tokens, 768).astype(np.float64)
    assert np.array_equal(got, np.broadcast_to(got[0], got.shape))
    fit = np.polyfit(want[0], got[0], 1)
    assert abs(fit[0] - 1.0) < 5e-7
    assert norm_error(got[0], np.polyval(fit, want[0])) <= 5.5e-8
