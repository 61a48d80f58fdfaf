"""GPU parity: sti_layer_forward / sti_model_forward (through the C ABI) against the
CPU oracle.

Tolerance: max |y_gpu - y_ref| / max |y_ref| <= 1e-5 for the float32 path (a float32 dot
product of length K <= 3072 carries about sqrt(K) * 2^-24 of relative error and LayerNorm
renormalises after every block) and <= 2e-2 for the binary16 matrix-core path (operands and
activations rounded to binary16, float32 accumulation).
"""
import json
import math
import os

import numpy as np
import pytest

import sti_synth as S
import tiles
from parity import assert_parity

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "mfma": 2e-2}
GOLDEN = os.path.join(os.path.dirname(__file__), "golden")
SMALL = S.Dims(48, 3, 16, 32, 1e-12)
MID = S.Dims(128, 4, 64, 64, 1e-12)


@pytest.fixture(scope="module")
def gpu():
    import torch
    import paper_2207_05022_amd as P
    from paper_2207_05022_amd import device as D
    assert torch.cuda.is_available(), "needs a GPU"
    return torch, P, D


def rel_err(got, want):
    return float(np.max(np.abs(got.astype(np.float64) - want)) / max(np.max(np.abs(want)), 1e-30))


def run_gpu(gpu, wl, prec, model=True, x=None):
    torch, P, D = gpu
    precision = P.STI_PREC_F32 if prec == "f32" else P.STI_PREC_F16_MFMA
    shards, params, xd = D.upload_workload(wl)
    if x is not None:
        xd = torch.from_numpy(np.ascontiguousarray(x)).cuda()
    y = torch.full_like(xd, float("nan"))
    B, L = int(xd.shape[0]), int(xd.shape[1])
    nbytes = P.sti_workspace_bytes(wl.dims, B, L, precision)
    assert nbytes > 0
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    if model:
        P.sti_model_forward(wl.dims, D.store_from_plan(shards), params, wl.plan, xd, y, precision, ws)
    else:
        assert wl.n_layers == 1
        P.sti_layer_forward(wl.dims, shards[0], params[0], xd, y, precision, ws)
    torch.cuda.synchronize()
    return y.float().cpu().numpy()


# ------------------------------------------------------------------ float32 path

def test_f32_tiny_hand_derived_layer(gpu):
    """The hand-derived fixture, straight against its printed expectations."""
    fx = json.load(open(os.path.join(GOLDEN, "tiny_layer.json")))
    dims = S.Dims(**fx["dims"])
    s = math.sqrt(math.sqrt(2.0) * math.log(3.0))
    mat = lambda m: np.array([[s if v == "s" else v for v in row] for row in m], dtype=np.float32)
    shards = []
    for name in ("shard0", "shard1"):
        b = fx[name]
        flat = np.concatenate([mat(b[k]).ravel() for k in ("Wq", "Wk", "Wv", "Wo", "W1", "W2")])
        shards.append(S.Shard(32, flat, None))
    params = S.LayerParams(**{k: np.array(v, dtype=np.float32) for k, v in fx["params"].items()})
    wl = S.Workload("tiny", dims, 1, 2, np.array([[32, 32]], dtype=np.int8), [shards], [params],
                    np.array(fx["x"], dtype=np.float32))
    y = run_gpu(gpu, wl, "f32", model=False)
    assert_parity(y, np.array(fx["expected"]["y"]), 1e-5)


@pytest.mark.parametrize("B,L", [(1, 1), (2, 7), (3, 70), (1, 130)])
def test_f32_small_mixed_layer(gpu, oracle_mod, B, L):
    wl = S.small_workload(100 + L, SMALL, 1, B, L, plan=np.array([[3, 32, 6]]))
    want = oracle_mod.layer_forward(SMALL, wl.shards[0], wl.params[0], wl.x)
    got = run_gpu(gpu, wl, "f32", model=False)
    assert_parity(got, want, TOL["f32"])


@pytest.mark.parametrize("plan", [[0, 0, 0], [0, 5, 0], [2, 0, 4]])
def test_f32_absent_shards(gpu, oracle_mod, plan):
    wl = S.small_workload(7, SMALL, 1, 2, 9, plan=np.array([plan]))
    want = oracle_mod.layer_forward(SMALL, wl.shards[0], wl.params[0], wl.x)
    got = run_gpu(gpu, wl, "f32", model=False)
    assert_parity(got, want, TOL["f32"])


@pytest.mark.parametrize("io", ["f32", "f16"])
def test_f32_small_model_all_bitwidths(gpu, oracle_mod, io):
    wl = S.small_workload(9, MID, 3, 2, 33, n_absent=1, io_dtype=io)
    want = oracle_mod.model_forward(MID, wl.shards, wl.params, wl.x)
    got = run_gpu(gpu, wl, "f32")
    tol = TOL["f32"] if io == "f32" else 1e-3  # output rounded to binary16
    assert_parity(got, want, tol)


def test_f32_bf16_io(gpu, oracle_mod):
    torch, P, D = gpu
    wl = S.small_workload(10, MID, 2, 1, 17)
    xb = torch.from_numpy(wl.x).to(torch.bfloat16)
    wl.x = xb.float().numpy()
    want = oracle_mod.model_forward(MID, wl.shards, wl.params, wl.x)
    shards, params, _ = D.upload_workload(wl)
    xd = xb.cuda(); y = torch.empty_like(xd)
    ws = torch.empty(P.sti_workspace_bytes(MID, 1, 17, P.STI_PREC_F32), dtype=torch.uint8, device="cuda")
    P.sti_model_forward(MID, D.store_from_plan(shards), params, wl.plan, xd, y, P.STI_PREC_F32, ws)
    torch.cuda.synchronize()
    assert_parity(y.float().cpu().numpy(), want, 8e-3)  # output rounded to bfloat16


@pytest.mark.parametrize("B,L", [(1, 40), (5, 128)])   # few-token kernels / wide-tile kernels
def test_mfma_bf16_io(gpu, oracle_mod, B, L):
    torch, P, D = gpu
    wl = S.small_workload(11, MID, 2, B, L)
    xb = torch.from_numpy(wl.x).to(torch.bfloat16)
    wl.x = xb.float().numpy()
    want = oracle_mod.model_forward(MID, wl.shards, wl.params, wl.x)
    shards, params, _ = D.upload_workload(wl)
    xd = xb.cuda(); y = torch.empty_like(xd)
    prec = P.STI_PREC_F16_MFMA
    ws = torch.empty(P.sti_model_workspace_bytes(MID, 2, B, L, prec), dtype=torch.uint8, device="cuda")
    P.sti_model_forward(MID, D.store_from_plan(shards), params, wl.plan, xd, y, prec, ws)
    torch.cuda.synchronize()
    assert y.dtype == torch.bfloat16
    assert_parity(y.float().cpu().numpy(), want, TOL["mfma"])


def test_f32_config0(gpu, oracle_mod):
    wl = S.config0()
    want = oracle_mod.layer_forward(wl.dims, wl.shards[0], wl.params[0], wl.x)
    got = run_gpu(gpu, wl, "f32", model=False)
    assert_parity(got, want, TOL["f32"])


def test_f32_config2(gpu, oracle_mod):
    wl = S.config2()
    want = oracle_mod.model_forward(wl.dims, wl.shards, wl.params, wl.x)
    got = run_gpu(gpu, wl, "f32")
    assert_parity(got, want, TOL["f32"])


def test_f32_config3(gpu, oracle_mod):
    wl = S.config3()
    want = oracle_mod.model_forward(wl.dims, wl.shards, wl.params, wl.x)
    got = run_gpu(gpu, wl, "f32")
    assert_parity(got, want, TOL["f32"])


def test_f32_random_shapes(gpu, oracle_mod):
    """Thirty seeded random shapes on the float32 path, which takes any dimensions: d_model 8-128,
    1-8 shards of 4-64 wide heads and 4-64 FFN neurons, 1-200 keys, 1-3 layers, float32 or
    binary16 activations at the boundary."""
    rng = np.random.default_rng(777)
    for case in range(30):
        M = int(rng.integers(1, 9))
        dh = int(rng.choice([4, 8, 12, 16, 20, 32, 64]))
        f = int(rng.choice([4, 8, 24, 32, 40, 64]))
        d = int(rng.choice([8, 16, 24, 40, 48, 72, 96, 128]))
        dims = S.Dims(d, M, dh, f, 1e-12)
        L = int(rng.integers(1, 200))
        B = int(rng.integers(1, 6))
        n_abs = int(rng.integers(0, M)) if M > 1 else 0
        n_layers = int(rng.choice([1, 2, 3]))
        io = str(rng.choice(["f32", "f16"]))
        wl = S.small_workload(12000 + case, dims, n_layers, B, L, n_absent=n_abs, io_dtype=io)
        S.make_every_term_matter(wl, case, amp=float(rng.choice([1.0, 4.0])))
        want = oracle_mod.model_forward(dims, wl.shards, wl.params, wl.x)
        got = run_gpu(gpu, wl, "f32")
        tol = TOL["f32"] if io == "f32" else 2e-3    # binary16 output: half an ulp of the largest value
        assert_parity(got, want, tol, (case, d, M, dh, f, B, L, n_abs, n_layers, io))


@pytest.mark.parametrize("d,M,f,B,L,masked", [
    (768, 12, 256, 4, 107, False),    # the last 128 rows with 44; 96-column tiles
    (768, 12, 256, 1, 430, True),     # one sequence; the last row block with 14 rows
    (1024, 16, 128, 3, 171, True),    # Q, K, V and O take more room than both FFN matrices
    (448, 12, 192, 25, 39, False),    # d_model of 7 cells, columns that are no multiple of a tile's
    (768, 13, 256, 2, 513 // 2, False),
])
def test_f32_on_bfloat16_matrix_cores(gpu, oracle_mod, d, M, f, B, L, masked):
    """float32 layers of 3e9 multiplications and more (three bfloat16 values per operand): three layers, the second with outlier
    dictionaries (float32 matrix instructions, planes handed on behind it), the third with every shard absent but two."""
    torch, P, D = gpu
    dims = S.Dims(d, M, 64, f, 1e-12)
    wl = S.small_workload(43000 + d + L, dims, 3, B, L, n_absent=1)
    wl.plan[2, :M - 2] = 0
    for i in range(M - 2):
        wl.shards[2][i] = None
    plain = wl.shards
    wl = _with_outliers(wl, 7, fraction=0.002)
    wl.shards[0], wl.shards[2] = plain[0], plain[2]
    S.make_every_term_matter(wl, L, amp=2.0)
    lens = _key_lengths(L, B, L) if masked else None
    if masked and B == 1:
        lens[0] = L - 3
    want = oracle_mod.model_forward(wl.dims, wl.shards, wl.params, wl.x, key_lengths=lens)
    got = _run_masked(gpu, wl, "f32", lens, "model").float().cpu().numpy()
    assert_parity(got, want, TOL["f32"])


@pytest.mark.parametrize("io,empty", [("f32", 1), ("f16", 0), ("f32", 2)])
def test_f32_planes_through_a_layer_without_shards(gpu, oracle_mod, io, empty):
    """A first, middle or last layer with every shard absent hands its rows on to layers on the bfloat16 matrix cores."""
    wl = S.small_workload(43100 + empty, S.Dims(768, 12, 64, 256, 1e-12), 3, 3, 151, io_dtype=io)
    wl.plan[empty, :] = 0
    for i in range(12):
        wl.shards[empty][i] = None
    S.make_every_term_matter(wl, empty, amp=2.0)
    want = oracle_mod.model_forward(wl.dims, wl.shards, wl.params, wl.x)
    got = _run_masked(gpu, wl, "f32", None, "model").float().cpu().numpy()
    assert_parity(got, want, TOL["f32"] if io == "f32" else 2e-3)    # binary16 output: half an ulp of the largest value


@pytest.mark.parametrize("layers,converted", [("oo", 0), ("po", 1), ("op", 1), ("oopeo", 1), ("pep", 1), ("e", 0),
                                              ("s", 0), ("sp", 1), ("ps", 1)])
def test_f32_planes_are_written_for_layers_that_take_them(gpu, oracle_mod, layers, converted):
    """p: a layer without, o: with outlier dictionaries, s: with 3 of 12 shards, e: with every shard absent.  Rows become planes in a
    launch of their own only in front of a p: at the beginning and behind an o or s."""
    torch, P, D = gpu
    wl = S.small_workload(43200 + len(layers), S.Dims(768, 12, 64, 256, 1e-12), len(layers), 3, 151, n_absent=0)
    rng = np.random.default_rng(17)
    for l, kind in enumerate(layers):
        for i, s in enumerate(wl.shards[l]):
            if kind == "o" and s is not None:
                S.add_outliers(rng, s, wl.dims.weights_per_shard, 0.002)
            elif kind == "e" or (kind == "s" and i not in (1, 4, 11)):
                wl.plan[l, i], wl.shards[l][i] = 0, None
    S.make_every_term_matter(wl, 5, amp=2.0)
    want = oracle_mod.model_forward(wl.dims, wl.shards, wl.params, wl.x)
    P.sti_profile_begin()
    got = _run_masked(gpu, wl, "f32", None, "model").float().cpu().numpy()
    count = {k: n for k, (n, _) in P.sti_profile_end().items()}
    assert_parity(got, want, TOL["f32"])
    assert count["convert"] == converted and count["decode"] == layers.count("o") + layers.count("s") + 2 * layers.count("p")


@pytest.mark.parametrize("d,M,f,B,L,shift,present", [
    (768, 12, 256, 8, 128, 0, (12, 12, 6, 12, 0, 12)),     # more shards than the layer before has: over its sums, not beside its LayerNorm
    (1024, 16, 256, 3, 101, 0, (16, 14, 15, 16)),
    (1088, 17, 256, 3, 101, 0, (17, 17, 17)),              # rows too long for one launch of both, more than 16 descriptors
    (320, 32, 64, 7, 150, 0, (32, 32, 30, 32)),            # few neurons per shard
    (768, 4, 256, 20, 100, 0, (4, 4)),                     # room for four descriptors
    (768, 12, 256, 5, 100, 1, (12, 12)),                   # unaligned parameters: a LayerNorm of single features
])
def test_f32_weights_decompressed_beside_a_layernorm(gpu, d, M, f, B, L, shift, present):
    """Layers one after another give the bits of one call per layer: what a LayerNorm's launch decompresses for the next layer is what
    that layer decompresses for itself, and nothing that is still read lies below it."""
    import types
    torch, P, D = gpu
    dims = S.Dims(d, M, 64, f, 1e-12)
    wl = S.small_workload(44000 + d + M, dims, len(present), B, L)
    for l, m in enumerate(present):
        for i in range(m, M):
            wl.plan[l, (i * 5 + l) % M], wl.shards[l][(i * 5 + l) % M] = 0, None
    S.make_every_term_matter(wl, 4, amp=2.0)
    shards, params, x = D.upload_workload(wl)
    if shift:
        moved = []
        for p in params:
            q = types.SimpleNamespace()
            for n, _ in P.StiLayerParams._fields_:
                setattr(q, n, torch.cat([torch.zeros(shift, device="cuda"), getattr(p, n).reshape(-1)])[shift:])
            moved.append(q)
        params = moved
    prec = P.STI_PREC_F32
    ws = torch.empty(P.sti_workspace_bytes(dims, B, L, prec), dtype=torch.uint8, device="cuda")
    y = torch.full_like(x, float("nan"))
    P.sti_model_forward(dims, D.store_from_plan(shards), params, wl.plan, x, y, prec, ws)
    cur = x
    for l in range(len(present)):
        nxt = torch.full_like(x, float("nan"))
        P.sti_layer_forward(dims, shards[l], params[l], cur, nxt, prec, ws)
        cur = nxt
    torch.cuda.synchronize()
    assert torch.isfinite(y).all() and torch.equal(y, cur)


@pytest.mark.parametrize("d,M,f,B,L,present,beside", [
    (768, 12, 256, 8, 128, (12, 12, 6, 12), (1, 1, 1)),
    (768, 12, 256, 8, 128, (9, 10, 10, 9), (0, 1, 1)),     # FFN2's sums lie behind its weights: a shard more goes over them
    (768, 12, 192, 4, 128, (12, 12, 8, 9), (0, 1, 0)),
    (1024, 16, 128, 4, 128, (16, 16, 16), (0, 0)),
    (1024, 16, 256, 3, 101, (16, 14, 15, 16), (1, 0, 0)),
    (1088, 17, 256, 3, 101, (16, 17, 17), (0, 1)),         # a decompression of its own behind the LayerNorm
    (512, 4, 256, 20, 100, (4, 4), (1,)),                  # room for four descriptors
])
def test_f32_weights_not_over_sums_that_layernorm_reads(gpu, d, M, f, B, L, present, beside):
    """Which layers have the next one's Q, K, V and O decompressed beside their last LayerNorm: those where FFN2's sums are not in the way."""
    ask = gpu[1].lib.sti_internal_next_layer_beside_layernorm
    assert tuple(ask(B * L, d, M, f, a, b) for a, b in zip(present, present[1:])) == beside
    test_f32_weights_decompressed_beside_a_layernorm(gpu, d, M, f, B, L, 0, present)


@pytest.mark.parametrize("d,shift,joint", [(1024, 0, True), (1088, 0, False), (1024, 1, False)])
def test_float32_decompressions_are_timed_with_layernorm_or_by_themselves(gpu, d, shift, joint):
    """48 shards of 64 and of 256 neurons: as much of Q, K, V and O to decompress, four times as much of FFN1 and FFN2, half as much and
    twice as much as of Q, K, V and O.  By itself (long rows, unaligned parameters) that is decompressions of 1.5 and of 3 units in
    all; beside the first LayerNorm half of that launch counts as LayerNorm.  (LayerNorm by itself is not the same in both: FFN2
    leaves more planes of sums for a longer K.)"""
    import types
    torch, P, D = gpu
    prec, B, L = P.STI_PREC_F32, 2, 100
    times = []
    for f in (64, 256):
        dims = S.Dims(d, 48, 64, f, 1e-12)
        wl = S.small_workload(45000 + f, dims, 1, B, L, plan=np.full((1, 48), 2, dtype=np.int8))
        shards, (prm,), x = D.upload_workload(wl)
        if shift:
            prm = types.SimpleNamespace(**{n: torch.cat([torch.zeros(1, device="cuda"), getattr(prm, n).reshape(-1)])[1:] for n, _ in P.StiLayerParams._fields_})
        ws = torch.empty(P.sti_workspace_bytes(dims, B, L, prec), dtype=torch.uint8, device="cuda")
        y = torch.empty_like(x)
        runs = []
        for _ in range(5):
            P.sti_profile_begin()
            P.sti_layer_forward(dims, shards[0], prm, x, y, prec, ws)
            runs.append(P.sti_profile_end())
        assert all((r["decode"][0], r["layernorm"][0], r["convert"][0]) == (2, 2, 1 + shift) for r in runs)
        times.append([min(r[k][1] for r in runs) for k in ("decode", "layernorm")])
    decode, layernorm = (b / a for a, b in zip(*times))
    if joint:
        assert layernorm > 1.5, times
    else:
        assert decode > 1.5, times


@pytest.mark.parametrize("d,M,dh,f,B,L", [
    (768, 3, 64, 256, 1, 1),      # one token: the smallest tile, K split over workgroups
    (100, 5, 36, 64, 3, 21),      # K with a part tile, 16-byte rows
    (132, 2, 64, 96, 1, 65),      # one column past two tiles
    (97, 3, 33, 51, 2, 67),       # odd everywhere: scalar loads, odd row ends
    (192, 4, 16, 32, 7, 129),     # narrow heads and blocks, one key past two blocks
    (96, 2, 100, 64, 2, 70),      # padded features
    (64, 2, 128, 32, 1, 64), (64, 2, 130, 32, 2, 40),   # widest head on the matrix cores, one beyond
    (256, 4, 64, 128, 16, 130),   # several workgroups per compute unit
])
def test_f32_tile_edges(gpu, oracle_mod, d, M, dh, f, B, L):
    """Edges of the float32 products' tiles, K splits and attention blocks."""
    dims = S.Dims(d, M, dh, f, 1e-12)
    wl = S.small_workload(13000 + d + L, dims, 2, B, L, n_absent=1)
    S.make_every_term_matter(wl, d, amp=2.0)
    want = oracle_mod.model_forward(dims, wl.shards, wl.params, wl.x)
    assert_parity(run_gpu(gpu, wl, "f32"), want, TOL["f32"])


def test_empty_batch_and_zero_layers(gpu):
    torch, P, D = gpu
    wl = S.small_workload(3, SMALL, 1, 1, 4)
    shards, params, xd = D.upload_workload(wl)
    ws = torch.empty(max(256, P.sti_workspace_bytes(SMALL, 1, 4, 0)), dtype=torch.uint8, device="cuda")
    y = torch.zeros_like(xd)
    P.sti_model_forward(SMALL, D.store_from_plan([]), [], np.zeros((0, 3), np.int8), xd, y, 0, ws)
    torch.cuda.synchronize()
    assert torch.equal(xd, y)
    x0 = xd[:0].contiguous(); y0 = torch.empty_like(x0)
    P.sti_layer_forward(SMALL, shards[0], params[0], x0, y0, 0, ws)
    torch.cuda.synchronize()


# ------------------------------------------------------------------ binary16 matrix-core path

# (96, 97, 127, and 224, 225, 255: the last 32-key block of the two short-sequence attention paths
# full, one key in, one short; 256, 257: the longest short sequence and the first long one)
@pytest.mark.parametrize("B,L", [(1, 1), (2, 33), (1, 128), (3, 100), (1, 300), (2, 96), (2, 97), (1, 127),
                                 (1, 129), (40, 128), (1, 224), (2, 225), (1, 255), (3, 256), (1, 257)])
def test_mfma_small_mixed_layer(gpu, oracle_mod, B, L):
    wl = S.small_workload(200 + L, MID, 1, B, L, plan=np.array([[3, 32, 6, 5]]))
    want = oracle_mod.layer_forward(MID, wl.shards[0], wl.params[0], wl.x)
    got = run_gpu(gpu, wl, "mfma", model=False)
    assert_parity(got, want, TOL["mfma"])


@pytest.mark.parametrize("plan", [[0, 0, 0, 0], [0, 4, 0, 0], [2, 0, 32, 0]])
def test_mfma_absent_shards(gpu, oracle_mod, plan):
    wl = S.small_workload(17, MID, 1, 2, 40, plan=np.array([plan]))
    want = oracle_mod.layer_forward(MID, wl.shards[0], wl.params[0], wl.x)
    got = run_gpu(gpu, wl, "mfma", model=False)
    assert_parity(got, want, TOL["mfma"])


@pytest.mark.parametrize("B,L", [(2, 40), (3, 100), (9, 256)])
def test_mfma_layers_with_every_shard_absent(gpu, oracle_mod, B, L):
    """A layer without shards is valid at any token count (the working-buffer route once returned
    a HIP error for it): alone, and between layers that have shards."""
    plan = np.array([[4, 0, 32, 3], [0, 0, 0, 0], [2, 6, 0, 5]], dtype=np.int8)
    wl = S.small_workload(606, MID, 3, B, L, plan=plan, io_dtype="f16")
    S.make_every_term_matter(wl, 6, amp=4.0)
    want = oracle_mod.model_forward(MID, wl.shards, wl.params, wl.x)
    got = run_gpu(gpu, wl, "mfma")
    assert_parity(got, want, TOL["mfma"])
    alone = S.small_workload(607, MID, 1, B, L, plan=np.zeros((1, 4), dtype=np.int8), io_dtype="f16")
    S.make_every_term_matter(alone, 7)
    want = oracle_mod.layer_forward(MID, alone.shards[0], alone.params[0], alone.x)
    got = run_gpu(gpu, alone, "mfma", model=False)
    assert_parity(got, want, TOL["mfma"])


@pytest.mark.parametrize("io", ["f32", "f16"])
def test_mfma_small_model(gpu, oracle_mod, io):
    wl = S.small_workload(19, MID, 4, 2, 65, n_absent=1, io_dtype=io)
    want = oracle_mod.model_forward(MID, wl.shards, wl.params, wl.x)
    got = run_gpu(gpu, wl, "mfma")
    assert_parity(got, want, TOL["mfma"])


def test_mfma_config0(gpu, oracle_mod):
    wl = S.config0()
    want = oracle_mod.layer_forward(wl.dims, wl.shards[0], wl.params[0], wl.x)
    got = run_gpu(gpu, wl, "mfma", model=False)
    assert_parity(got, want, TOL["mfma"])


def test_mfma_config2(gpu, oracle_mod):
    wl = S.config2()
    want = oracle_mod.model_forward(wl.dims, wl.shards, wl.params, wl.x)
    got = run_gpu(gpu, wl, "mfma")
    assert_parity(got, want, TOL["mfma"])


def test_mfma_config3(gpu, oracle_mod):
    wl = S.config3()
    want = oracle_mod.model_forward(wl.dims, wl.shards, wl.params, wl.x)
    got = run_gpu(gpu, wl, "mfma")
    assert_parity(got, want, TOL["mfma"])


def test_mfma_config4_full_batch_sampled_sequences(gpu, oracle_mod):
    """Full-size batched run; sequences are independent, so the oracle checks a sample."""
    wl = S.config4()
    got = run_gpu(gpu, wl, "mfma")
    assert np.all(np.isfinite(got))
    for b in (0, 13, 31):
        want = oracle_mod.model_forward(wl.dims, wl.shards, wl.params, wl.x[b:b + 1])
        assert_parity(got[b:b + 1], want, TOL["mfma"], b)


def test_mfma_full_size_every_term_matters(gpu, oracle_mod):
    """The shapes and launch configurations of configurations 4 (32 x 128 tokens, wide-tile
    kernels), 0 (1 x 128 tokens, few-token kernels) and 3, with weights three times as large
    and random gains, shifts and biases: at this size dropping bq, bv, b1 or a gain moves the
    reference by 10-40 %."""
    wl = S.config4(n_layers=3)
    S.make_every_term_matter(wl, 4, amp=3.0)
    got = run_gpu(gpu, wl, "mfma")
    assert np.all(np.isfinite(got))
    for b in (0, 31):
        want = oracle_mod.model_forward(wl.dims, wl.shards, wl.params, wl.x[b:b + 1])
        assert_parity(got[b:b + 1], want, TOL["mfma"], b)
    one = S.Workload("one_sequence", wl.dims, 1, wl.seq, wl.plan, wl.shards, wl.params, wl.x[5:6], wl.io_dtype)
    got = run_gpu(gpu, one, "mfma")
    want = oracle_mod.model_forward(wl.dims, wl.shards, wl.params, wl.x[5:6])
    assert_parity(got, want, TOL["mfma"])
    # configuration 3's shape (d_model 1024, 12 of 16 shards, 256 tokens: K split over workgroups)
    wl3 = S.config3(n_layers=2)
    S.make_every_term_matter(wl3, 5, amp=3.0)
    got = run_gpu(gpu, wl3, "mfma")
    want = oracle_mod.model_forward(wl3.dims, wl3.shards, wl3.params, wl3.x)
    assert_parity(got, want, TOL["mfma"])


@pytest.mark.parametrize("d,M,f,B,L,masked,outliers", [
    (256, 4, 64, 1, 1, False, False),      # one token: a row block with one row
    (256, 3, 64, 1, 33, True, False),      # a second row block with one row; two attention waves
    (320, 5, 128, 1, 95, True, True),      # ragged end, weights from the working buffer
    (768, 12, 256, 3, 64, True, False),    # several sequences of whole row blocks
    (768, 12, 256, 5, 40, True, False),    # sequences that straddle row blocks: row-major Q/K/V
    (1024, 16, 256, 1, 300, True, False),  # more workgroups than compute units; ten key blocks for four waves
    (256, 4, 64, 2, 512, False, False),    # the longest sequence
    (512, 20, 64, 1, 130, False, False),   # more than 16 weight blocks
    (320, 4, 320, 1, 97, True, False),     # K of 5 tiles and blocks of 5; four row blocks, the last with one row
    (576, 9, 192, 1, 128, False, False),   # K of 9 tiles: twelve waves, three without one
    (832, 13, 64, 2, 32, True, False),     # K of 13 tiles: sixteen waves
    (1088, 17, 64, 1, 65, False, True),    # K of 17 tiles: eight waves, of which one has three
    (960, 8, 256, 1, 330, True, False),    # K of 15 tiles over four waves
    (896, 16, 192, 2, 200, False, False),  # 16 tiles to a K split of FFN2
    (768, 12, 256, 5, 140, True, False),   # where the workspace queries leave room for either route
])
def test_few_token_tiles_and_attention(gpu, oracle_mod, d, M, f, B, L, masked, outliers):
    """Edges of the few-token route: part row blocks, K splits, both attention kernels, float32 and binary16
    inputs (tiled by a launch of its own, or read row by row), two layers (tiled activations in between)."""
    torch, P, D = gpu
    dims = S.Dims(d, M, 64, f, 1e-12)
    for io in ("f32", "f16"):
        wl = S.small_workload(41000 + d + L, dims, 2, B, L, n_absent=1, io_dtype=io)
        if outliers:
            wl = _with_outliers(wl, 5, fraction=0.005)
        S.make_every_term_matter(wl, L, amp=2.0)
        lens = _key_lengths(L, B, L) if masked else None
        if B == 1 and masked:
            lens[0] = max(1, L - 1)
        want = oracle_mod.model_forward(dims, wl.shards, wl.params, wl.x, key_lengths=lens)
        got = _run_masked(gpu, wl, "mfma", lens, "model").float().cpu().numpy()
        assert_parity(got, want, TOL["mfma"], io)


@pytest.mark.parametrize("d,M,f,absent,B,L,masked,outliers,together", [
    (256, 1, 64, 0, 1, 1, False, False, True),       # one head, one token
    (256, 5, 128, 1, 1, 32, True, False, True),      # one whole group of heads, one whole block of keys
    (256, 6, 256, 1, 1, 33, True, False, True),      # a group with one head, a second block with one key
    (768, 12, 256, 1, 1, 64, True, True, True),      # the most keys; weights from the working buffer
    (320, 9, 256, 0, 2, 32, True, False, True),      # several sequences
    (512, 8, 256, 0, 2, 64, True, False, True),
    (256, 20, 256, 1, 1, 40, False, False, True),    # more than 16 weight blocks
    (1024, 13, 256, 1, 1, 64, False, False, True),   # as many workgroups as one launch takes
    (1024, 13, 256, 0, 1, 64, False, False, False),  # one head more
    (256, 12, 64, 0, 1, 23, True, False, False),     # no room for the planes
    (256, 4, 128, 0, 1, 65, True, False, False),     # one key more
])
def test_few_token_attention_with_the_output_projection(gpu, oracle_mod, d, M, f, absent, B, L, masked, outliers, together):
    """Edges of the launch that does both, and both sides of its line; every bitwidth in turn.  One launch counts half its time in
    either class, so that the two sums are the same value; those of two launches are in 10 ns steps, and not the same three times."""
    dims = S.Dims(d, M, 64, f, 1e-12)
    wl = S.small_workload(52000 + d + L, dims, 2, B, L, n_absent=absent, io_dtype="f32")
    if outliers:
        wl = _with_outliers(wl, 5, fraction=0.005)
    S.make_every_term_matter(wl, L, amp=2.0)
    lens = _key_lengths(L, B, L) if masked else None
    if B == 1 and masked:
        lens[0] = max(1, L - 1)
    want = oracle_mod.model_forward(dims, wl.shards, wl.params, wl.x, key_lengths=lens)
    same = []
    for _ in range(3):
        gpu[1].sti_profile_begin()
        got = _run_masked(gpu, wl, "mfma", lens, "model").float().cpu().numpy()
        prof = gpu[1].sti_profile_end()
        assert prof["attention"][0] == prof["gemm_out"][0] == 2
        same.append(prof["attention"][1] == prof["gemm_out"][1])
    assert all(same) == together
    assert_parity(got, want, TOL["mfma"])


def test_less_workspace_than_the_few_token_kernels_take(gpu, oracle_mod):
    """Between the two lines a call that has room for the wide-tile kernels only is accepted and takes those."""
    torch, P, D = gpu
    wl = S.small_workload(41900, S.Dims(768, 12, 64, 256, 1e-12), 1, 5, 140, n_absent=1)
    S.make_every_term_matter(wl, 3, amp=2.0)
    want = oracle_mod.model_forward(wl.dims, wl.shards, wl.params, wl.x)
    shards, params, x = D.upload_workload(wl)
    nbytes = P.sti_workspace_bytes(wl.dims, 5, 140, P.STI_PREC_F16_MFMA)
    for n in (nbytes, nbytes - 1):
        y = torch.full_like(x, float("nan"))
        P.sti_layer_forward(wl.dims, shards[0], params[0], x, y, P.STI_PREC_F16_MFMA, torch.empty(n, dtype=torch.uint8, device="cuda"))
        torch.cuda.synchronize()
        assert_parity(y.cpu().numpy(), want, TOL["mfma"])


@pytest.mark.parametrize("d,M", [(768, 16), (768, 17), (832, 13), (832, 17), (512, 8), (1024, 16)])
@pytest.mark.parametrize("B,L,masked", [(1, 1, False), (1, 33, False), (2, 61, True)])
def test_few_token_rows_in_float32_and_binary16_give_the_same(gpu, d, M, B, L, masked):
    """The Q/K/V projection reads float32 rows as they are with up to 12 K tiles and 16 blocks of weights, else a launch in front of
    it rounds and tiles them: rows that binary16 holds exactly give the layers of binary16 rows on either side of both limits, up to the last
    rounding (to binary16 or not, by two instantiations of LayerNorm: half an ulp of binary16 and a few float32 roundings)."""
    torch, P, D = gpu
    wl = S.small_workload(42000 + d + M, S.Dims(d, M, 64, 128, 1e-12), 2, B, L, n_absent=0, io_dtype="f16")
    S.make_every_term_matter(wl, 5, amp=2.0)
    lens = _key_lengths(L, B, L) if masked else None
    y16 = _run_masked(gpu, wl, "mfma", lens, "model")
    wl.x, wl.io_dtype = wl.x.astype(np.float32), "f32"
    P.sti_profile_begin()
    y32 = _run_masked(gpu, wl, "mfma", lens, "model")
    converted = {k: n for k, (n, _) in P.sti_profile_end().items()}["convert"]
    assert converted == (0 if d <= 768 and M <= 16 else 1)
    assert y32.dtype == torch.float32 and torch.isfinite(y32).all()
    assert ((y32 - y16.float()).abs() <= 2.0 ** -11 * y32.abs() + 2.0 ** -20).all()


def test_any_sufficient_workspace_gives_the_same(gpu):
    """Between the two lines: one layer's buffers, those of several, and the fixed array."""
    torch, P, D = gpu
    wl = S.small_workload(41901, S.Dims(768, 12, 64, 256, 1e-12), 1, 5, 140, n_absent=1)
    S.make_every_term_matter(wl, 3, amp=2.0)
    outs = [_run_masked(gpu, wl, "mfma", None, route) for route in ("layer", "model", "whole")]
    shards, params, x = D.upload_workload(wl)
    store = D.store_from_plan(shards * 3)
    for nbytes in (P.sti_workspace_bytes(wl.dims, 5, 140, P.STI_PREC_F16_MFMA), P.sti_model_workspace_bytes(wl.dims, 3, 5, 140, P.STI_PREC_F16_MFMA)):
        y = torch.full_like(x, float("nan"))
        P.sti_model_forward(wl.dims, store, params * 3, np.concatenate([wl.plan] * 3), x, y, P.STI_PREC_F16_MFMA,
                            torch.empty(nbytes, dtype=torch.uint8, device="cuda"))
        torch.cuda.synchronize()
        outs.append(y)
    y = torch.full_like(x, float("nan"))
    P.sti_layer_forward_static(wl.dims, shards[0], params[0], x, y, P.STI_PREC_F16_MFMA)
    torch.cuda.synchronize()
    assert all(torch.equal(o, y) for o in outs[:3]) and torch.equal(outs[3], outs[4])


@pytest.mark.parametrize("prec,dims,B,L", [("f32", SMALL, 2, 19), ("mfma", MID, 1, 66), ("mfma", MID, 12, 100), ("mfma", MID, 64, 128),
                                           ("f32", S.Dims(768, 12, 64, 256, 1e-12), 4, 107)])   # (planes made behind the LayerNorm)
def test_parameters_begin_at_any_float(gpu, prec, dims, B, L):
    """Biases and LayerNorm parameters 4, 8 and 12 bytes past a 16-byte boundary."""
    import types
    torch, P, D = gpu
    wl = S.small_workload(8600 + L, dims, 1, B, L, io_dtype="f32")
    S.make_every_term_matter(wl, 3)
    shards, params, x = D.upload_workload(wl)
    precision = P.STI_PREC_F32 if prec == "f32" else P.STI_PREC_F16_MFMA
    ws = torch.empty(P.sti_workspace_bytes(dims, B, L, precision), dtype=torch.uint8, device="cuda")
    outs = []
    for shift in range(4):
        moved = types.SimpleNamespace()
        for n, _ in P.StiLayerParams._fields_:
            t = getattr(params[0], n).reshape(-1)
            room = torch.empty(t.numel() + 4, device="cuda")
            room[shift:shift + t.numel()] = t
            setattr(moved, n, room[shift:shift + t.numel()])
            assert getattr(moved, n).data_ptr() % 16 == 4 * shift
        y = torch.full_like(x, float("nan"))
        P.sti_layer_forward(dims, shards[0], moved, x, y, precision, ws)
        torch.cuda.synchronize()
        outs.append(y)
    assert torch.isfinite(outs[0]).all()
    # LayerNorm takes rows with unaligned parameters by single features: other order of its sums.  In binary16 that
    # can move a row's value between the two LayerNorms to its neighbour, 2^-11 of it, which the residual hands on.
    for y in outs[1:]:
        assert torch.equal(y, outs[1])
        assert rel_err(y.cpu().numpy(), outs[0].cpu().numpy().astype(np.float64)) <= (1e-6 if prec == "f32" else 2.0 ** -11)


@pytest.mark.parametrize("prec,d,B,L,absent", [
    ("mfma", 448, 1, 40, False),    # sums of the few-token kernels
    ("mfma", 960, 2, 64, False),
    ("mfma", 832, 1, 23, True),     # bias and residual alone
    ("mfma", 448, 40, 100, False),  # finished binary16 rows, 32 lanes each
    ("mfma", 896, 20, 200, False),
    ("f32", 832, 1, 33, False),
    ("f32", 448, 10, 130, False),   # planes of bfloat16 values behind the row
])
def test_rows_of_equal_values_have_no_variance(gpu, prec, d, B, L, absent):
    """A row of one value throughout is its own mean, so that LayerNorm's result is the shift: sums of small integers are exact
    in any order, and so are their quotients by d.  (Products with a rounded 1 / d are not at these widths, and the
    square of that difference is far above an eps of 1e-12.)"""
    M = d // 64
    wl = S.small_workload(55000 + d + L, S.Dims(d, M, 64, 256, 1e-12), 1, B, L, plan=np.zeros((1, M), dtype=np.int8) if absent else None)
    S.make_every_term_matter(wl, 9, amp=0.0)
    prm = wl.params[0]
    prm.bo[:], prm.ln1_b[:], prm.b2[:] = 1.0, 5.0, 2.0     # both rows: x + 1, and 5 + 2
    wl.x[:] = (np.arange(B * L) % 40).reshape(B, L, 1)
    got = run_gpu(gpu, wl, prec, model=False)
    np.testing.assert_array_equal(got, np.broadcast_to(prm.ln2_b, got.shape))


@pytest.mark.parametrize("d,M,f,B,L,absent,planes", [
    (768, 12, 256, 8, 128, 0, (1, 1)),
    (768, 12, 192, 7, 101, 0, (1, 1)),     # 12 and 36 K tiles
    (768, 12, 256, 11, 93, 2, (0, 1)),
    (1024, 16, 256, 5, 128, 0, (1, 1)),
    (512, 8, 128, 14, 96, 0, (0, 1)),
    (384, 6, 128, 16, 128, 0, (0, 1)),     # 12 K tiles
    (192, 12, 256, 3, 100, 0, (2, 4)),     # K split over workgroups
    (1088, 17, 256, 2, 65, 0, (0, 2)),
])
def test_sums_before_layernorm_keep_what_binary16_would_lose(gpu, d, M, f, B, L, absent, planes):
    """Biases of 0.01 on residual rows of 64, whose neighbours in binary16 are 0.06 away: LayerNorm sees the biases, since few
    tokens' sums reach it in float32.  Bound of an output y with |y| < 5: half a unit of the sum at 64 (3.8e-6) against a spread of
    0.01 in the row and once more in its mean, and y's own rounding, 2^-11 |y|, here twice (h, and LayerNorm over h)."""
    torch, P, D = gpu
    m = M - absent
    have = tuple(tiles.sum_planes(P, kind, B * L, m, d, cols) for kind, cols in ((tiles.O, 64), (tiles.FFN2, f)))
    assert have == planes
    plan = np.full((1, M), 4, dtype=np.int8)
    plan[0, 1:1 + absent] = 0
    wl = S.small_workload(57000 + d + B, S.Dims(d, M, 64, f, 1e-12), 1, B, L, plan=plan, io_dtype="f16")
    S.make_every_term_matter(wl, 10, amp=0.0)
    prm, rng = wl.params[0], np.random.default_rng(d + B)
    normalised = lambda v: (v - v.mean()) / v.std()
    small = (rng.standard_normal(d) * 0.01).clip(-0.04, 0.04).astype(np.float32)
    want = normalised(small.astype(np.float64)).astype(np.float32)
    wl.x[:] = 64.0
    prm.ln1_g[:], prm.ln1_b[:], prm.ln2_g[:], prm.ln2_b[:] = 1.0, 0.0, 1.0, 0.0
    for bo, ln1_b, b2, n in ((small, 0.0, 0.0, planes[0]), (0.0, 64.0, small, planes[1])):     # the first LayerNorm's row, or the second one's
        if n == 0:
            continue
        prm.bo[:], prm.b2[:], prm.ln1_b[:] = bo, b2, ln1_b
        prm.ln1_g[:] = 1.0 if ln1_b == 0.0 else 0.0
        got = run_gpu(gpu, wl, "mfma", model=False)
        bound = 2 * 3.8e-6 / small.std() * (1 + np.abs(want)) + 2 * 2.0 ** -11 * np.abs(want)
        assert np.all(np.abs(got - want) <= bound), float(np.max(np.abs(got - want) / bound))


def test_mfma_rejects_unsupported_dims(gpu):
    torch, P, D = gpu
    assert P.sti_workspace_bytes(SMALL, 1, 8, P.STI_PREC_F16_MFMA) == 0
    wl = S.small_workload(3, SMALL, 1, 1, 8)
    shards, params, xd = D.upload_workload(wl)
    y = torch.empty_like(xd)
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    with pytest.raises(P.StiError) as ei:
        P.sti_layer_forward(SMALL, shards[0], params[0], xd, y, P.STI_PREC_F16_MFMA, ws)
    assert ei.value.status == 2


@pytest.mark.parametrize("prec", ["f32", "mfma"])
@pytest.mark.parametrize("B,L", [(2, 40), (5, 128)])
def test_rejected_calls_report_their_status_and_write_nothing(gpu, prec, B, L):
    """Every argument is checked before the first launch: a call that is rejected because of its last
    layer's plan, its workspace or its buffers leaves the output as it was."""
    torch, P, D = gpu
    precision = P.STI_PREC_F32 if prec == "f32" else P.STI_PREC_F16_MFMA
    wl = S.small_workload(1, MID, 4, B, L, n_absent=1, io_dtype="f16")
    shards, params, x = D.upload_workload(wl)
    store = P.make_store(D.store_from_plan(shards))
    ws = torch.empty(P.sti_model_workspace_bytes(MID, 4, B, L, precision), dtype=torch.uint8, device="cuda")

    def rejected(status, plan=wl.plan, xin=x, workspace=ws):
        y = torch.full_like(x, float("nan"))
        with pytest.raises(P.StiError) as ei:
            P.sti_model_forward(MID, store, params, plan, xin, y, precision, workspace)
        torch.cuda.synchronize()
        assert ei.value.status == status
        assert bool(torch.isnan(y.float()).all())

    present = int(np.argwhere(wl.plan[3] != 0)[0][0])
    plan = wl.plan.copy()
    plan[3, present] = [k for k in (2, 3, 4, 5, 6, 32) if k != wl.plan[3, present]][0]
    rejected(4, plan=plan)                                   # a version the store does not hold
    plan = wl.plan.copy()
    plan[3, present] = 7
    rejected(3, plan=plan)                                   # not a bitwidth
    one_layer = P.sti_workspace_bytes(MID, B, L, precision)  # least the model call can work in
    rejected(6, workspace=ws[:one_layer - 1])                # workspace too small
    shifted = torch.empty(x.numel() + 8, dtype=x.dtype, device="cuda")[1:1 + x.numel()].view_as(x)
    rejected(5, xin=shifted)                                 # input not 16-byte aligned


# ------------------------------------------------------------------ outlier dictionary

def _with_outliers(wl, seed, fraction=0.0015):
    rng = np.random.default_rng(seed)
    for row in wl.shards:
        for s in row:
            if s is not None:
                S.add_outliers(rng, s, wl.dims.weights_per_shard, fraction)
    return wl


@pytest.mark.parametrize("prec,B,L", [("f32", 2, 9), ("mfma", 1, 40), ("mfma", 5, 128)])
def test_layers_apply_outlier_dictionaries(gpu, oracle_mod, prec, B, L):
    wl = _with_outliers(S.small_workload(300 + L, MID, 2, B, L, n_absent=1), 5, fraction=0.05)
    want = oracle_mod.model_forward(MID, wl.shards, wl.params, wl.x)
    plain = [[None if s is None else S.Shard(s.bitwidth, s.data, s.codebook) for s in row]
             for row in wl.shards]
    without = oracle_mod.model_forward(MID, plain, wl.params, wl.x)
    assert rel_err(without, want) > 3 * TOL[prec]     # the dictionaries matter at this tolerance
    got = run_gpu(gpu, wl, prec)
    assert_parity(got, want, TOL[prec])


def test_mfma_whole_model_decode_matches_per_layer_route(gpu, oracle_mod):
    """With a workspace of sti_model_workspace_bytes the layers are decompressed ahead, into a ring of buffers;
    the result must be the very bits of the per-layer route (same kernels, same order of
    arithmetic) and within tolerance of the oracle; outlier dictionaries included."""
    torch, P, D = gpu
    wl = S.small_workload(777, MID, 4, 5, 128, n_absent=1, bit_choices=(2, 3, 4, 5, 6, 32), io_dtype="f16")
    wl = _with_outliers(wl, 3, fraction=0.01)
    prec = P.STI_PREC_F16_MFMA
    shards, params, xd = D.upload_workload(wl)
    store = P.make_store(D.store_from_plan(shards))
    small = P.sti_workspace_bytes(wl.dims, 5, 128, prec)
    big = P.sti_model_workspace_bytes(wl.dims, wl.n_layers, 5, 128, prec)
    assert big > small
    outs = []
    for nbytes in (small, big):
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        y = torch.full_like(xd, float("nan"))
        P.sti_model_forward(wl.dims, store, params, wl.plan, xd, y, prec, ws)
        torch.cuda.synchronize()
        outs.append(y)
    assert torch.equal(outs[0], outs[1])
    want = oracle_mod.model_forward(wl.dims, wl.shards, wl.params, wl.x)
    assert_parity(outs[1].float().cpu().numpy(), want, TOL["mfma"])
    # on the few-token route the query falls back to the one-layer size
    assert P.sti_model_workspace_bytes(wl.dims, wl.n_layers, 1, 128, prec) == P.sti_workspace_bytes(wl.dims, 1, 128, prec)


def _run_model_route(gpu, wl, nbytes, key_lengths=None):
    """sti_model_forward(_masked) on the matrix-core path with a workspace of `nbytes`."""
    torch, P, D = gpu
    shards, params, xd = D.upload_workload(wl)
    store = P.make_store(D.store_from_plan(shards))
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    y = torch.full_like(xd, float("nan"))
    if key_lengths is None:
        P.sti_model_forward(wl.dims, store, params, wl.plan, xd, y, P.STI_PREC_F16_MFMA, ws)
    else:
        P.sti_model_forward_masked(wl.dims, store, params, wl.plan, xd, y,
                                   torch.tensor(key_lengths, dtype=torch.int32, device="cuda"),
                                   P.STI_PREC_F16_MFMA, ws)
    torch.cuda.synchronize()
    return y


def test_mfma_config4_on_the_timed_route_every_sequence(gpu, oracle_mod):
    """Configuration 4 exactly as bench.py times it (Section "Submodel execution": layers in
    order): 12 layers, a workspace of sti_model_workspace_bytes, hence a ring of four working buffers
    and non-zero table offsets; the first layer is decompressed by a launch of its own,
    every other one by the idle workgroups of the Q/K/V + attention launch before it; unmasked.
    All 32 sequences against the oracle; the bits of the per-layer route."""
    torch, P, D = gpu
    wl = S.config4()
    prec = P.STI_PREC_F16_MFMA
    big = P.sti_model_workspace_bytes(wl.dims, wl.n_layers, wl.batch, wl.seq, prec)
    small = P.sti_workspace_bytes(wl.dims, wl.batch, wl.seq, prec)
    layer_w16 = wl.dims.n_heads * wl.dims.weights_per_shard * 2
    assert 3 * layer_w16 <= big - small < 4 * layer_w16      # a ring of four working buffers: the 12 layers wrap it three times
    timed = _run_model_route(gpu, wl, big)
    per_layer = _run_model_route(gpu, wl, small)
    assert torch.equal(timed, per_layer)
    want = oracle_mod.model_forward(wl.dims, wl.shards, wl.params, wl.x)
    got = timed.float().cpu().numpy()
    assert_parity(got, want, TOL["mfma"])
    for b in range(wl.batch):
        assert_parity(got[b], want[b], TOL["mfma"], b)


def test_next_layer_decompressed_beside_the_projection_with_outlier_dictionaries(gpu, oracle_mod):
    """32 sequences of 128 tokens with 9 of 12 shards per layer: the fused Q/K/V + attention launch
    has 160 tiles (the last pair of heads is half empty), and the whole-model route lets its idle
    workgroups decompress the following layer (Section "Submodel execution": the next layer is made
    ready while this one computes); the outlier dictionaries of that layer go in behind the launch.
    Bits of the per-layer route, oracle on every sequence."""
    torch, P, D = gpu
    wl = S.small_workload(515, S.BERT_BASE, 4, 32, 128, n_absent=3, bit_choices=(2, 3, 4, 5, 6, 32), io_dtype="f16")
    wl = _with_outliers(wl, 17, fraction=0.01)
    S.make_every_term_matter(wl, 29, amp=2.0)
    prec = P.STI_PREC_F16_MFMA
    big = P.sti_model_workspace_bytes(wl.dims, wl.n_layers, wl.batch, wl.seq, prec)
    small = P.sti_workspace_bytes(wl.dims, wl.batch, wl.seq, prec)
    rolling = _run_model_route(gpu, wl, big)
    per_layer = _run_model_route(gpu, wl, small)
    assert torch.equal(rolling, per_layer)
    want = oracle_mod.model_forward(wl.dims, wl.shards, wl.params, wl.x)
    got = rolling.float().cpu().numpy()
    assert_parity(got, want, TOL["mfma"])
    for b in range(wl.batch):
        assert_parity(got[b], want[b], TOL["mfma"], b)


@pytest.mark.parametrize("B,L,entries", [
    (11, 93, 1),        # one entry per dictionary; K of the output projection split over workgroups
    (11, 93, 769),      # one more than a workgroup takes
    (9, 113, 5461),     # 12 shards: the most entries that go in beside the projection ...
    (9, 113, 5462),     # ... and one more, by a launch of their own
    (32, 128, 885),     # the projection's tiles fill the chip
    (26, 61, 256),
])
def test_outlier_dictionaries_beside_the_output_projection(gpu, B, L, entries):
    """The dictionaries of a layer that was decompressed beside its predecessor's Q/K/V projection: the bits of
    the per-layer route, where a launch of their own puts them in."""
    torch, P, D = gpu
    dims = S.BERT_BASE
    plan = np.full((3, 12), 3, dtype=np.int8)
    plan[1, ::3] = 32          # shards without a dictionary among those with one
    plan[2] = 5
    wl = S.small_workload(700 + entries, dims, 3, B, L, plan=plan, io_dtype="f16")
    wl = _with_outliers(wl, entries, fraction=entries / dims.weights_per_shard)
    assert all(len(s.outlier_pos) == entries for s in wl.shards[2])
    prec = P.STI_PREC_F16_MFMA
    big = P.sti_model_workspace_bytes(dims, 3, B, L, prec)
    small = P.sti_workspace_bytes(dims, B, L, prec)
    assert big > small
    whole = _run_model_route(gpu, wl, big)
    assert torch.equal(whole, _run_model_route(gpu, wl, small))
    assert torch.isfinite(whole.float()).all()


@pytest.mark.parametrize("d,M,f,absent,B,L,entries", [
    (768, 12, 256, (0, 1, 1), 11, 93, 1),       # K of the output projection split over workgroups
    (768, 12, 256, (0, 1, 1), 11, 93, 769),
    (768, 12, 256, (0, 1, 1), 9, 113, 5957),    # 11 shards: the most entries beside the output projection ...
    (768, 12, 256, (0, 1, 1), 9, 113, 5958),    # ... and one more
    (768, 12, 256, (2, 2, 2), 60, 64, 3),       # the fastest tiles of Q/K/V alone would leave no compute unit ...
    (1024, 16, 256, (0, 0, 0), 40, 64, 2),
    (768, 12, 256, (2, 2, 2), 56, 64, 0),       # ... or too few
    (1024, 4, 64, (0, 1, 1), 28, 100, 300),     # output projection in 64 x 384 tiles, where 128 x 256 alone would be faster ...
    (1024, 8, 64, (0, 1, 1), 55, 100, 257),     # ... and in 64 x 192, two to a unit
])
def test_a_layer_rides_where_that_is_faster_than_a_launch_of_its_own(gpu, d, M, f, absent, B, L, entries):
    """Layers behind the first are decompressed beside the Q/K/V projection in front of them (one decompression
    launch in all), their dictionaries beside its output projection: the bits of the per-layer route."""
    torch, P, D = gpu
    dims = S.Dims(d, M, 64, f, 1e-12)
    plan = np.full((3, M), 4, dtype=np.int8)
    for l, n in enumerate(absent):
        plan[l, 1:1 + n] = 0
    if entries:
        beside = tiles.layer_tiles(gpu[1], dims, B * L, M - absent[0], outliers=entries)["o"]
        assert beside == {1024 * 28 * 100: "64x384/132", 1024 * 55 * 100: "64x192/516"}.get(d * B * L, f"64x192*/{-(-d // 192) * -(-B * L // 64)}")
    wl = S.small_workload(810 + entries, dims, 3, B, L, plan=plan, io_dtype="f16")
    if entries:
        wl = _with_outliers(wl, entries, fraction=entries / dims.weights_per_shard)
    prec = P.STI_PREC_F16_MFMA
    P.sti_profile_begin()
    whole = _run_model_route(gpu, wl, P.sti_model_workspace_bytes(dims, 3, B, L, prec))
    assert P.sti_profile_end()["decode"][0] == 1
    assert torch.equal(whole, _run_model_route(gpu, wl, P.sti_workspace_bytes(dims, B, L, prec)))
    assert torch.isfinite(whole.float()).all()


@pytest.mark.parametrize("d,M,f,absent,B,L,entries,carrier,tile,planes", [
    (768, 12, 256, 0, 32, 128, 885, "o", "64x192*/256", 0),
    (1024, 8, 64, 0, 55, 100, 257, "o", "64x192/516", 0),         # 128 x 256 tiles alone ...
    (1024, 6, 64, 0, 41, 100, 300, "o", "64x384/195", 0),         # ... and next to 64 x 384
    (768, 12, 256, 0, 11, 93, 769, "ffn2", "64x64*/192", 1),      # one entry more than three workgroups of 256 threads take
    (768, 12, 256, 2, 11, 93, 900, "ffn2", "64x64*/192", 1),
    (768, 12, 256, 6, 34, 100, 100, "ffn2", "64x192*/216", 0),    # O alone with K not shared by groups of waves
    (192, 12, 256, 0, 3, 100, 200, "ffn2", "32x96*/20", 4),       # K split over workgroups, one in four of which has entries to put in
    (1088, 17, 256, 0, 2, 65, 400, "ffn2", "32x96*/60", 2),
])
def test_outlier_dictionaries_beside_o_or_ffn2(gpu, d, M, f, absent, B, L, entries, carrier, tile, planes):
    """Which of the two projections takes the next layer's dictionaries along, in which tile and with how many planes of sums: the bits of
    the per-layer route, where a launch of their own puts them in."""
    torch, P, D = gpu
    dims, m = S.Dims(d, M, 64, f, 1e-12), M - absent
    assert tiles.out_carries(P, dims, B * L, m, entries) == (carrier == "o")
    assert tiles.layer_tiles(P, dims, B * L, m, entries if carrier == "o" else 0)[carrier] == tile
    assert tiles.sum_planes(P, tiles.O if carrier == "o" else tiles.FFN2, B * L, m, d, 64 if carrier == "o" else f, entries) == planes
    plan = np.full((3, M), 4, dtype=np.int8)
    plan[:, m:] = 0
    wl = S.small_workload(820 + entries, dims, 3, B, L, plan=plan, io_dtype="f16")
    wl = _with_outliers(wl, entries, fraction=entries / dims.weights_per_shard)
    S.make_every_term_matter(wl, 31, amp=2.0)
    prec = P.STI_PREC_F16_MFMA
    P.sti_profile_begin()
    whole = _run_model_route(gpu, wl, P.sti_model_workspace_bytes(dims, 3, B, L, prec))
    assert P.sti_profile_end()["decode"][0] == 1
    assert torch.equal(whole, _run_model_route(gpu, wl, P.sti_workspace_bytes(dims, B, L, prec)))
    assert torch.isfinite(whole.float()).all()


def test_layers_that_can_and_cannot_take_the_next_layer_along(gpu, oracle_mod):
    """38 sequences: a full layer has 228 tiles and no compute unit to spare, a layer with 9 or 10 shards
    190 tiles and 64; with an all-absent layer in between.  Layers 0 to 3 are decompressed as a group,
    layer 3 takes layer 4 along, layer 5 is decompressed alone."""
    torch, P, D = gpu
    rng = np.random.default_rng(77)
    plan = rng.choice([2, 3, 4, 5, 6, 32], size=(6, 12)).astype(np.int8)
    plan[1, [2, 7]] = 0
    plan[2, :] = 0
    plan[3, [0, 5, 11]] = 0
    plan[5, [4, 9]] = 0
    wl = S.small_workload(616, S.BERT_BASE, 6, 38, 128, plan=plan, io_dtype="f16")
    wl = _with_outliers(wl, 19, fraction=0.005)
    prec = P.STI_PREC_F16_MFMA
    big = P.sti_model_workspace_bytes(wl.dims, wl.n_layers, wl.batch, wl.seq, prec)
    small = P.sti_workspace_bytes(wl.dims, wl.batch, wl.seq, prec)
    mixed = _run_model_route(gpu, wl, big)
    per_layer = _run_model_route(gpu, wl, small)
    assert torch.equal(mixed, per_layer)
    want = oracle_mod.model_forward(wl.dims, wl.shards, wl.params, wl.x)
    assert_parity(mixed.float().cpu().numpy(), want, TOL["mfma"])


def test_whole_model_route_random_sweep_is_the_per_layer_route(gpu):
    """Seeded sweep over 128-token batches of 6 to 43 sequences, three shapes, 2 to 5 layers with 0 to all
    shards absent per layer, with and without outlier dictionaries and key lengths: whichever layers
    are decompressed by launches of their own or beside their predecessor's projection, the whole-model
    route gives the bits of the per-layer route (which the other tests hold against the oracle)."""
    torch, P, D = gpu
    prec = P.STI_PREC_F16_MFMA
    rng = np.random.default_rng(2024)
    shapes = [S.BERT_BASE, S.Dims(512, 8, 64, 256, 1e-12), S.Dims(1024, 16, 64, 256, 1e-12)]
    for it in range(18):
        dims = shapes[it % 3]
        M = dims.n_heads
        n_layers = int(rng.integers(2, 6))
        B = int(rng.integers(6, 44))
        plan = rng.choice([2, 3, 4, 5, 6, 32], size=(n_layers, M)).astype(np.int8)
        for l in range(n_layers):
            k = int(rng.integers(0, M + 1)) if rng.random() < 0.15 else int(rng.integers(0, 5))
            plan[l, rng.choice(M, k, replace=False)] = 0
        wl = S.small_workload(9000 + it, dims, n_layers, B, 128, plan=plan, io_dtype="f16")
        if it % 2:
            wl = _with_outliers(wl, it, fraction=0.003)
        lengths = rng.integers(1, 129, size=B).astype(np.int32) if it % 4 == 3 else None
        big = P.sti_model_workspace_bytes(dims, n_layers, B, 128, prec)
        small = P.sti_workspace_bytes(dims, B, 128, prec)
        whole = _run_model_route(gpu, wl, big, key_lengths=lengths)
        per_layer = _run_model_route(gpu, wl, small, key_lengths=lengths)
        assert torch.equal(whole, per_layer), (it, dims.d_model, B, [int((plan[l] != 0).sum()) for l in range(n_layers)])
        assert torch.isfinite(whole.float()).all()


def test_mfma_one_layer_per_decompression_group_with_outlier_dictionaries(gpu, oracle_mod):
    """d_model 2048 with 32 shards: one layer's working buffer (100 MB) alone exceeds a 64 MiB group,
    so every layer of the whole-model route is a group of its own (table and buffer offsets of
    layers 1 and 2 are non-zero); outlier dictionaries on every shard, two shards absent per layer."""
    torch, P, D = gpu
    dims = S.Dims(2048, 32, 64, 256, 1e-12)
    wl = S.small_workload(4242, dims, 3, 2, 128, n_absent=2, bit_choices=(2, 3, 4, 5, 6, 32), io_dtype="f16")
    wl = _with_outliers(wl, 11, fraction=0.01)
    S.make_every_term_matter(wl, 23, amp=2.0)
    prec = P.STI_PREC_F16_MFMA
    big = P.sti_model_workspace_bytes(dims, wl.n_layers, 2, 128, prec)
    small = P.sti_workspace_bytes(dims, 2, 128, prec)
    assert dims.n_heads * dims.weights_per_shard * 2 > (64 << 20) and big > small
    grouped = _run_model_route(gpu, wl, big)
    per_layer = _run_model_route(gpu, wl, small)
    assert torch.equal(grouped, per_layer)
    want = oracle_mod.model_forward(dims, wl.shards, wl.params, wl.x)
    assert_parity(grouped.float().cpu().numpy(), want, TOL["mfma"])


WIDE = S.Dims(128, 12, 64, 64, 1e-12)


@pytest.mark.parametrize("prec,dims,B,L", [("f32", SMALL, 2, 19), ("mfma", MID, 1, 66), ("mfma", MID, 3, 100),
                                           ("mfma", WIDE, 5, 128), ("mfma", WIDE, 9, 256), ("mfma", MID, 2, 200),
                                           ("mfma", MID, 2, 300)])
def test_every_term_of_the_layer_matters(gpu, oracle_mod, prec, dims, B, L):
    """With the configurations' recipe a kernel could leave out the score scale, bq or b1, or a
    LayerNorm gain, and stay inside the binary16 tolerance (tests/test_oracle_layer.py measures
    that on the reference).  Here weights are six times as large and gains, shifts and biases
    are random, on every route: float32; few-token, partial-sum and wide-tile matrix-core
    GEMMs; attention with all scores in registers (up to 128 keys) and with the running maximum
    (more keys)."""
    wl = S.small_workload(31000 + B * L, dims, 2, B, L, n_absent=1, io_dtype="f32" if prec == "f32" else "f16")
    S.make_every_term_matter(wl, 77 + B)
    want = oracle_mod.model_forward(dims, wl.shards, wl.params, wl.x)
    got = run_gpu(gpu, wl, prec)
    assert_parity(got, want, TOL[prec])


def test_mfma_many_column_tiles_take_the_band_order(gpu, oracle_mod):
    """More than 12 column tiles (here 32 shards: 16 column tiles for Q/K/V, 22 for FFN1) make the
    wide-tile GEMM walk its tiles in bands of 8 row tiles; 11 row tiles leave a short last band
    and 1400 tokens a ragged last row tile."""
    dims = S.Dims(128, 32, 64, 256, 1e-12)
    wl = S.small_workload(2048, dims, 1, 7, 200, n_absent=3, io_dtype="f16")
    S.make_every_term_matter(wl, 9, amp=3.0)
    want = oracle_mod.model_forward(dims, wl.shards, wl.params, wl.x)
    got = run_gpu(gpu, wl, "mfma")
    assert_parity(got, want, TOL["mfma"])


@pytest.mark.parametrize("B,L,n_absent", [(40, 150, 0), (37, 161, 1)])
def test_mfma_many_tiles_shared_compute_units(gpu, oracle_mod, B, L, n_absent):
    """Q/K/V in one tile of 256 x 256 per compute unit, FFN1 in up to two of 192 x 256: part tiles in both directions."""
    dims = S.Dims(256, 12, 64, 256, 1e-12)
    chosen = tiles.layer_tiles(gpu[1], dims, B * L, dims.n_heads - n_absent)
    assert chosen["qkv"] == "256x256L/216" and chosen["ffn1"] == ("192x256L/352" if n_absent else "192x256L/384")
    wl = S.small_workload(52000 + B, dims, 1, B, L, n_absent=n_absent, io_dtype="f16")
    S.make_every_term_matter(wl, B, amp=2.0)
    want = oracle_mod.model_forward(dims, wl.shards, wl.params, wl.x)
    assert_parity(run_gpu(gpu, wl, "mfma"), want, TOL["mfma"])


@pytest.mark.parametrize("n_absent", [0, 1])
def test_mfma_output_projections_with_shared_compute_units(gpu, oracle_mod, n_absent):
    """O, FFN1 and FFN2 in 128 x 256 tiles, Q/K/V in up to two of 192 x 256 per compute unit, residual and a ragged last row tile:
    sampled sequences, the last tile's among them."""
    dims = S.Dims(1024, 16, 64, 64, 1e-12)
    assert tiles.layer_tiles(gpu[1], dims, 5500, 16 - n_absent) == {"qkv": "192x256L/348", "o": "128x256L/172", "ffn1": "128x256L/172",
                                                                    "ffn2": "128x256L/172"}
    wl = S.small_workload(53000, dims, 1, 55, 100, n_absent=n_absent, io_dtype="f16")
    S.make_every_term_matter(wl, 6, amp=2.0)
    got = run_gpu(gpu, wl, "mfma")
    assert np.all(np.isfinite(got))
    for b in (0, 21, 53, 54):
        want = oracle_mod.model_forward(dims, wl.shards, wl.params, wl.x[b:b + 1])
        assert_parity(got[b:b + 1], want, TOL["mfma"], b)


@pytest.mark.parametrize("d,M,f,B,L,n_absent,chosen", [
    (128, 32, 256, 23, 259, 0, {"qkv": "192x256L/768", "ffn1": "192x256L/1024"}),    # three and four tiles to a workgroup, K of two tiles, bands of row tiles
    (1024, 16, 64, 44, 125, 0, {"qkv": "192x256L/348", "o": "128x256L/172", "ffn2": "128x256L/172"}),   # residual, a last tile of 124 rows
    (448, 14, 128, 25, 360, 0, {"ffn1": "256x256L/252", "o": "128x256L/142", "ffn2": "128x256L/142"}),  # 192 columns in the last column tile
    (1024, 2, 64, 31, 297, 0, {"o": "192x256L/192", "ffn2": "192x256L/192"}),        # K of two tiles
    (256, 12, 256, 40, 150, 1, {"qkv": "256x256L/216"}),                             # 64 columns in the last column tile
    (128, 29, 256, 7, 200, 0, {"qkv": "128x256L/242"}),
])
def test_mfma_large_tiles(gpu, oracle_mod, d, M, f, B, L, n_absent, chosen):
    """Tiles of 128, 192 and 256 rows x 256 columns: first, middle and last sequences against the oracle (sequences do not
    depend on each other), all rows finite."""
    dims = S.Dims(d, M, 64, f, 1e-12)
    assert chosen.items() <= tiles.layer_tiles(gpu[1], dims, B * L, M - n_absent).items()
    wl = S.small_workload(54000 + d + M, dims, 1, B, L, n_absent=n_absent, io_dtype="f16")
    S.make_every_term_matter(wl, 8, amp=2.0)
    got = run_gpu(gpu, wl, "mfma")
    assert np.all(np.isfinite(got))
    for b in (0, B // 2, B - 1):
        want = oracle_mod.model_forward(dims, wl.shards, wl.params, wl.x[b:b + 1])
        assert_parity(got[b:b + 1], want, TOL["mfma"], b)


@pytest.mark.parametrize("prec,d,M,f,B,L", [
    ("mfma", 128, 4, 64, 3, 100),        # kernels for many tokens, small tiles
    ("mfma", 768, 12, 256, 32, 128),     # 128 x 384
    ("mfma", 128, 32, 512, 20, 207),     # 192 x 256
    ("mfma", 256, 4, 64, 1, 50),         # for few tokens
    ("f32", 256, 4, 64, 1, 50),
    ("f32", 768, 12, 256, 4, 128),       # planes of three bfloat16 values
])
@pytest.mark.parametrize("value", [float("-inf"), float("inf"), float("nan")])
def test_an_argument_of_gelu_that_is_no_number_is_not_lost(gpu, prec, d, M, f, B, L, value):
    """One neuron's bias is infinite or NaN: no row of the layer is finite (-inf Phi(-inf) is -inf times zero), on any route."""
    dims = S.Dims(d, M, 64, f, 1e-12)
    if (d, M) in ((768, 12), (128, 32)) and prec == "mfma":
        assert tiles.layer_tiles(gpu[1], dims, B * L, M)["ffn1"].startswith("128x384" if d == 768 else "192x256L")
    wl = S.small_workload(61000 + d, dims, 1, B, L)
    wl.params[0].b1[f + 5] = value
    assert not np.isfinite(run_gpu(gpu, wl, prec)).any()


@pytest.mark.parametrize("k_tiles", range(1, 10))
def test_mfma_k_tiles_in_and_out_of_whole_rounds(gpu, oracle_mod, k_tiles):
    """K loops of one to nine K tiles (rounds of three whose loads all exist, then the rest): 64-row tiles with unsplit K (Q/K/V and
    FFN1), K shared evenly and unevenly by two groups of waves (O and FFN2), Q/K/V tiles of whole sequences, and tiles of 192 rows."""
    for M, B, L, chosen in ((k_tiles + 1, 11, 100, {"ffn2": "32x96*"} if k_tiles > 2 else None), (8, 32, 128, None),
                            (32, 17, 100, {"qkv": "192x256L"} if k_tiles > 1 else None)):
        dims = S.Dims(64 * k_tiles, M, 64, 64, 1e-12)
        have = tiles.layer_tiles(gpu[1], dims, B * L, M)
        assert chosen is None or all(have[name].split("/")[0] == shape for name, shape in chosen.items()), have
        wl = S.small_workload(58000 + 10 * k_tiles + B, dims, 1, B, L, io_dtype="f16")
        S.make_every_term_matter(wl, 8, amp=2.0)
        got = run_gpu(gpu, wl, "mfma")
        assert np.all(np.isfinite(got))
        for b in (0, B // 2, B - 1):
            want = oracle_mod.model_forward(dims, wl.shards, wl.params, wl.x[b:b + 1])
            assert_parity(got[b:b + 1], want, TOL["mfma"], (M, b))


@pytest.mark.parametrize("d,M,f,B,L,n_absent,chosen", [
    (768, 12, 256, 11, 93, 2, {"qkv": "64x128/240", "o": "32x96*/256", "ffn2": "64x64*/192"}),
    (768, 12, 256, 12, 93, 1, {"o": "64x64*/216", "ffn1": "64x128/396", "ffn2": "64x64*/216"}),    # eleven K tiles to two groups
    (768, 12, 256, 16, 127, 0, {"o": "64x96*/256"}),
    (704, 7, 192, 13, 111, 0, {"qkv": "64x128/253", "o": "64x64*/253"}),
    (832, 8, 64, 13, 111, 0, {"o": "64x96*/207", "ffn2": "64x96*/207"}),   # 64 columns in the last column tile, a ragged last row tile
    (448, 5, 64, 5, 301, 0, {"o": "32x96*/240", "ffn1": "64x128/72"}),   # 64 columns in the last column tile, five K tiles
])
def test_mfma_small_tiles(gpu, oracle_mod, d, M, f, B, L, n_absent, chosen):
    """Tiles of few values, K shared by two groups of waves or not: all rows against the float32 route, some against the oracle."""
    dims = S.Dims(d, M, 64, f, 1e-12)
    assert chosen.items() <= tiles.layer_tiles(gpu[1], dims, B * L, M - n_absent).items()
    wl = S.small_workload(59000 + d + L, dims, 1, B, L, n_absent=n_absent, io_dtype="f16")
    S.make_every_term_matter(wl, 8, amp=2.0)
    got = run_gpu(gpu, wl, "mfma")
    for b in (0, B - 1):
        want = oracle_mod.model_forward(dims, wl.shards, wl.params, wl.x[b:b + 1])
        assert_parity(got[b:b + 1], want, TOL["mfma"], b)
    assert_parity(got, run_gpu(gpu, wl, "f32"), TOL["mfma"])


@pytest.mark.parametrize("d,M,f,B,L,n_absent,chosen", [
    (128, 9, 192, 74, 125, 0, {"qkv": "128x256L/511", "ffn1": "128x256L/511"}),      # two K tiles
    (128, 32, 512, 20, 207, 1, {"qkv": "256x256L/408", "ffn1": "192x256L/1364"}),    # bands of row tiles, up to six to a workgroup
    (128, 12, 512, 20, 205, 0, {"ffn1": "256x256L/408"}),
    (1024, 12, 256, 99, 93, 0, {"qkv": "192x256L/432", "ffn1": "256x256L/432"}),     # many K tiles
    (1536, 2, 64, 27, 300, 0, {"o": "128x256L/384", "ffn2": "128x256L/384"}),        # residual rows, two K tiles
    (2048, 8, 64, 62, 100, 0, {"o": "128x256L/392", "ffn2": "128x256L/392"}),
    (2048, 7, 64, 60, 151, 0, {"o": "192x256L/384", "ffn2": "192x256L/384"}),        # an odd number of K tiles: stages change places
])
def test_mfma_large_tiles_one_after_another(gpu, oracle_mod, d, M, f, B, L, n_absent, chosen):
    """More than 256 tiles of every height, with and without residual: a workgroup's second tile begins in stages that were filled
    during the first one's last K tiles and its epilogue.  All rows against the float32 route, the ends and the middle against
    the oracle."""
    dims = S.Dims(d, M, 64, f, 1e-12)
    assert chosen.items() <= tiles.layer_tiles(gpu[1], dims, B * L, M - n_absent).items()
    wl = S.small_workload(56000 + d + M, dims, 1, B, L, n_absent=n_absent, io_dtype="f16")
    S.make_every_term_matter(wl, 8, amp=2.0)
    got = run_gpu(gpu, wl, "mfma")
    for b in (0, B // 2, B - 1):
        want = oracle_mod.model_forward(dims, wl.shards, wl.params, wl.x[b:b + 1])
        assert_parity(got[b:b + 1], want, TOL["mfma"], b)
    assert_parity(got, run_gpu(gpu, wl, "f32"), TOL["mfma"])


@pytest.mark.parametrize("B,L", [(1, 64), (3, 100)])   # few-token route / working-buffer route
def test_mfma_widest_supported_model(gpu, oracle_mod, B, L):
    """d_model 2048 (rows of 2048 features in LayerNorm, K = 2048 in the projections, 22-26 column
    tiles) with 32 shards of which two are absent; weights twice the recipe's scale."""
    dims = S.Dims(2048, 32, 64, 256, 1e-12)
    wl = S.small_workload(77, dims, 1, B, L, n_absent=2, io_dtype="f16")
    S.make_every_term_matter(wl, 21, amp=2.0)
    want = oracle_mod.model_forward(dims, wl.shards, wl.params, wl.x)
    got = run_gpu(gpu, wl, "mfma")
    assert_parity(got, want, TOL["mfma"])


@pytest.mark.parametrize("d_model", [2112, 4096])
@pytest.mark.parametrize("B,L", [(1, 40), (3, 100)])   # few-token route / working-buffer route
def test_mfma_rows_longer_than_2048_features(gpu, oracle_mod, d_model, B, L):
    """d_model beyond what the row kernels keep in registers (the working-buffer route once
    failed here, after its first launches, with a HIP error from the LayerNorm launcher)."""
    dims = S.Dims(d_model, 4, 64, 64, 1e-12)
    wl = S.small_workload(5, dims, 2, B, L, n_absent=1, io_dtype="f16")
    S.make_every_term_matter(wl, 8, amp=2.0)
    want = oracle_mod.model_forward(dims, wl.shards, wl.params, wl.x)
    got = run_gpu(gpu, wl, "mfma")
    # (gains up to 1.9 on rows of 4096 features with doubled weights: at d_model 4096, 1 of 163,840 and
    #  8 of 1,228,800 elements were measured past the per-element bound; none at d_model 2112)
    assert_parity(got, want, TOL["mfma"], max_violations=1e-4 if d_model == 4096 else 0.0)


def test_mfma_rows_beyond_2gib_of_activations(gpu):
    """350,000 tokens: the FFN activations (T x 3072 binary16) pass 2 GiB, so row addresses need
    64 bits.  Sequences are independent, so the first and the last sequence of the big batch
    must come out as when they run alone (up to the summation order of other tile shapes)."""
    torch, P, D = gpu
    dims = S.BERT_BASE
    B, L = 700, 500
    wl = S.small_workload(4242, dims, 1, 2, L, io_dtype="f16")
    shards, params, x2 = D.upload_workload(wl)
    prec = P.STI_PREC_F16_MFMA
    gen = torch.Generator(device="cuda").manual_seed(7)
    x = torch.randn(B, L, dims.d_model, device="cuda", generator=gen).to(torch.float16)
    x[0] = x2[0]
    x[B - 1] = x2[1]
    y = torch.empty_like(x)
    ws = torch.empty(P.sti_workspace_bytes(dims, B, L, prec), dtype=torch.uint8, device="cuda")
    P.sti_layer_forward(dims, shards[0], params[0], x, y, prec, ws)
    y2 = torch.empty_like(x2)
    ws2 = torch.empty(P.sti_workspace_bytes(dims, 2, L, prec), dtype=torch.uint8, device="cuda")
    P.sti_layer_forward(dims, shards[0], params[0], x2, y2, prec, ws2)
    torch.cuda.synchronize()
    assert torch.isfinite(y).all()
    for big, alone in ((y[0], y2[0]), (y[B - 1], y2[1])):
        assert_parity(big.float().cpu().numpy(), alone.float().cpu().numpy(), 4e-3)


def test_model_forward_can_be_stream_captured(gpu, oracle_mod):
    """The few-token path enqueues kernels only (no copies, no fills, no host waits), so a
    caller may capture it into a graph; replays, with eager calls between them, must give the
    eager result every time."""
    torch, P, D = gpu
    wl = S.small_workload(888, MID, 3, 2, 100, n_absent=1, io_dtype="f16")
    prec = P.STI_PREC_F16_MFMA
    shards, params, x = D.upload_workload(wl)
    store = P.make_store(D.store_from_plan(shards))
    ws = torch.empty(P.sti_workspace_bytes(MID, 2, 100, prec), dtype=torch.uint8, device="cuda")
    y_eager = torch.empty_like(x)
    P.sti_model_forward(MID, store, params, wl.plan, x, y_eager, prec, ws)
    torch.cuda.synchronize()
    want = oracle_mod.model_forward(MID, wl.shards, wl.params, wl.x)
    assert_parity(y_eager.float().cpu().numpy(), want, TOL["mfma"])
    y_graph = torch.full_like(x, float("nan"))
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            P.sti_model_forward(MID, store, params, wl.plan, x, y_graph, prec, ws)
    torch.cuda.synchronize()
    for _ in range(3):
        y_graph.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y_graph, y_eager)
        scratch = torch.empty_like(x)
        P.sti_model_forward(MID, store, params, wl.plan, x, scratch, prec, ws)   # eager work between replays
        torch.cuda.synchronize()
        assert torch.equal(scratch, y_eager)


def test_capture_never_records_the_shard_table_upload(gpu, oracle_mod):
    """With the model workspace the eager call takes the grouped route, whose shard table is
    uploaded through a pinned host buffer that later calls overwrite; a captured call must not
    record that copy: it runs the per-layer route (same bits), and replays stay right after
    eager calls with OTHER plans have reused the pinned buffer.  sti_decode_shards with more than
    64 shards, which has no other route, refuses to be captured."""
    torch, P, D = gpu
    wl = S.small_workload(4321, MID, 3, 3, 100, n_absent=1, io_dtype="f16")
    other = S.small_workload(1234, MID, 3, 3, 100, n_absent=2, io_dtype="f16")
    prec = P.STI_PREC_F16_MFMA
    shards, params, x = D.upload_workload(wl)
    store = P.make_store(D.store_from_plan(shards))
    o_shards, o_params, o_x = D.upload_workload(other)
    o_store = P.make_store(D.store_from_plan(o_shards))
    nbytes = P.sti_model_workspace_bytes(MID, 3, 3, 100, prec)
    assert nbytes > P.sti_workspace_bytes(MID, 3, 100, prec)
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    y_eager = torch.empty_like(x)
    P.sti_model_forward(MID, store, params, wl.plan, x, y_eager, prec, ws)
    torch.cuda.synchronize()
    assert_parity(y_eager.float().cpu().numpy(), oracle_mod.model_forward(MID, wl.shards, wl.params, wl.x), TOL["mfma"])
    y_graph = torch.full_like(x, float("nan"))
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            P.sti_model_forward(MID, store, params, wl.plan, x, y_graph, prec, ws)
    torch.cuda.synchronize()
    o_ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    o_y = torch.empty_like(o_x)
    for _ in range(3):
        for _ in range(5):   # more eager uploads than the pinned ring has slots
            P.sti_model_forward(MID, o_store, o_params, other.plan, o_x, o_y, prec, o_ws)
        torch.cuda.synchronize()
        y_graph.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y_graph, y_eager)
    # decode: 70 shards need the uploaded table
    n = 4096
    host = [S.make_shard(np.random.default_rng(s), n, 2 + s % 5) for s in range(70)]
    dev = [D.upload_shard(s) for s in host]
    out = torch.zeros(70 * n, dtype=torch.float16, device="cuda")
    dws = torch.empty(P.sti_decode_workspace_bytes(70), dtype=torch.uint8, device="cuda")
    g2 = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(g2, stream=side):
            with pytest.raises(P.StiError) as err:
                P.sti_decode_shards(dev, n, out, dws)
            P.sti_decode_shards(dev[:64], n, out[:64 * n], None)   # at most 64 shards: kernels only
    assert err.value.status == 9   # STI_ERR_UNSUPPORTED
    torch.cuda.synchronize()
    g2.replay()
    torch.cuda.synchronize()
    got = out.view(torch.int16).cpu().numpy().view(np.uint16).reshape(70, n)
    assert np.array_equal(got[:64], oracle_mod.decode_shards(host[:64], n, oracle_mod.F16))
    assert not got[64:].any()
    P.sti_decode_shards(dev, n, out, dws)   # eager: accepted
    torch.cuda.synchronize()
    got = out.view(torch.int16).cpu().numpy().view(np.uint16).reshape(70, n)
    assert np.array_equal(got, oracle_mod.decode_shards(host, n, oracle_mod.F16))


@pytest.mark.parametrize("B,L", [(1, 64), (4, 128)])   # few-token route / working-buffer route
def test_per_kernel_timing_counts_every_launch_and_changes_nothing(gpu, B, L):
    """sti_profile_begin/end: the launches carry timing events; the counts per kernel class
    are those of the route, every class with launches has a positive time, the sum of the
    kernel times is below the wall time of the forward, and the output is bit for bit what an
    untimed call gives."""
    import time
    torch, P, D = gpu
    n_layers = 3
    wl = S.small_workload(4100 + L, MID, n_layers, B, L, io_dtype="f16")
    shards, params, x = D.upload_workload(wl)
    store = P.make_store(D.store_from_plan(shards))
    prec = P.STI_PREC_F16_MFMA
    ws = torch.empty(P.sti_model_workspace_bytes(MID, n_layers, B, L, prec), dtype=torch.uint8, device="cuda")
    y0 = torch.empty_like(x)
    P.sti_model_forward(MID, store, params, wl.plan, x, y0, prec, ws)
    torch.cuda.synchronize()
    y1 = torch.full_like(x, float("nan"))
    P.sti_profile_begin()
    t0 = time.perf_counter()
    P.sti_model_forward(MID, store, params, wl.plan, x, y1, prec, ws)
    prof = P.sti_profile_end()          # waits for the events
    wall_ms = (time.perf_counter() - t0) * 1e3
    torch.cuda.synchronize()
    assert torch.equal(y0, y1)
    count = {k: v[0] for k, v in prof.items()}
    for k in ("gemm_qkv", "attention", "gemm_out", "gemm_ffn_up", "gemm_ffn_down"):
        assert count[k] == n_layers, (k, count)
    assert count["layernorm"] == 2 * n_layers
    few_tokens = B * L <= 128
    assert (count["decode"] == 0) if few_tokens else (1 <= count["decode"] <= n_layers)
    total = 0.0
    for k, (n, ms) in prof.items():
        assert (ms > 0.0) == (n > 0), (k, n, ms)
        total += ms
    assert total < wall_ms
    # a second begin/end pair starts from zero
    P.sti_profile_begin()
    assert all(n == 0 for n, _ in P.sti_profile_end().values())


def test_mfma_random_shapes(gpu, oracle_mod):
    """Forty seeded random shapes (1-32 shards of which any number absent, d_model 64-192, 64-256
    FFN neurons per shard, 1-400 keys, up to 3000 tokens, one or two layers; weights at the
    recipe's scale or three or six times larger) through whichever route and tile shapes they
    select.  (Four hundred cases of the same generator, up to 6000 tokens, were run once when
    this test was written: worst error 2.7e-3.)"""
    rng = np.random.default_rng(20240607)
    for case in range(40):
        M = int(rng.choice([1, 2, 3, 4, 7, 12, 16, 29, 32]))
        f = int(rng.choice([64, 128, 256]))
        d = int(rng.choice([64, 128, 192]))
        dims = S.Dims(d, M, 64, f, 1e-12)
        L = int(rng.integers(1, 400))
        B = max(1, min(int(rng.integers(1, max(2, 3000 // L))), 3000 // L))
        n_abs = int(rng.integers(0, M)) if M > 1 else 0
        n_layers = int(rng.choice([1, 2]))
        wl = S.small_workload(9000 + case, dims, n_layers, B, L, n_absent=n_abs, io_dtype="f16")
        S.make_every_term_matter(wl, case, amp=float(rng.choice([1.0, 3.0, 6.0])))
        want = oracle_mod.model_forward(dims, wl.shards, wl.params, wl.x)
        got = run_gpu(gpu, wl, "mfma")
        assert_parity(got, want, TOL["mfma"], (case, d, M, f, B, L, n_abs, n_layers))


def test_concurrent_calls_from_host_threads(gpu):
    """Four host threads, each with a stream and a workspace of its own, run model forwards of
    both routes (and decode calls that upload a shard table) at the same time: every result is
    bit for bit the single-threaded one.  (The library's only shared state is the pinned ring
    that table uploads go through.)"""
    import threading
    torch, P, D = gpu
    prec = P.STI_PREC_F16_MFMA
    prepared = []
    for seed, (B, L) in enumerate([(2, 60), (5, 128), (1, 100), (9, 256)]):
        wl = S.small_workload(8800 + seed, WIDE if seed == 3 else MID, 3, B, L, n_absent=1, io_dtype="f16")
        shards, params, x = D.upload_workload(wl)
        store = P.make_store(D.store_from_plan(shards))
        ws = torch.empty(P.sti_model_workspace_bytes(wl.dims, 3, B, L, prec), dtype=torch.uint8, device="cuda")
        ref = torch.empty_like(x)
        P.sti_model_forward(wl.dims, store, params, wl.plan, x, ref, prec, ws)
        prepared.append((wl, store, params, x, ref, shards))
    n = 4096
    host = [S.make_shard(np.random.default_rng(s), n, int(k))
            for s, k in enumerate(np.random.default_rng(0).choice([2, 3, 4, 5, 6], size=100))]
    dev = [D.upload_shard(s) for s in host]
    dref = torch.empty(len(dev) * n, dtype=torch.float16, device="cuda")
    dws = torch.empty(P.sti_decode_workspace_bytes(len(dev)), dtype=torch.uint8, device="cuda")
    P.sti_decode_shards(dev, n, dref, dws)
    torch.cuda.synchronize()
    bad = []

    def worker(i):
        wl, store, params, x, ref, _ = prepared[i]
        B, L = int(x.shape[0]), int(x.shape[1])
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            ws = torch.empty(P.sti_model_workspace_bytes(wl.dims, 3, B, L, prec), dtype=torch.uint8, device="cuda")
            y = torch.empty_like(x)
            out, ows = torch.empty_like(dref), torch.empty_like(dws)
            for it in range(30):
                y.fill_(float("nan"))
                P.sti_model_forward(wl.dims, store, params, wl.plan, x, y, prec, ws)
                P.sti_decode_shards(dev, n, out, ows)
                if it % 10 == 9:
                    stream.synchronize()
                    if not torch.equal(y, ref) or not torch.equal(out.view(torch.int16), dref.view(torch.int16)):
                        bad.append((i, it))
        stream.synchronize()

    threads = [threading.Thread(target=worker, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad, bad


# ------------------------------------------------------------------ padded sequences

def _key_lengths(L, B, seed):
    """Lengths that hit the edges (1, L, around multiples of 32) and random ones."""
    rng = np.random.default_rng(seed)
    edges = [L, 1, min(L, 32), min(L, 33), max(1, L - 1), min(L, 64), min(L, 31)]
    lens = [edges[b] if b < len(edges) else int(rng.integers(1, L + 1)) for b in range(B)]
    return np.asarray(lens, dtype=np.int32)


def _run_masked(gpu, wl, prec, lens, route):
    torch, P, D = gpu
    precision = P.STI_PREC_F32 if prec == "f32" else P.STI_PREC_F16_MFMA
    shards, params, xd = D.upload_workload(wl)
    ld = None if lens is None else torch.from_numpy(lens).cuda()
    y = torch.full_like(xd, float("nan"))
    B, L = int(xd.shape[0]), int(xd.shape[1])
    store = P.make_store(D.store_from_plan(shards))
    if route == "whole":      # room for every layer's working buffer
        ws = torch.empty(P.sti_model_workspace_bytes(wl.dims, wl.n_layers, B, L, precision), dtype=torch.uint8, device="cuda")
    else:
        ws = torch.empty(P.sti_workspace_bytes(wl.dims, B, L, precision), dtype=torch.uint8, device="cuda")
    if route == "layer":
        assert wl.n_layers == 1
        if ld is None:
            P.sti_layer_forward(wl.dims, shards[0], params[0], xd, y, precision, ws)
        else:
            P.sti_layer_forward_masked(wl.dims, shards[0], params[0], xd, y, ld, precision, ws)
    elif ld is None:
        P.sti_model_forward(wl.dims, store, params, wl.plan, xd, y, precision, ws)
    else:
        P.sti_model_forward_masked(wl.dims, store, params, wl.plan, xd, y, ld, precision, ws)
    torch.cuda.synchronize()
    return y


@pytest.mark.parametrize("prec,dims,B,L,route", [
    ("f32", SMALL, 5, 19, "layer"), ("f32", MID, 8, 70, "model"),
    ("mfma", MID, 3, 40, "layer"),      # two-wave workgroups, scores in registers
    ("mfma", MID, 2, 64, "model"),      # few-token route
    ("mfma", MID, 9, 128, "model"),
    ("mfma", MID, 8, 200, "whole"),     # keys in blocks of 64, every layer's working buffer
    ("mfma", MID, 48, 128, "model"),    # four-wave workgroups
    ("mfma", MID, 64, 128, "model"),    # attention inside the Q/K/V projection; 3 present heads: a tile with one head
    ("mfma", WIDE, 24, 128, "whole"),   # the same with 11 present heads, every layer's working buffer
    ("mfma", MID, 7, 300, "whole"),
    ("mfma", MID, 2, 512, "model"),
])
def test_padded_sequences_match_the_reference(gpu, oracle_mod, prec, dims, B, L, route):
    """Keys beyond a sequence's length take no attention weight (all rows compared, padded ones
    included); full lengths give the bits of the plain entry point; the mask matters at this scale."""
    torch = gpu[0]
    n_layers = 1 if route == "layer" else 2
    wl = S.small_workload(8000 + L, dims, n_layers, B, L, n_absent=1)
    S.make_every_term_matter(wl, 3, amp=6.0 if dims is MID else 3.0)
    lens = _key_lengths(L, B, L)
    want = oracle_mod.model_forward(dims, wl.shards, wl.params, wl.x, key_lengths=lens)
    got = _run_masked(gpu, wl, prec, lens, route)
    assert_parity(got.float().cpu().numpy(), want, TOL[prec])
    plain = _run_masked(gpu, wl, prec, None, route)
    assert rel_err(plain.float().cpu().numpy(), want) > 3 * TOL[prec]
    full = _run_masked(gpu, wl, prec, np.full(B, L, dtype=np.int32), route)
    assert torch.equal(full, plain)


@pytest.mark.parametrize("L", [129, 160, 161, 192, 224, 255])
def test_attention_over_any_part_of_a_key_block(gpu, oracle_mod, L):
    """Keys in blocks of 64: sequences whose last block holds 1, 31, 32, 33, 63 and 64 keys, or is the first."""
    wl = S.small_workload(8700 + L, MID, 1, 12, L)
    S.make_every_term_matter(wl, 5)
    lens = np.array([L, 128, 127, 97, 96, 95, 65, 64, 63, 33, 32, 1], dtype=np.int32)
    want = oracle_mod.model_forward(MID, wl.shards, wl.params, wl.x, key_lengths=lens)
    assert_parity(_run_masked(gpu, wl, "mfma", lens, "layer").float().cpu().numpy(), want, TOL["mfma"])


@pytest.mark.parametrize("dims,n_absent", [(MID, 1), (MID, 0), (WIDE, 3)])
def test_attention_inside_the_projection_matches_the_separate_kernels(gpu, oracle_mod, dims, n_absent):
    """With sequences of 128 tokens and enough of them, the Q/K/V projection's workgroups run the
    attention of the two heads they hold.  Against the reference on every sequence (odd and even
    numbers of present heads), and against the same sequences sent as four smaller batches, which take
    the separate projection and attention kernels: the two compute the same values in the same order up
    to the tile shapes that the batch size selects for the other projections."""
    torch, P, D = gpu
    B = 256 // ((dims.n_heads - n_absent + 1) // 2)
    wl = S.small_workload(9100 + n_absent, dims, 2, B, 128, n_absent=n_absent, io_dtype="f16")
    S.make_every_term_matter(wl, 12, amp=3.0)
    want = oracle_mod.model_forward(dims, wl.shards, wl.params, wl.x)
    got = run_gpu(gpu, wl, "mfma")
    assert_parity(got, want, TOL["mfma"])
    for b in (0, B // 2, B - 1):
        assert_parity(got[b], want[b], TOL["mfma"], b)
    q = B // 4
    for part in range(4):
        sub = run_gpu(gpu, wl, "mfma", x=wl.x[part * q:(part + 1) * q])
        assert_parity(sub, got[part * q:(part + 1) * q], 4e-3, part)


def test_padded_sequences_ignore_what_the_padding_holds(gpu):
    """Real rows come out bit for bit the same whatever finite values the padded rows of x hold, and
    lengths outside 1..seq are clamped."""
    torch, P, D = gpu
    B, L = 6, 96
    wl = S.small_workload(8100, MID, 2, B, L, n_absent=1, io_dtype="f16")
    S.make_every_term_matter(wl, 4)
    lens = _key_lengths(L, B, 1)
    a = _run_masked(gpu, wl, "mfma", lens, "model")
    rng = np.random.default_rng(2)
    for b, n in enumerate(lens):
        wl.x[b, n:] = rng.normal(0, 30, wl.x[b, n:].shape).astype(wl.x.dtype)
    bb = _run_masked(gpu, wl, "mfma", lens, "model")
    for b, n in enumerate(lens):
        assert torch.equal(a[b, :n], bb[b, :n]), b
    wild = lens.copy()
    wild[0], wild[1] = L + 1000, -5            # clamped to L and to 1
    assert lens[0] == L and lens[1] == 1
    assert torch.equal(_run_masked(gpu, wl, "mfma", wild, "model"), bb)


@pytest.mark.parametrize("prec,dims,B,L,route", [
    ("mfma", MID, 1, 95, "model"), ("mfma", MID, 3, 64, "model"),     # few tokens: values in tiles, one and several sequences
    ("mfma", MID, 6, 32, "layer"), ("mfma", MID, 2, 96, "model"),
    ("mfma", MID, 3, 50, "model"),                                    # few tokens, sequences that straddle row blocks
    ("mfma", MID, 7, 93, "model"), ("mfma", MID, 4, 200, "whole"),    # keys staged in LDS: all of them, block by block
    ("mfma", MID, 64, 128, "model"),                                  # attention inside the Q/K/V projection
    ("f32", MID, 3, 70, "model"),
    ("f32", S.Dims(768, 12, 64, 256, 1e-12), 4, 119, "model"),        # bfloat16 matrix cores; rows of a tile behind the last token
])
def test_no_value_in_the_padding_reaches_a_real_row(gpu, prec, dims, B, L, route):
    """Real rows have the bits they have over zero padding when the padding holds values beyond binary16's range,
    infinities or NaN: a masked key has weight zero, and nothing multiplies that by its value."""
    torch, P, D = gpu
    lens = _key_lengths(L, B, 1)
    if B == 1:
        lens[0] = L - 20
    for io, fills in (("f32", (1e6, float("inf"), float("nan"))), ("f16", (6e4, float("-inf")))):
        wl = S.small_workload(8150 + L, dims, 1 if route == "layer" else 2, B, L, n_absent=1, io_dtype=io)
        S.make_every_term_matter(wl, 4)
        outs = []
        for fill in (0.0,) + fills:
            for b, n in enumerate(lens):
                wl.x[b, n:] = fill
            outs.append(_run_masked(gpu, wl, prec, lens, route))
        for fill, y in zip(fills, outs[1:]):
            for b, n in enumerate(lens):
                assert torch.equal(y[b, :n], outs[0][b, :n]), (io, fill, b, int(n))


@pytest.mark.parametrize("prec,dims,B,L", [
    ("f32", SMALL, 2, 150), ("f32", MID, 1, 130),
    ("mfma", MID, 1, 95), ("mfma", MID, 1, 160), ("mfma", MID, 2, 128),   # few tokens: a wave's blocks of 32 keys
    ("mfma", MID, 3, 50), ("mfma", MID, 3, 200), ("mfma", WIDE, 9, 130),  # all scores at once; blocks of 64 keys
])
def test_keys_with_scores_of_minus_infinity_have_weight_zero(gpu, oracle_mod, prec, dims, B, L):
    """The first keys' scores overflow to -infinity (K in binary16, the product in float32), whole key blocks of
    them, and the others are finite: the softmax is that of the finite ones, as over all scores at once."""
    d, dh = dims.d_model, dims.d_head
    n_overflow = min(96, L - 10)
    wl = S.small_workload(8400 + L, dims, 1, B, L, bit_choices=(32,), io_dtype="f32")
    for s in wl.shards[0]:
        rows = s.data.reshape(-1)
        rows[:d] = 0.0                        # Q feature 0: its bias
        rows[dh * d:(dh + 1) * d] = 0.0       # K feature 0: -2000 or -1e30 times x feature 0
        rows[dh * d] = -2000.0 if prec == "mfma" else -1e30
    wl.params[0].bq.reshape(-1, dh)[:, 0] = 1.0 if prec == "mfma" else 1e10
    wl.params[0].bk.reshape(-1, dh)[:, 0] = 0.0
    wl.x[:, :, 0] = 0.0
    wl.x[:, :n_overflow, 0] = 60.0
    with np.errstate(over="ignore"):
        want = oracle_mod.model_forward(dims, wl.shards, wl.params, wl.x)
    assert np.all(np.isfinite(want))
    assert_parity(run_gpu(gpu, wl, prec), want, TOL[prec])


def test_captured_masked_forward_follows_the_lengths_in_device_memory(gpu):
    """The key lengths are read by the kernels, not by the host: a graph captured once serves
    other lengths by rewriting the device array between replays."""
    torch, P, D = gpu
    B, L = 3, 60
    wl = S.small_workload(889, MID, 2, B, L, n_absent=1, io_dtype="f16")
    S.make_every_term_matter(wl, 6)
    prec = P.STI_PREC_F16_MFMA
    shards, params, x = D.upload_workload(wl)
    store = P.make_store(D.store_from_plan(shards))
    ws = torch.empty(P.sti_workspace_bytes(MID, B, L, prec), dtype=torch.uint8, device="cuda")
    lens = torch.tensor([L, 7, 33], dtype=torch.int32, device="cuda")
    y_graph = torch.full_like(x, float("nan"))
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            P.sti_model_forward_masked(MID, store, params, wl.plan, x, y_graph, lens, prec, ws)
    torch.cuda.synchronize()
    seen = []
    for new in ([L, 7, 33], [1, L, 32], [59, 31, 2], [L, 7, 33]):
        lens.copy_(torch.tensor(new, dtype=torch.int32))
        y_graph.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        eager = torch.full_like(x, float("nan"))
        P.sti_model_forward_masked(MID, store, params, wl.plan, x, eager, lens, prec, ws)
        torch.cuda.synchronize()
        assert torch.equal(y_graph, eager), new
        seen.append(eager.clone())
    assert not torch.equal(seen[0], seen[1]) and torch.equal(seen[0], seen[3])


def test_padded_sequences_at_configuration_4_size(gpu, oracle_mod):
    """32 x 128 tokens of BERT-base (three layers, whole-model route, the launch shapes the
    benchmark times) with a length mix from 1 to 128: sampled sequences against the reference,
    each run alone at its padded length."""
    wl = S.config4(n_layers=3)
    S.make_every_term_matter(wl, 4, amp=3.0)
    rng = np.random.default_rng(12)
    lens = rng.integers(1, wl.seq + 1, wl.x.shape[0]).astype(np.int32)
    lens[0], lens[31], lens[7] = wl.seq, 1, 65
    got = _run_masked(gpu, wl, "mfma", lens, "whole").float().cpu().numpy()
    assert np.all(np.isfinite(got))
    for b in (0, 7, 19, 31):
        want = oracle_mod.model_forward(wl.dims, wl.shards, wl.params, wl.x[b:b + 1], key_lengths=lens[b:b + 1])
        assert_parity(got[b:b + 1], want, TOL["mfma"], (b, int(lens[b])))
