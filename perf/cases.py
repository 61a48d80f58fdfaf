"""Workloads of the shard-decode + encoder-layer library, as its users run it.

Five families, one per thing the library is asked to do:

``model``     layers of shards over a batch of sequences (one layer: ``sti_layer_forward``; several:
              ``sti_model_forward``; padded batches: the ``*_masked`` entry points), in both precisions
``decode``    shards decompressed by themselves (``sti_decode_shards``)
``quantize``  a layer's float32 shards turned into a k-bit version (``sti_quantize_layer``)
``pipeline``  a model whose packed shards stay in pinned host memory (``StiPipeline``)

A case is a dict of plain values.  Shards and activations are drawn on the GPU from the seed: index
streams are uniform (the quantizer cuts clusters of equal population), centroids sit at Gaussian quantiles,
weights have the spread of a trained encoder (0.04), biases and LayerNorm parameters are large enough for
every term of a layer to show in its output.
"""
from __future__ import annotations

import math
import random
from statistics import NormalDist
from types import SimpleNamespace

import numpy as np
import torch

import paper_2207_05022_amd as sti

DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
PARAM_NAMES = ("bq", "bk", "bv", "bo", "b1", "b2", "ln1_g", "ln1_b", "ln2_g", "ln2_b")
SIGMA = 0.04
ALIGN = 256

BERT_BASE = {"d_model": 768, "heads": 12, "d_head": 64, "ffn": 256}
BERT_LARGE = {"d_model": 1024, "heads": 16, "d_head": 64, "ffn": 256}


def model(name, dims, layers, batch, seq, bits, **more):
    case = {"name": name, "kind": "model", **dims, "layers": layers, "batch": batch, "seq": seq, "bits": bits,
            "absent": 0, "io": "f32", "precision": "f16", "padded": False, "outliers": False}
    case.update(more)
    return case


def listed():
    return [
        # one short query through one layer: the smallest call, all launches and host path
        model("layer_short_query", BERT_BASE, 1, 1, 23, "4"),
        # one layer at the padded length the paper profiles with, 4-bit shards
        model("layer_128_4bit", BERT_BASE, 1, 1, 128, "4"),
        # single-input inference of a mixed-fidelity submodel, a quarter of the shards left out
        model("base_single_128", BERT_BASE, 12, 1, 128, "2,3,4,5,6,32", absent=3),
        # the same for the larger shape and a longer input
        model("large_single_256", BERT_LARGE, 24, 1, 256, "2,3,4,5,6", absent=4),
        # a small ragged serving batch, padded to its longest sequence; shards with outlier dictionaries
        model("base_padded_batch", BERT_BASE, 12, 11, 93, "2,3,4,6", absent=2, io="bf16", padded=True, outliers=True),
        # batched serving at the padded length
        model("base_batch_32x128", BERT_BASE, 12, 32, 128, "2,3,4,6,32", io="f16"),
        # bulk scoring of long documents: the largest forward
        model("large_batch_24x384", BERT_LARGE, 24, 24, 384, "2,3,4,5,6", io="f16"),
        # the paper's own float32 arithmetic, for results to be compared against
        model("base_float32_8x128", BERT_BASE, 12, 8, 128, "2,3,4,5,6,32", precision="f32"),
        # one gigabyte of packed shards to binary16: a whole store decompressed
        {"name": "decode_1GiB_f16", "kind": "decode", "shards": 4221, "weights": 589824, "bits": "2,3,4,5,6", "out": "f16",
         "outliers": False},
        # one layer's shards with outlier dictionaries to float32, for a caller that computes by itself
        {"name": "decode_layer_f32", "kind": "decode", "shards": 12, "weights": 589824, "bits": "2,3,4,5,6,32", "out": "f32",
         "outliers": True},
        # preprocessing of a model, one layer and one bitwidth per call
        {"name": "quantize_layer_4bit", "kind": "quantize", **BERT_BASE, "bits": 4},
        # single-input inference with the shards in host memory and a preload buffer of a few layers
        {"name": "pipeline_base_128", "kind": "pipeline", **BERT_BASE, "layers": 12, "batch": 1, "seq": 128,
         "bits": "2,3,4,5,6,32", "absent": 3, "preload_mib": 16, "slots": 4},
    ]


# ---------------------------------------------------------------------------
# More cases of the same ranges
# ---------------------------------------------------------------------------

def log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw_dims(rng):
    """Encoder shapes between a distilled model and the larger BERT shape."""
    d_model = 64 * rng.randint(4, 16)
    heads = rng.randint(max(2, d_model // 128), d_model // 64)
    return {"d_model": d_model, "heads": heads, "d_head": 64, "ffn": rng.choice((64, 128, 192, 256))}


def draw_forward(rng):
    dims = rng.choice((BERT_BASE, BERT_BASE, BERT_LARGE, draw_dims(rng)))
    largest = 24 * 24 * 384 * shard_weights(BERT_LARGE) * BERT_LARGE["heads"]
    seq = log_int(rng, 8, 512)
    batch = log_int(rng, 1, 96)
    layers = rng.choice((1, 2, 4, 6, 12, 12, 24))
    while layers * batch * seq * shard_weights(dims) * dims["heads"] > largest or batch * seq > 24 * 384:
        batch = (batch + 1) // 2
    return {"kind": "model", **dims, "layers": layers, "batch": batch, "seq": seq,
            "bits": rng.choice(("4", "2,3,4,5,6", "2,3,4,6,32", "2,3,4,5,6,32", "6")),
            "absent": rng.choice((0, 0, dims["heads"] // 4, dims["heads"] // 2)), "io": rng.choice(("f32", "f16", "bf16")),
            "precision": "f16", "padded": rng.random() < 0.35, "outliers": rng.random() < 0.25}


def draw_float32(rng):
    """The float32 path takes any dimensions."""
    if rng.random() < 0.5:
        dims = BERT_BASE
    else:
        dims = {"d_model": rng.randint(96, 768), "heads": rng.randint(2, 12), "d_head": rng.randint(16, 80),
                "ffn": rng.randint(48, 256)}
    largest = 12 * 8 * 128 * shard_weights(BERT_BASE) * BERT_BASE["heads"]
    seq, batch, layers = log_int(rng, 8, 384), log_int(rng, 1, 32), rng.choice((1, 2, 4, 12))
    while layers * batch * seq * shard_weights(dims) * dims["heads"] > largest or batch * seq > 2048:
        batch, seq = (batch + 1) // 2, (seq if batch > 1 else (seq + 1) // 2)
    return {"kind": "model", **dims, "layers": layers, "batch": batch, "seq": seq, "bits": "2,3,4,5,6,32",
            "absent": rng.choice((0, dims["heads"] // 4)), "io": "f32", "precision": "f32", "padded": rng.random() < 0.35,
            "outliers": False}


def draw_decode(rng):
    weights = log_int(rng, 10_000, 1_200_000)
    if rng.random() < 0.6:
        weights = weights // 1024 * 1024 + 1024     # shards of real models; the others have ragged ends
    most = 4221 * 589824 // weights
    out = rng.choice(("f32", "f16", "f16", "bf16"))
    return {"kind": "decode", "shards": log_int(rng, 1, min(4096, most // (2 if out == "f32" else 1))), "weights": weights,
            "bits": rng.choice(("2", "3", "4", "5", "6", "2,3,4,5,6", "2,3,4,5,6,32")), "out": out,
            "outliers": rng.random() < 0.4}


def draw_quantize(rng):
    return {"kind": "quantize", **draw_dims(rng), "bits": rng.randint(2, 6)}


def draw_pipeline(rng):
    dims = rng.choice((BERT_BASE, draw_dims(rng)))
    return {"kind": "pipeline", **dims, "layers": rng.choice((2, 4, 6, 12)), "batch": log_int(rng, 1, 8),
            "seq": log_int(rng, 16, 256), "bits": rng.choice(("4", "2,3,4,5,6", "2,3,4,5,6,32")),
            "absent": rng.choice((0, dims["heads"] // 4)), "preload_mib": rng.choice((0, 4, 16, 64)), "slots": rng.choice((2, 4, 8))}


def draw(rng: random.Random):
    family = rng.choices((draw_forward, draw_float32, draw_decode, draw_quantize, draw_pipeline), (9, 2, 4, 3, 2))[0]
    return family(rng)


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def shard_weights(c):
    return c["d_model"] * (4 * c["d_head"] + 2 * c["ffn"])


def plan_counts(c):
    """Bitwidth -> number of shards: which shard gets which is drawn, how many is not."""
    bits = [int(b) for b in c["bits"].split(",")]
    slots = c["layers"] * (c["heads"] - c["absent"]) if "layers" in c else c["shards"]
    return {b: slots // len(bits) + (i < slots % len(bits)) for i, b in enumerate(bits)}


def draw_plan(c, gen):
    """[layers][heads] of bitwidth or 0: the same number of absent shards in every layer."""
    flat = np.concatenate([np.full(n, b, dtype=np.int8) for b, n in plan_counts(c).items()])
    gen.shuffle(flat)
    plan = np.zeros((c["layers"], c["heads"]), dtype=np.int8)
    present = c["heads"] - c["absent"]
    for l in range(c["layers"]):
        plan[l, np.sort(gen.permutation(c["heads"])[:present])] = flat[l * present:(l + 1) * present]
    return plan


def stream_bytes(bits, weights):
    return weights * 4 if bits == 32 else (weights * bits + 7) // 8


def outliers_per_shard(c):
    """The paper reports 0.14 - 0.17 % of the weights."""
    weights = c["weights"] if c["kind"] == "decode" else shard_weights(c)
    return max(1, weights * 3 // 2000) if c["outliers"] else 0


def draw_shards(bitwidths, weights, n_outliers, gen, host=False):
    """Shard objects of the given bitwidths with their streams in one device (or pinned host) pool."""
    n = len(bitwidths)
    sizes = [stream_bytes(b, weights) for b in bitwidths]
    offsets, total = [], 0
    for s in sizes:
        offsets.append(total)
        total += -(-s // ALIGN) * ALIGN
    pool = torch.randint(0, 256, (total,), dtype=torch.uint8, device="cuda", generator=gen)
    for b, at in zip(bitwidths, offsets):
        if b == 32:
            pool[at:at + 4 * weights].view(torch.float32).normal_(0.0, SIGMA, generator=gen)
        elif weights * b % 8:
            pool[at + (weights * b + 7) // 8 - 1] &= 0xFF >> (8 - weights * b % 8)
    if host:
        pinned = torch.empty(total, dtype=torch.uint8, pin_memory=True)
        pinned.copy_(pool)
        pool = pinned
    quantiles = torch.zeros(7, 64, device="cuda")
    for b in set(bitwidths) - {32}:
        q = [NormalDist().inv_cdf((j + 0.5) / (1 << b)) for j in range(1 << b)]
        quantiles[b, :1 << b] = torch.tensor(q, device="cuda")
    rows = torch.tensor([0 if b == 32 else b for b in bitwidths], device="cuda")
    scale = SIGMA * (0.8 + 0.4 * torch.rand(n, 1, device="cuda", generator=gen))
    books = quantiles[rows] * scale
    if n_outliers:
        step = weights // n_outliers     # one in each stretch: distinct, ascending, spread over the shard
        at = torch.arange(n_outliers, device="cuda") * step
        pos = (at + torch.randint(0, step, (n, n_outliers), device="cuda", generator=gen)).to(torch.int32)
        val = (3.0 + 3.0 * torch.rand(n, n_outliers, device="cuda", generator=gen)) * SIGMA
        val *= torch.randint(0, 2, (n, n_outliers), device="cuda", generator=gen) * 2 - 1
    shards = []
    for i, (b, at) in enumerate(zip(bitwidths, offsets)):
        listed_out = n_outliers and b != 32
        shards.append(SimpleNamespace(bitwidth=b, data=pool[at:at + sizes[i]], codebook=books[i] if b != 32 else None,
                                      outlier_pos=pos[i] if listed_out else None, outlier_val=val[i] if listed_out else None))
    return shards


def draw_params(c, gen):
    d, M, dh, f = c["d_model"], c["heads"], c["d_head"], c["ffn"]
    sizes = {"bq": M * dh, "bk": M * dh, "bv": M * dh, "b1": M * f}
    params = []
    for _ in range(c["layers"]):
        p = SimpleNamespace(**{n: torch.randn(sizes.get(n, d), device="cuda", generator=gen) * 0.1 for n in PARAM_NAMES})
        p.ln1_g += 1.0
        p.ln2_g += 1.0
        params.append(p)
    return params


def prepare_forward(c, seed, gen):
    host = c["kind"] == "pipeline"
    s = SimpleNamespace(kind=c["kind"])
    s.dims = sti.StiDims(c["d_model"], c["heads"], c["d_head"], c["ffn"], 1e-12)
    s.plan = draw_plan(c, np.random.default_rng(seed))
    n_outliers = 0 if host else outliers_per_shard(c)
    shards = iter(draw_shards([int(b) for b in s.plan.ravel() if b], shard_weights(c), n_outliers, gen, host))
    rows = [[next(shards) if b else None for b in row] for row in s.plan]
    s.params = draw_params(c, gen)
    s.x = torch.randn(c["batch"], c["seq"], c["d_model"], device="cuda", generator=gen).to(DTYPES[c.get("io", "f32")])
    s.y = torch.empty_like(s.x)
    s.precision = sti.STI_PREC_F32 if c.get("precision") == "f32" else sti.STI_PREC_F16_MFMA
    s.key_lengths = None
    if c.get("padded"):
        lengths = torch.randint(max(1, c["seq"] // 4), c["seq"] + 1, (c["batch"],), device="cuda", generator=gen)
        lengths[0] = c["seq"]
        s.key_lengths = lengths.to(torch.int32)
    s.keep = rows
    if not host and c["layers"] == 1:
        s.kind = "layer"
        s.shards = sti.shard_array(rows[0])
        size = sti.sti_workspace_bytes(s.dims, c["batch"], c["seq"], s.precision)
    else:
        s.store = sti.make_store([[{r.bitwidth: r} if r is not None else {} for r in row] for row in rows])
        size = (sti.sti_workspace_bytes(s.dims, c["batch"], c["seq"], s.precision) if host else
                sti.sti_model_workspace_bytes(s.dims, c["layers"], c["batch"], c["seq"], s.precision))
    s.workspace = torch.empty(size, dtype=torch.uint8, device="cuda")
    if host:
        slot = sti.sti_pipeline_staging_bytes(s.dims) // 2
        staging = torch.empty(c["slots"] * slot, dtype=torch.uint8, device="cuda")
        preload = torch.empty(c["preload_mib"] << 20, dtype=torch.uint8, device="cuda") if c["preload_mib"] else None
        s.pipeline = sti.StiPipeline(s.dims, preload, staging)
    return s


def prepare_decode(c, seed, gen):
    s = SimpleNamespace(kind="decode", weights=c["weights"])
    bitwidths = np.concatenate([np.full(n, b) for b, n in plan_counts(c).items()])
    np.random.default_rng(seed).shuffle(bitwidths)
    s.keep = draw_shards([int(b) for b in bitwidths], c["weights"], outliers_per_shard(c), gen)
    s.shards = sti.shard_array(s.keep)
    s.out = torch.empty(c["shards"] * c["weights"], dtype=DTYPES[c["out"]], device="cuda")
    s.workspace = torch.empty(max(16, sti.sti_decode_workspace_bytes(c["shards"])), dtype=torch.uint8, device="cuda")
    return s


def quantize_room(c):
    """Entries of a shard's outlier dictionary: several times what a Gaussian with a light tail has."""
    return max(64, shard_weights(c) // 100)


def prepare_quantize(c, seed, gen):
    s = SimpleNamespace(kind="quantize", bits=c["bits"])
    s.dims = sti.StiDims(c["d_model"], c["heads"], c["d_head"], c["ffn"], 1e-12)
    M, n = c["heads"], shard_weights(c)
    s.weights = torch.randn(M, n, device="cuda", generator=gen) * SIGMA
    tail = torch.rand(M, n, device="cuda", generator=gen) < 0.0015
    s.weights = torch.where(tail, s.weights.sign() * SIGMA * (3.5 + 2.5 * torch.rand(M, n, device="cuda", generator=gen)), s.weights)
    s.packed = torch.empty(M, n * c["bits"] // 8, dtype=torch.uint8, device="cuda")
    s.codebook = torch.empty(1 << c["bits"], device="cuda")
    s.pos = torch.zeros(M, quantize_room(c), dtype=torch.int32, device="cuda")   # (entries past a count stay as they are)
    s.val = torch.zeros(M, quantize_room(c), device="cuda")
    s.count = torch.empty(M, dtype=torch.int32, device="cuda")
    s.stats = torch.zeros(32, dtype=torch.uint8, device="cuda")
    s.workspace = torch.empty(sti.sti_quantize_workspace_bytes(s.dims), dtype=torch.uint8, device="cuda")
    s.result = {"packed": s.packed, "codebook": s.codebook, "outlier_pos": s.pos, "outlier_val": s.val,
                "outlier_count": s.count, "mean_variance": s.stats[:16].view(torch.float64),
                "n_outliers": s.stats[16:24].view(torch.int64), "status": s.stats[24:28].view(torch.int32)}
    return s


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    if case["kind"] == "decode":
        return prepare_decode(case, seed, gen)
    if case["kind"] == "quantize":
        return prepare_quantize(case, seed, gen)
    return prepare_forward(case, seed, gen)


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def run(s):
    if s.kind == "decode":
        sti.sti_decode_shards(s.shards, s.weights, s.out, s.workspace)
        return s.out
    if s.kind == "quantize":
        sti.sti_quantize_layer(s.dims, s.weights, s.bits, s.packed, s.codebook, s.pos, s.val, s.count, s.stats, s.workspace)
        return s.result
    if s.kind == "pipeline":
        s.pipeline.forward(s.store, s.params, s.plan, s.x, s.y, s.precision, s.workspace)
    elif s.kind == "layer" and s.key_lengths is not None:
        sti.sti_layer_forward_masked(s.dims, s.shards, s.params[0], s.x, s.y, s.key_lengths, s.precision, s.workspace)
    elif s.kind == "layer":
        sti.sti_layer_forward(s.dims, s.shards, s.params[0], s.x, s.y, s.precision, s.workspace)
    elif s.key_lengths is not None:
        sti.sti_model_forward_masked(s.dims, s.store, s.params, s.plan, s.x, s.y, s.key_lengths, s.precision, s.workspace)
    else:
        sti.sti_model_forward(s.dims, s.store, s.params, s.plan, s.x, s.y, s.precision, s.workspace)
    return s.y


# ---------------------------------------------------------------------------
# What a pass cannot do without, and how closely two correct passes agree
# ---------------------------------------------------------------------------

def work(c):
    if c["kind"] == "quantize":
        n = shard_weights(c) * c["heads"]
        return {"bytes": 4 * n + n * c["bits"] / 8 + 8 * 0.0016 * n, "flops": 0}
    weights = c["weights"] if c["kind"] == "decode" else shard_weights(c)
    n_outliers = 0 if c["kind"] == "pipeline" else outliers_per_shard(c)
    bytes_ = 0
    for b, n in plan_counts(c).items():
        bytes_ += n * (stream_bytes(b, weights) + (0 if b == 32 else 4 * (1 << b) + 8 * n_outliers))
    if c["kind"] == "decode":
        return {"bytes": bytes_ + c["shards"] * weights * (4 if c["out"] == "f32" else 2), "flops": 0}
    tokens, present = c["batch"] * c["seq"], c["heads"] - c["absent"]
    io = 4 if c.get("io", "f32") == "f32" else 2
    bytes_ += 2 * tokens * c["d_model"] * io
    bytes_ += c["layers"] * 4 * (present * (3 * c["d_head"] + c["ffn"]) + 6 * c["d_model"])
    keys = c["seq"] * (0.625 if c.get("padded") else 1.0)   # mean key length of a padded batch
    flops = c["layers"] * tokens * present * (2 * weights + 4 * keys * c["d_head"])
    return {"bytes": bytes_, "flops": flops}


def tolerance(c):
    if c["kind"] == "decode":
        return "exact"
    if c["kind"] == "quantize":
        return {"rel": 1e-6, "max": 1e-6, "differ": 0.0}   # float64 sums, rounded once; indexes and dictionaries are whole values
    if c.get("precision") == "f32":
        return {"rel": 1e-5}
    return {"rel": 5e-3}   # binary16 operands and activations over up to 24 layers
