"""What is timed of this library, through its public entry points, and over which ranges.

Layers are Gaussian matrices pruned by magnitude and weight-shared (k values, by equal bins or by
1-D k-means), as in the paper's experiments; batches are ReLU(N(0,1)).  A case is one of

  dot      Y = X.W on a HAC, sHAC or Rice-coded sHAC blob (inference with one compressed layer)
  im       Y = X.W on an index map (a quantized, unpruned convolutional layer as its im2col product)
  forward  a fully connected block, layer after layer, on a network blob with one shared dictionary
  encode   a layer that was pruned and quantized on the GPU, encoded there
  encode_host  the same from a numpy matrix, as a program that prepares a model does it

Shapes and sparsities are those of the workloads of this repository (VGG16 / VGG19 fully connected
layers, a 3x3x512 convolution, the tiny layer of the examples) and what lies between them.
"""
from __future__ import annotations

import math
import statistics

import numpy as np
import torch

import paper_2108_12704_amd as hac

DEV = "cuda:0"
FORMATS = {"hac": hac.HAC_FORMAT_HAC, "shac": hac.HAC_FORMAT_SHAC, "rice": hac.HAC_FORMAT_SHAC}
# the work of the largest product listed (12544 patches of a 4608 x 512 convolution layer)
MOST_MACS = 12544 * 4608 * 512

# (n, m) per layer, fraction pruned per layer
BLOCKS = {
    "tiny-fc": (((500, 300), (300, 120), (120, 10)), (0.7, 0.7, 0.5)),
    "vgg19-fc": (((512, 4096), (4096, 4096), (4096, 10)), (0.9, 0.96, 0.8)),
}


def dot(name, fmt, n, m, prune, k, quant, batch, buffers):
    return {"name": name, "kind": "dot", "format": fmt, "n": n, "m": m, "prune": prune, "k": k, "quant": quant,
            "batch": batch, "buffers": buffers}


def listed():
    return [
        # the smallest call: a layer of a small network and a handful of inputs (launch and host time)
        dot("tiny-hac-b8", "hac", 500, 300, 0.70, 16, "uniform", 8, "none"),
        # the last classifier layer of VGG16 at an ordinary batch
        dot("fc3-shac-b64", "shac", 4096, 1000, 0.90, 32, "kmeans", 64, "none"),
        # a hidden layer with many shared values (long codewords)
        dot("hidden-hac-b128", "hac", 4096, 4096, 0.96, 256, "kmeans", 128, "none"),
        # VGG16's first fully connected layer: one input at a time in a serving loop that allocates nothing
        dot("fc1-hac-b1", "hac", 25088, 4096, 0.98, 32, "uniform", 1, "inside"),
        # ... a small batch in a program that keeps its output and workspace
        dot("fc1-shac-b32", "shac", 25088, 4096, 0.98, 32, "uniform", 32, "kept"),
        # ... and a large one
        dot("fc1-hac-b256", "hac", 25088, 4096, 0.98, 32, "uniform", 256, "none"),
        # nothing a power of two or a multiple of anything: odd sizes and batch, row gaps coded in the stream
        dot("odd-rice-b37", "rice", 9973, 1511, 0.93, 50, "kmeans", 37, "none"),
        # a convolution as its im2col product (a batch of 64 maps of 14 x 14), two fifths of the weights left
        dot("conv-hac-b12544", "hac", 4608, 512, 0.60, 256, "kmeans", 12544, "kept"),
        # the same layer quantized but not pruned, as an index map, on four maps
        {"name": "conv-im-b784", "kind": "im", "n": 4608, "m": 512, "k": 64, "quant": "kmeans", "batch": 784},
        # the fully connected block whose matrices the paper times, as one call on a network blob
        {"name": "vgg19-fc-b32", "kind": "forward", "block": "vgg19-fc", "k": 32, "quant": "uniform", "batch": 32},
        # encoding on the GPU: the largest layer
        {"name": "encode-shac-fc1", "kind": "encode", "format": "shac", "n": 25088, "m": 4096, "prune": 0.98, "k": 32, "quant": "uniform"},
        # encoding from host memory: the hidden layer
        {"name": "encode-host-hac-hidden", "kind": "encode_host", "format": "hac", "n": 4096, "m": 4096, "prune": 0.96, "k": 256, "quant": "kmeans"},
    ]


def log_int(rng, lo, hi):
    return min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def draw(rng):
    kind = rng.choice(("dot", "dot", "dot", "dot", "im", "forward", "encode", "encode_host"))
    k, quant = log_int(rng, 16, 256), rng.choice(("uniform", "kmeans"))
    if kind == "forward":
        return {"kind": kind, "block": rng.choice(sorted(BLOCKS)), "k": k, "quant": quant, "batch": log_int(rng, 1, 256)}
    n, m = log_int(rng, 500, 25088), log_int(rng, 10, 4096)
    if kind == "im":
        n, m = log_int(rng, 64, 4608), log_int(rng, 10, 4096)
        return {"kind": kind, "n": n, "m": m, "k": k, "quant": quant, "batch": log_int(rng, 1, min(12544, MOST_MACS // (n * m)))}
    prune = round(rng.uniform(0.60, 0.99), 3)
    fmt = rng.choice(sorted(FORMATS))
    if kind == "encode_host":
        n = min(n, 4096)
    if kind != "dot":
        return {"kind": kind, "format": fmt, "n": n, "m": m, "prune": prune, "k": k, "quant": quant}
    return {"kind": kind, "format": fmt, "n": n, "m": m, "prune": prune, "k": k, "quant": quant,
            "batch": log_int(rng, 1, 512), "buffers": rng.choice(("none", "kept"))}


# ---- inputs -------------------------------------------------------------------------------------


def kmeans_values(sample, k):
    """1-D k-means centroids of a sample of the surviving weights (float32, ascending)."""
    v = np.sort(sample.astype(np.float64))
    cent = np.quantile(v, (np.arange(k) + 0.5) / k)
    csum = np.concatenate(([0.0], np.cumsum(v)))
    for _ in range(30):
        edges = np.concatenate(([0], np.searchsorted(v, 0.5 * (cent[:-1] + cent[1:]), side="right"), [v.size]))
        cnt = np.diff(edges)
        cent = np.where(cnt > 0, (csum[edges[1:]] - csum[edges[:-1]]) / np.maximum(cnt, 1), cent)
    return np.unique(cent.astype(np.float32))


def make_weights(shapes, prunes, k, quant, seed):
    """Pruned layers on the GPU whose survivors share one set of k values."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    raw, keeps = [], []
    for (n, m), prune in zip(shapes, prunes):
        w = torch.randn((n, m), generator=g, device=DEV) * 0.02
        raw.append(w)
        keeps.append(w.abs() > 0.02 * statistics.NormalDist().inv_cdf((1 + prune) / 2) if prune > 0 else torch.ones_like(w, dtype=torch.bool))
    kept = [w[s] for w, s in zip(raw, keeps)]
    if quant == "uniform":
        lo, hi = min(float(v.min()) for v in kept), max(float(v.max()) for v in kept)
        step = (hi - lo) / k
        values = (lo + (np.arange(k) + 0.5) * step).astype(np.float32)
        index = [torch.clamp(torch.floor((v.double() - lo) / step), 0, k - 1).long() for v in kept]
    else:
        values = kmeans_values(torch.cat([v[:: max(1, v.numel() // 65536)] for v in kept]).cpu().numpy(), k)
        bounds = torch.from_numpy(0.5 * (values[:-1].astype(np.float64) + values[1:])).to(DEV)
        index = [torch.bucketize(v.double(), bounds) for v in kept]
    values = np.where(values == 0.0, np.float32(1e-6), values).astype(np.float32)        # 0.0 stays the pruned entry
    table = torch.from_numpy(values).to(DEV)
    out = []
    for w, s, i in zip(raw, keeps, index):
        full = torch.zeros_like(w)
        full[s] = table[i]
        out.append(full)
    return out


def make_batch(rows, n, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed + 1)
    return torch.randn((rows, n), generator=g, device=DEV).clamp_min_(0.0)


def coding(fmt):
    return hac.RI_RICE if fmt == "rice" else hac.RI_FIELDS


def arena_bytes(case):
    """Room a program sets aside for one encoded layer: its blob (whose size depends on the weights),
    with the index and tables beside the stream."""
    size = blob_bytes(case["format"], case["n"], case["m"], case["prune"], case["k"], case["quant"])
    return int(1.5 * size) + 300 * case["m"] + 65536


def prepare(case, seed):
    kind = case["kind"]
    if kind == "forward":
        shapes, prunes = BLOCKS[case["block"]]
        ws = make_weights(shapes, prunes, case["k"], case["quant"], seed)
        blobs = hac.hac_net_encode([w.cpu().numpy() for w in ws], [hac.HAC_FORMAT_SHAC] * len(ws)).to_device(DEV)
        g = torch.Generator(device=DEV)
        g.manual_seed(seed + 2)
        biases = [torch.randn(m, generator=g, device=DEV) * 0.1 for _, m in shapes]
        layers = [(b, bias, i + 1 < len(shapes)) for i, (b, bias) in enumerate(zip(blobs, biases))]
        return {"kind": kind, "layers": layers, "x": make_batch(case["batch"], shapes[0][0], seed)}
    n, m = case["n"], case["m"]
    (w,) = make_weights(((n, m),), (case.get("prune", 0.0),), case["k"], case["quant"], seed)
    if kind == "encode":
        return {"kind": kind, "w": w, "format": FORMATS[case["format"]], "coding": coding(case["format"]),
                "arena": torch.zeros(arena_bytes(case), dtype=torch.uint8, device=DEV)}
    if kind == "encode_host":
        return {"kind": kind, "w": w.cpu().numpy(), "format": case["format"], "arena": np.zeros(arena_bytes(case), np.uint8)}
    x = make_batch(case["batch"], n, seed)
    if kind == "im":
        return {"kind": kind, "blob": hac.im_encode(w.cpu().numpy()).to_device(DEV), "x": x}
    blob = hac.hac_encode_dev(w, FORMATS[case["format"]], ri_coding=coding(case["format"]))
    state = {"kind": kind, "call": hac.hac_dot if case["format"] == "hac" else hac.shac_dot, "blob": blob, "x": x,
             "buffers": case["buffers"]}
    if case["buffers"] != "none":
        state["y"] = torch.empty((case["batch"], m), device=DEV)
    if case["buffers"] == "kept":
        need = hac.hac_workspace_bytes(blob.desc, case["batch"])
        state["workspace"] = torch.empty(max(need, 256), dtype=torch.uint8, device=DEV)
    return state


# ---- one pass -----------------------------------------------------------------------------------


def run(state):
    kind = state["kind"]
    if kind == "dot":
        if state["buffers"] == "none":
            return state["call"](state["blob"], state["x"])
        if state["buffers"] == "kept":
            return state["call"](state["blob"], state["x"], Y=state["y"], workspace=state["workspace"])
        return hac.hac_dot_noalloc(state["blob"], state["x"], state["y"])
    if kind == "im":
        return hac.im_dot(state["blob"], state["x"])
    if kind == "forward":
        return hac.hac_forward(state["layers"], state["x"])
    if kind == "encode":
        blob = hac.hac_encode_dev(state["w"], state["format"], ri_coding=state["coding"]).tensor
        state["arena"][:blob.numel()].copy_(blob)
        return state["arena"]
    if state["format"] == "hac":
        data = hac.hac_encode(state["w"]).data
    else:
        data = hac.shac_encode(state["w"], ri_coding=coding(state["format"])).data
    state["arena"][:data.size] = data
    return state["arena"]


# ---- what a pass cannot do without ----------------------------------------------------------------


def value_bits(k, quant, prune):
    """Bits per non-zero's value: the entropy of the shared values of a pruned Gaussian layer."""
    if quant == "kmeans":
        return 0.95 * math.log2(k)
    cdf = statistics.NormalDist().cdf
    cut, top = (statistics.NormalDist().inv_cdf((1 + prune) / 2) if prune > 0 else 0.0), 5.3
    edges = [-top + 2 * top * i / k for i in range(k + 1)]
    p = []
    for a, b in zip(edges[:-1], edges[1:]):
        q = max(0.0, cdf(min(b, -cut)) - cdf(min(a, -cut))) + max(0.0, cdf(max(b, cut)) - cdf(max(a, cut)))
        p.append(q)
    total = sum(p)
    return -sum(q / total * math.log2(q / total) for q in p if q > 0)


def blob_bytes(fmt, n, m, prune, k, quant):
    """The compressed matrix itself: coded stream and row positions (tables and index left out)."""
    nz, bits = (1 - prune) * n * m, value_bits(k, quant, prune)
    if fmt == "hac":
        return (n * m + nz * bits) / 8                                  # about a bit per zero
    if fmt == "rice":
        return nz * (bits + 1.6 + max(0.0, math.log2(1 / (1 - prune)))) / 8
    return nz * (bits + max(1, math.ceil(math.log2(n)))) / 8 + 4 * (m + 1)


def work(case):
    kind = case["kind"]
    if kind == "forward":
        shapes, prunes = BLOCKS[case["block"]]
        b = case["batch"]
        size = sum(blob_bytes("shac", n, m, p, case["k"], case["quant"]) + 4 * m for (n, m), p in zip(shapes, prunes))
        return {"bytes": size + 4 * b * (shapes[0][0] + shapes[-1][1]),
                "flops": sum(2.0 * b * n * m * (1 - p) for (n, m), p in zip(shapes, prunes))}
    n, m = case["n"], case["m"]
    if kind == "im":
        return {"bytes": n * m + 4 * case["batch"] * (n + m), "flops": 2.0 * case["batch"] * n * m}
    size = blob_bytes(case["format"], n, m, case["prune"], case["k"], case["quant"])
    if kind in ("encode", "encode_host"):
        return {"bytes": 4 * n * m + size, "flops": 0}
    return {"bytes": size + 4 * case["batch"] * (n + m), "flops": 2.0 * case["batch"] * (1 - case["prune"]) * n * m}


def tolerance(case):
    """Sums of fp32 products: another order of the additions.  Blobs are whole bytes."""
    return "exact" if case["kind"].startswith("encode") else {"rel": 1e-5}
