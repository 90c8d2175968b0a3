"""The calls this library is used for, as cases to measure.

A case is one call of one layer: a convolution layer of a pruned network at some batch size (plain, or with
the bias and ReLU that follow it in a network, or the variant that allocates nothing), or a fully connected
layer.  The handle is made once from the pruned weights, as a program that serves a network keeps it; the
first call packs for the batch size.  Activations are what such layers see: rectified normals inside a
network, plain normals for the first layer's image.  Weights are normals under a Bernoulli mask, or under a
mask whose rows differ (some empty, some dense), which is what pruning with a penalty leaves.
"""
import math

import numpy as np
import torch

from paper_1608_01409_amd import binding
from paper_1608_01409_amd.workloads import Layer


def _conv(name, shape, n, density, entry="forward", mask="bernoulli"):
    c, hw, k, r, stride, pad, groups = shape
    return {"name": name, "kind": "conv", "c": c, "hw": hw, "k": k, "r": r, "stride": stride, "pad": pad, "groups": groups,
            "n": n, "density": density, "entry": entry, "mask": mask}


def _fc(name, c, k, n, density):
    return {"name": name, "kind": "fc", "c": c, "k": k, "n": n, "density": density}


# channels, height = width, filters, filter size, stride, padding, groups
CONV1 = (3, 227, 96, 11, 4, 0, 1)
CONV2 = (96, 27, 256, 5, 1, 2, 2)
CONV3 = (256, 13, 384, 3, 1, 1, 1)
CONV4 = (384, 13, 384, 3, 1, 1, 2)
CONV5 = (384, 13, 256, 3, 1, 1, 2)
GOOG3X3 = (192, 28, 128, 3, 1, 1, 1)
GOOG1X1 = (192, 28, 64, 1, 1, 0, 1)


def listed():
    return [
        # the latency of one image through one layer: the smallest convolution call
        _conv("conv3_n1", CONV3, 1, 0.10),
        # a server that gathers a few requests, bias and ReLU fused
        _conv("conv5_n16_fused", CONV5, 16, 0.10, "fused"),
        # throughput at batch 256, the densities that pruning reaches on these layers
        _conv("conv2_n256", CONV2, 256, 0.10),
        _conv("conv3_n256_fused", CONV3, 256, 0.10, "fused"),
        _conv("conv4_n256_skewed", CONV4, 256, 0.10, "forward", "skewed"),
        # both ends of the density sweep: strongly pruned, and a layer that pruning hardly touched
        _conv("conv5_n256_sparse", CONV5, 256, 0.02),
        _conv("conv4_n256_dense", CONV4, 256, 0.50),
        # inception-like layers at batch 64: 3x3 and the bandwidth-bound 1x1
        _conv("goog3x3_n64_fused", GOOG3X3, 64, 0.20, "fused"),
        _conv("goog1x1_n64", GOOG1X1, 64, 0.30),
        # the strided first layer, which stays rather dense
        _conv("conv1_n64", CONV1, 64, 0.30),
        # fully connected layers: a full batch, and a few requests
        _fc("fc7_n256", 4096, 4096, 256, 0.10),
        _fc("fc8_n4", 4096, 1000, 4, 0.25),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    density = round(_log_uniform(rng, 0.01, 1.0), 4)
    if rng.random() < 0.25:
        while True:
            c, k = int(_log_uniform(rng, 64, 9216)), int(_log_uniform(rng, 16, 4096))
            n = 4 * int(_log_uniform(rng, 1, 256.99))
            if c * k * n * 2 <= 3.5e10 and c * k <= 1.7e7:
                return {k2: v for k2, v in _fc("", c, k, n, density).items() if k2 != "name"}
    while True:
        groups = rng.choice((1, 1, 1, 2))
        c, k = groups * int(_log_uniform(rng, 16, 512) / groups), groups * int(_log_uniform(rng, 16, 512) / groups)
        r = rng.choice((1, 3, 3, 3, 5))
        stride = rng.choice((1, 1, 1, 1, 2)) if r < 5 else 1
        hw = int(_log_uniform(rng, 7, 56.99))
        n = int(_log_uniform(rng, 1, 256.99))
        entry = rng.choice(("forward", "fused")) if n > 2 else rng.choice(("forward", "noalloc"))
        mask = rng.choice(("bernoulli", "bernoulli", "bernoulli", "skewed"))
        if mask == "skewed" and density > 0.3:
            mask = "bernoulli"
        case = _conv("", (c, hw, k, r, stride, r // 2, groups), n, density, entry, mask)
        w = work(case)
        # no more work and no more traffic than the largest listed ones
        if w["flops"] <= 2.8e10 and w["flops"] / density <= 1.1e11 and w["bytes"] <= 2.5e8:
            return {k2: v for k2, v in case.items() if k2 != "name"}


def _layer(case):
    if case["kind"] == "fc":
        return binding.fc_layer(case["c"], case["k"])
    return Layer("layer", case["c"], case["hw"], case["hw"], case["k"], case["r"], case["r"], case["stride"], case["pad"], case["groups"])


def _row_densities(case, rng, k):
    """Per-row densities: all the same, or a fifth of the rows empty and a power law over the others."""
    if case.get("mask", "bernoulli") == "bernoulli":
        return np.full(k, case["density"])
    d = (1.0 - rng.random(k)) ** -0.5
    d[rng.random(k) < 0.2] = 0.0
    for _ in range(20):
        d = np.minimum(d * (case["density"] / max(d.mean(), 1e-9)), 0.8)
    return d


def _data(case, seed):
    """(layer, input on the GPU, pruned weights [K][Cg][R][S] on the host, bias on the GPU or None)"""
    layer = _layer(case)
    rng = np.random.default_rng([160801409, seed])
    k, cols = layer.K, layer.Cg * layer.R * layer.S
    w = rng.standard_normal((k, cols), dtype=np.float32) * np.float32(0.01)
    w[rng.random((k, cols), dtype=np.float32) >= _row_densities(case, rng, k)[:, None]] = 0.0
    bias = torch.from_numpy((rng.standard_normal(k) * 0.05).astype(np.float32)).cuda()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    shape = (case["c"], case["n"]) if case["kind"] == "fc" else (case["n"], layer.C, layer.H, layer.W)
    x = torch.randn(shape, generator=gen, device="cuda")
    if layer.C > 3:
        x.clamp_(min=0.0)
    return layer, x, w.reshape(k, layer.Cg, layer.R, layer.S), bias


def prepare(case, seed):
    layer, x, w, bias = _data(case, seed)
    csr = binding.sconv_create_csr(layer, w)
    shape = (layer.K, case["n"]) if case["kind"] == "fc" else (case["n"], layer.K, layer.OH, layer.OW)
    out = torch.empty(shape, device="cuda")
    entry = case.get("entry", "fc")
    if entry == "noalloc":
        # this entry point wants the packing for the batch size on the device: one ordinary call
        binding.sconv_forward(csr, x, out)
    return {"csr": csr, "x": x, "out": out, "bias": bias, "entry": entry}


def run(state):
    csr, x, out, entry = state["csr"], state["x"], state["out"], state["entry"]
    if entry == "forward":
        return binding.sconv_forward(csr, x, out)
    if entry == "fused":
        return binding.sconv_forward_fused(csr, x, state["bias"], True, out)
    if entry == "noalloc":
        return binding.sconv_forward_noalloc(csr, x, out)
    return binding.sconv_fc_forward(csr, x, state["bias"], True, out)


def work(case):
    layer = _layer(case)
    weights = layer.K * layer.Cg * layer.R * layer.S * case["density"]
    n, positions = case["n"], layer.OH * layer.OW
    return {"bytes": int(4 * n * (layer.C * layer.H * layer.W + layer.K * positions) + 8 * weights),
            "flops": int(2 * weights * positions * n)}


def tolerance(case):
    # fp32 sums in any order: a few 1e-7 of the result against 64 bits, a little more for the longest dense rows
    return {"rel": 2e-6, "max": 2e-5}


def exact(case, seed):
    layer, x, w, bias = _data(case, seed)
    x, b = x.double(), bias.double()
    wd = torch.from_numpy(w).cuda().double()
    if case["kind"] == "fc":
        return (wd.reshape(layer.K, -1) @ x + b[:, None]).clamp_(min=0.0)
    out = torch.empty((case["n"], layer.K, layer.OH, layer.OW), dtype=torch.float64, device="cuda")
    kg = layer.K // layer.groups
    for n in range(case["n"]):
        for g in range(layer.groups):
            cols = torch.nn.functional.unfold(x[n:n + 1, g * layer.Cg:(g + 1) * layer.Cg], (layer.R, layer.S),
                                              padding=layer.pad, stride=layer.stride)[0]
            out[n, g * kg:(g + 1) * kg] = (wd[g * kg:(g + 1) * kg].reshape(kg, -1) @ cols).reshape(kg, layer.OH, layer.OW)
    if case["entry"] == "fused":
        out = (out + b[None, :, None, None]).clamp_(min=0.0)
    return out
