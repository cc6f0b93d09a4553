"""The work that programs built on this library have it do, as cases to be timed and compared.

A case is a dict of plain values.  `kind` says which public entry points it goes through:

  layer    ConvLayer.forward: one stride-1 int8 convolution layer, int32 output (rnswino_conv2d);
  requant  rnswino_conv2d_requant: the layer as a chain runs it, int8 output after shift and clamp, optionally pooled;
  stack    ConvStack.forward: the 13-layer 3x3 chain of the VGG16 configuration, every layer's int8 activations;
  filter   ConvLayer.set_weights: the filter transform of a layer, run when weights are loaded;
  direct   rnswino_direct_conv2d: the library's direct convolution (the method's comparison baseline).

Values are uniform int8, as in the benchmark and the tests.  Every result is an integer and has to be the same to the bit.
"""
from __future__ import annotations

import math

import torch

import paper_2007_12216_amd as rn
import synth_inputs as si
from paper_2007_12216_amd.layer import ConvLayer
from paper_2007_12216_amd.stack import ConvStack

DEVICE = "cuda:0"
THREE, FOUR, WIDE = (251, 241, 239), (251, 241, 239, 233), (65521, 65519)
MODULI = {"three": THREE, "four": FOUR, "wide": WIDE}


def _layer(name, kind, N, C, K, H, W, r, m, moduli, trusted=False, shift=0, pool=False):
    return dict(name=name, kind=kind, N=N, C=C, K=K, H=H, W=W, r=r, m=m, pad=r // 2, moduli=moduli, trusted=trusted,
                shift=shift, pool=pool)


def listed():
    return [
        # the smallest layer of the configurations: nothing but launches and latency
        _layer("layer 16ch 16x16", "layer", 1, 16, 16, 16, 16, 3, 8, "three"),
        # the headline layer: one image through a middle layer of VGG16
        _layer("layer 256ch 56x56", "layer", 1, 256, 256, 56, 56, 3, 8, "four"),
        # the largest transform tile with a 5x5 filter, one image
        _layer("layer 5x5 128ch 28x28", "layer", 1, 128, 128, 28, 28, 5, 12, "four"),
        # the 16-bit number system: two residues of two bytes, one image
        _layer("layer 512ch 28x28 16-bit", "layer", 1, 512, 512, 28, 28, 3, 14, "wide"),
        # the paper's own setting (F(14,3), three moduli with a trusted range) on a batch of a late layer
        _layer("layer 512ch 28x28 trusted b4", "layer", 4, 512, 512, 28, 28, 3, 14, "three", trusted=True),
        # an Inception-style 5x5 layer at batch 8, odd plane
        _layer("layer 5x5 48ch 35x35 b8", "layer", 8, 48, 64, 35, 35, 5, 12, "four"),
        # nothing fits anything: odd planes, channels and filters off every block size, a tile of 6
        _layer("layer 100ch 57x43 ragged b3", "layer", 3, 100, 75, 57, 43, 3, 6, "four"),
        # an early layer of a batch as a chain runs it, with pooling
        _layer("requant 64ch 112x112 b8", "requant", 8, 64, 128, 112, 112, 3, 8, "four", shift=11, pool=True),
        # one image through the whole chain: 13 layers, the latency of a single request
        dict(name="stack b1", kind="stack", N=1, HW=224),
        # the whole chain at the batch of the configuration: the largest work here
        dict(name="stack b8", kind="stack", N=8, HW=224),
        # the weights of the largest layers of that chain, transformed once when they are loaded
        _layer("filter 512x512", "filter", 1, 512, 512, 28, 28, 3, 8, "four"),
        # the direct convolution on the headline layer's shape at batch 8
        _layer("direct 256ch 56x56 b8", "direct", 8, 256, 256, 56, 56, 3, 8, "four"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    limit = work(dict(kind="stack", N=8, HW=224))
    while True:
        kind = rng.choice(("layer", "layer", "layer", "layer", "requant", "requant", "stack", "filter", "direct"))
        if kind == "stack":
            return dict(kind="stack", N=rng.randint(1, 8), HW=16 * rng.randint(2, 13))
        r, m = rng.choice(((3, 8), (3, 8), (3, 8), (3, 6), (3, 7), (3, 4), (3, 14), (3, 10), (5, 12), (5, 8), (5, 4)))
        C, K = _log_int(rng, 3, 512), _log_int(rng, 8, 512)
        H = _log_int(rng, 7, 224)
        W = H if rng.random() < 0.5 else _log_int(rng, 7, 224)
        worst = (1 << 14) * r * r * C
        moduli = "wide" if rng.random() < 0.2 and m != 4 else "three" if worst <= 7228674 else "four"
        trusted = moduli == "four" and rng.random() < 0.15
        pool = kind == "requant" and m in (4, 8) and W % 4 == 0 and H % 2 == 0 and rng.random() < 0.5
        shift = int(round(math.log2(74.0 * math.sqrt(r * r * C)))) if kind == "requant" else 0
        case = _layer(None, kind, rng.randint(1, 8), C, K, H, W, r, m, "three" if trusted else moduli, trusted, shift, pool)
        del case["name"]
        w = work(case)
        # no larger than the largest listed case, and a transform domain that leaves room for three states
        tiles = case["N"] * -(-H // m) * -(-W // m)
        domain = tiles * (m + r - 1) ** 2 * len(MODULI[case["moduli"]]) * (2 if case["moduli"] == "wide" else 1) * (C + K)
        if w["bytes"] <= limit["bytes"] and w["flops"] <= limit["flops"] / 4 and domain <= 1 << 29:
            return case


def _moduli_flags(case):
    return MODULI[case["moduli"]], rn.FLAG_ALLOW_UNCHECKED_RANGE if case["trusted"] else 0


def _uniform(gen, shape):
    return torch.randint(-128, 128, shape, dtype=torch.int8, device=DEVICE, generator=gen)


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE).manual_seed(int(seed))
    if case["kind"] == "stack":
        layers = si.vgg16_stack(batch=case["N"], hw=case["HW"])
        stack = ConvStack(layers, device=DEVICE)
        stack.set_weights([_uniform(gen, (l["K"], l["C"], l["r"], l["r"])).cpu().numpy() for l in layers])
        return dict(kind="stack", stack=stack, x=_uniform(gen, (case["N"], 3, case["HW"], case["HW"])))
    N, C, K, H, W, r, pad = (case[k] for k in ("N", "C", "K", "H", "W", "r", "pad"))
    x = _uniform(gen, (N, C, H, W))
    w = _uniform(gen, (K, C, r, r))
    Ho, Wo = H + 2 * pad - r + 1, W + 2 * pad - r + 1
    state = dict(kind=case["kind"], x=x, w=w)
    if case["kind"] == "direct":
        stream = torch.cuda.current_stream().cuda_stream
        state["wt"] = torch.empty(rn.rnswino_direct_filter_bytes(C, K, r), dtype=torch.uint8, device=DEVICE)
        state["ws"] = torch.empty(rn.rnswino_direct_workspace_bytes(N, C, H, W, pad), dtype=torch.uint8, device=DEVICE)
        state["y"] = torch.empty((N, K, Ho, Wo), dtype=torch.int32, device=DEVICE)
        state["dims"] = (N, C, K, H, W, r, pad)
        rn.rnswino_direct_filter_pack(w, state["wt"], C, K, r, stream)
        return state
    moduli, flags = _moduli_flags(case)
    state["layer"] = ConvLayer(N, C, K, H, W, r, case["m"], pad, moduli, flags, device=DEVICE)
    if case["kind"] != "filter":
        state["layer"].set_weights(w)
    if case["kind"] == "requant":
        pool = case["pool"]
        state["shift"], state["pool"] = case["shift"], pool
        state["a"] = torch.empty((N, K, Ho // 2, Wo // 2) if pool else (N, K, Ho, Wo), dtype=torch.int8, device=DEVICE)
    return state


def run(state):
    kind = state["kind"]
    if kind == "layer":
        return state["layer"].forward(state["x"])
    if kind == "stack":
        state["stack"].forward(state["x"])
        return list(state["stack"].act)
    if kind == "filter":
        state["layer"].set_weights(state["w"])
        return state["layer"].U
    stream = torch.cuda.current_stream().cuda_stream
    if kind == "requant":
        layer = state["layer"]
        rn.rnswino_conv2d_requant(layer.plan, state["x"], layer.U, state["a"], state["shift"], state["pool"], layer.workspace, stream)
        return state["a"]
    rn.rnswino_direct_conv2d(state["x"], state["wt"], state["y"], *state["dims"], state["ws"], stream)
    return state["y"]


def _layer_work(N, C, K, H, W, r, m, pad, moduli, out_bytes):
    """One layer: the activations and the transformed filter read, the output written; the products of the residue GEMM
    (a 16-bit product is four int8 products on this chip)."""
    Ho, Wo, t = H + 2 * pad - r + 1, W + 2 * pad - r + 1, m + r - 1
    wide = moduli[0] > 255
    tiles = N * -(-Ho // m) * -(-Wo // m)
    domain = len(moduli) * t * t * K * C
    return {"bytes": N * C * H * W + domain * (2 if wide else 1) + out_bytes, "flops": 2 * domain * tiles * (4 if wide else 1)}


def work(case):
    if case["kind"] == "stack":
        total = {"bytes": case["N"] * 3 * case["HW"] ** 2, "flops": 0}
        for l in si.vgg16_stack(batch=case["N"], hw=case["HW"]):
            out = l["N"] * l["K"] * l["H"] * l["W"] // (4 if l["pool"] else 1)
            w = _layer_work(l["N"], l["C"], l["K"], l["H"], l["W"], l["r"], l["m"], l["pad"], l["moduli"], out)
            # a layer's activations are written once and read once by the next
            total["bytes"] += w["bytes"]
            total["flops"] += w["flops"]
        total["bytes"] -= case["N"] * 3 * case["HW"] ** 2          # the first layer's input was counted twice
        return total
    N, C, K, H, W, r, pad, m = (case[k] for k in ("N", "C", "K", "H", "W", "r", "pad", "m"))
    Ho, Wo, t = H + 2 * pad - r + 1, W + 2 * pad - r + 1, m + r - 1
    moduli, _ = _moduli_flags(case)
    if case["kind"] == "filter":
        n, rb = len(moduli), 2 if moduli[0] > 255 else 1
        return {"bytes": K * C * r * r + n * t * t * K * C * rb, "flops": 2 * n * K * C * (t * r * r + t * t * r)}
    if case["kind"] == "direct":
        return {"bytes": N * C * H * W + K * C * r * r + 4 * N * K * Ho * Wo, "flops": 2 * N * K * C * Ho * Wo * r * r}
    if case["kind"] == "requant":
        return _layer_work(N, C, K, H, W, r, m, pad, moduli, N * K * Ho * Wo // (4 if case["pool"] else 1))
    return _layer_work(N, C, K, H, W, r, m, pad, moduli, 4 * N * K * Ho * Wo)


def tolerance(case):
    return "exact"
