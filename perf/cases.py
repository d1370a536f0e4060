"""What a user of this library has it do, as measurable cases: inference from compressed
fully connected layers and stacks (one request up to large batches), convolutions, a whole
network, several resident models at once, decoding a layer, compressing one, and bringing a
stored one onto the device.

A model is what a program keeps: it is compressed once per process, from weights drawn from
a seed of its own, and shared by all states of a case; what the seed of prepare() changes is
the request (activations, or the weights to compress).  Shapes, densities and bit widths are
those of the benchmark configurations in workloads.py; draw() spreads over the same ranges.
"""
from __future__ import annotations

import math
from collections import OrderedDict

import numpy as np
import torch

import paper_1711_00244_amd as cl
from paper_1711_00244_amd import network

BLOCK = 128                      # the block size all benchmark configurations use
PATHS = {"auto": cl.PATH_AUTO, "bf16": cl.PATH_MFMA_BF16}


# --------------------------------------------------------------------------- #
# the cases
# --------------------------------------------------------------------------- #
def _stack(name, widths, densities, k, batch, path="auto"):
    c = dict(kind="stack", k0=widths[0], m1=widths[1], m2=widths[2], m3=widths[3], d1=densities[0], d2=densities[1],
             d3=densities[2], r=5, k=k, batch=batch, path=path)
    return dict(c, name=name) if name else c


ALEXNET = ((9216, 4096, 4096, 1000), (0.09, 0.09, 0.25), 4)
VGG16 = ((25088, 4096, 4096, 1000), (0.04, 0.04, 0.23), 5)


def listed():
    return [
        # the smallest call: one request through one small layer (configuration 1); launches and the host path are all of it
        dict(name="fc1024-b1", kind="fc", M=1024, K=1024, density=0.10, r=5, k=4, batch=1, path="auto"),
        # a single request through the FC stack: the latency of interactive serving (configuration 3, batch 1)
        _stack("alexnet-fc-b1", *ALEXNET, 1),
        # a few requests taken together (configuration 3, batch 16)
        _stack("alexnet-fc-b16", *ALEXNET, 16),
        # the batch the variable-batch planner picks for the larger stack under its memory cap (configuration 5)
        _stack("vgg16-fc-b64", *VGG16, 64),
        # throughput serving, the headline batch (configuration 3, batch 256)
        _stack("alexnet-fc-b256", *ALEXNET, 256),
        # the same on the looser-tolerance bf16 tiles
        _stack("alexnet-fc-b256-bf16", *ALEXNET, 256, "bf16"),
        # one request for each of sixteen resident models of one shape, served in one grid
        dict(name="fc7-group16-b1", kind="group", n=16, M=4096, K=4096, density=0.09, r=5, k=4, batch=1),
        # one convolution for one image (VGG-16 conv4_2)
        dict(name="vgg16-conv4-b1", kind="conv", C=512, H=28, W=28, R=3, stride=1, pad=1, groups=1, OC=512, density=0.27, r=8, k=5,
             batch=1, path="auto"),
        # the whole network, a throughput batch: convolutions, normalisation, pooling, FC (configurations 3 and 4)
        dict(name="alexnet-net-b64", kind="net", batch=64),
        # decoding a layer to symbols and dense weights (fc6)
        dict(name="fc6-decode", kind="decode", M=4096, K=9216, density=0.09, r=5, k=4),
        # compressing a layer on the host and storing it (fc7)
        dict(name="fc7-compress", kind="compress", M=4096, K=4096, density=0.09, r=5, k=4),
        # a stored model brought onto the device, up to its first answer (fc6)
        dict(name="fc6-load", kind="load", M=4096, K=9216, density=0.09, r=5, k=4),
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def layer(most=38_000_000):
        while True:
            M, K = log(96, 4608), log(128, 25088)
            if 40_000 <= M * K <= most:
                return dict(M=M, K=K, density=round(math.exp(rng.uniform(math.log(0.04), math.log(0.30))), 3), r=5, k=rng.choice((4, 5)))

    kind = rng.choices(("fc", "stack", "group", "conv", "net", "decode", "compress", "load"), (12, 34, 10, 18, 6, 8, 6, 6))[0]
    if kind == "fc":
        return dict(kind=kind, batch=log(1, 1024), path=rng.choice(("auto", "auto", "auto", "bf16")), **layer())
    if kind == "stack":
        widths = (log(1024, 25088), log(512, 4608), log(512, 4608), log(10, 1200))
        densities = tuple(round(rng.uniform(lo, hi), 3) for lo, hi in ((0.03, 0.12), (0.03, 0.12), (0.15, 0.30)))
        return _stack(None, widths, densities, rng.choice((4, 5)), log(1, 1024), rng.choice(("auto",) * 5 + ("bf16",)))
    if kind == "group":
        return dict(kind=kind, n=log(2, 32), batch=rng.choice((1, 2, 4, 8)), **layer(10_000_000))
    if kind == "conv":
        while True:
            groups = rng.choice((1, 1, 1, 2))
            R = rng.choice((3, 3, 3, 5, 11))
            C, OC, H = log(3, 512) // groups * groups, log(32, 512), log(7, 224)
            if groups > 1:
                C, OC = max(groups, C), max(32, OC // 32 * 32)
            stride = rng.choice((1, 1, 1, 2, 4)) if R > 3 else rng.choice((1, 1, 1, 2))
            c = dict(kind=kind, C=C, H=max(H, R), W=max(H, R), R=R, stride=stride, pad=R // 2, groups=groups, OC=OC,
                     density=round(rng.uniform(0.20, 0.85), 3), r=8, k=rng.choice((5, 8)), batch=log(1, 64),
                     path=rng.choice(("auto", "auto", "auto", "bf16")))
            P = (c["H"] + 2 * c["pad"] - R) // stride + 1
            dense = 2.0 * OC * (C // groups) * R * R * P * P * c["batch"]
            if 2e7 <= dense <= 4e10 and c["batch"] * C * c["H"] * c["W"] <= 1 << 26:
                return c
    if kind == "net":
        return dict(kind=kind, batch=log(1, 63))
    return dict(kind=kind, **layer(17_000_000 if kind == "compress" else 38_000_000))


# --------------------------------------------------------------------------- #
# models: kept by the process, as by a program that serves them
# --------------------------------------------------------------------------- #
_kept: OrderedDict = OrderedDict()


def _keep(key, make):
    if key not in _kept:
        _kept[key] = make()
        while len(_kept) > 24:
            _kept.popitem(last=False)
    _kept.move_to_end(key)
    return _kept[key]


def _weights(M, K, density, seed, mask_seed=None):
    """Pruned weights on the host: N(0, 0.01), each kept with probability `density`."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    W = torch.randn((M, K), generator=g, device="cuda").mul_(0.01)
    if mask_seed is not None:
        g.manual_seed(mask_seed)
    W[torch.rand((M, K), generator=g, device="cuda") >= density] = 0.0
    return W.cpu().numpy()


def _layer(M, K, density, r, k, block_h=BLOCK, copy=0):
    def make():
        return cl.compress_layer(_weights(M, K, density, 1711 + copy), r, k, block_h, BLOCK, upload=True)
    return _keep((M, K, density, r, k, block_h, copy), make)


def _stored(c):
    return _keep(("stored", c["M"], c["K"], c["density"], c["r"], c["k"]), lambda: _layer(c["M"], c["K"], c["density"], c["r"], c["k"]).serialize())


def _group(c):
    # resident models of one shape: four different ones, the rest copies with device memory of their own
    def make():
        made = [cl.compress_layer(_weights(c["M"], c["K"], c["density"], 1711 + i), c["r"], c["k"], BLOCK, BLOCK) for i in range(min(4, c["n"]))]
        stored = [L.serialize() for L in made]
        return cl.LayerGroup([cl.layer_deserialize(stored[i % len(stored)]).upload() for i in range(c["n"])])
    return _keep(("group", c["n"], c["M"], c["K"], c["density"], c["r"], c["k"]), make)


def _stack_layers(c):
    widths = (c["k0"], c["m1"], c["m2"], c["m3"])
    return [_layer(widths[i + 1], widths[i], c["d%d" % (i + 1)], c["r"], c["k"]) for i in range(3)]


def _conv(c):
    geom = {n: c[n] for n in ("C", "H", "W", "R", "stride", "pad", "groups", "OC")}
    geom["S"] = c["R"]
    bh = cl.conv_block_h(c["OC"], c["groups"], BLOCK)
    return geom, _layer(c["OC"], c["C"] // c["groups"] * c["R"] * c["R"], c["density"], c["r"], c["k"], bh)


def _net():
    return _keep("net", network.alexnet)


# --------------------------------------------------------------------------- #
# a case's state and one pass
# --------------------------------------------------------------------------- #
def _relu_normal(shape, g):
    return torch.randn(shape, generator=g, device="cuda").clamp_(min=0)


def _bias(n, g):
    return torch.randn(n, generator=g, device="cuda").mul_(0.05)


def _scratch(n):
    return torch.empty(max(256, n), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    c, kind = case, case["kind"]
    g = torch.Generator(device="cuda").manual_seed(seed)
    s = {"kind": kind}
    if kind == "fc":
        L = _layer(c["M"], c["K"], c["density"], c["r"], c["k"])
        s.update(layer=L, path=PATHS[c["path"]], X=_relu_normal((c["batch"], L.K), g), bias=_bias(L.M, g),
                 out=torch.empty((c["batch"], L.M), device="cuda"))
        s["ws"] = _scratch(cl.fc_workspace_bytes(L, c["batch"], s["path"]))
    elif kind == "stack":
        layers = _stack_layers(c)
        s.update(layers=layers, path=PATHS[c["path"]], X=_relu_normal((c["batch"], c["k0"]), g), biases=[_bias(L.M, g) for L in layers],
                 out=torch.empty((c["batch"], c["m3"]), device="cuda"))
        s["ws"] = _scratch(cl.fc_stack_workspace_bytes(layers, c["batch"], s["path"]))
    elif kind == "group":
        G = _group(c)
        s.update(group=G, X=_relu_normal((c["n"], c["batch"], c["K"]), g), bias=_bias(c["n"] * c["M"], g).view(c["n"], c["M"]),
                 out=torch.empty((c["n"], c["batch"], c["M"]), device="cuda"), ws=_scratch(G.workspace_bytes(c["batch"])))
    elif kind == "conv":
        geom, L = _conv(c)
        P = (c["H"] + 2 * c["pad"] - c["R"]) // c["stride"] + 1
        s.update(layer=L, geom=geom, path=PATHS[c["path"]], bias=_bias(c["OC"], g),
                 X=torch.rand((c["batch"], c["C"], c["H"], c["W"]), generator=g, device="cuda"),
                 out=torch.empty((c["batch"], c["OC"], P, P), device="cuda"))
        s["ws"] = _scratch(cl.conv_workspace_bytes(L, geom, c["batch"], s["path"]))
    elif kind == "net":
        s.update(net=_net(), X=torch.rand((c["batch"], 3, 227, 227), generator=g, device="cuda"))
    elif kind == "decode":
        # (nothing but the layer goes in, so its weights follow from the seed; where they sit does
        # not, which keeps the number of entries the same)
        def make():
            return cl.compress_layer(_weights(c["M"], c["K"], c["density"], seed, 1711), c["r"], c["k"], BLOCK, BLOCK, upload=True)
        s["layer"] = _keep((c["M"], c["K"], c["density"], c["r"], c["k"], "values", seed), make)
    elif kind == "compress":
        # the stored form's size varies with the weights: a buffer that holds any
        s.update(W=_weights(c["M"], c["K"], c["density"], seed), r=c["r"], k=c["k"],
                 stored=np.zeros(int(4 * c["density"] * c["M"] * c["K"]) + (1 << 16), np.uint8))
    elif kind == "load":
        s.update(stored=_stored(c), layer=None, X=_relu_normal((1, c["K"]), g), bias=_bias(c["M"], g), out=torch.empty((1, c["M"]), device="cuda"))
        s["ws"] = _scratch(cl.fc_workspace_bytes(_layer(c["M"], c["K"], c["density"], c["r"], c["k"]), 1))
    else:
        raise ValueError(kind)
    return s


def run(s):
    kind = s["kind"]
    if kind == "fc":
        return cl.compressed_fc_forward(s["layer"], s["X"], s["bias"], relu=True, path=s["path"], out=s["out"], workspace=s["ws"])
    if kind == "stack":
        return cl.compressed_fc_stack_forward(s["layers"], s["X"], s["biases"], path=s["path"], out=s["out"], workspace=s["ws"])
    if kind == "group":
        return s["group"].forward(s["X"], bias=s["bias"], relu=True, out=s["out"], workspace=s["ws"])
    if kind == "conv":
        return cl.compressed_conv_forward(s["layer"], s["geom"], s["X"], s["bias"], relu=True, path=s["path"], out=s["out"], workspace=s["ws"])
    if kind == "net":
        return s["net"].run(s["X"])
    if kind == "decode":
        return cl.decode_layer(s["layer"])
    if kind == "compress":
        L = cl.compress_layer(s["W"], s["r"], s["k"], BLOCK, BLOCK)
        data = L.serialize()
        L.free()
        s["stored"][:len(data)] = np.frombuffer(data, np.uint8)
        return {"size": len(data), "data": s["stored"]}
    # load: the model of the pass before gives way to the one that is brought in
    if s["layer"] is not None:
        s["layer"].free()
    s["layer"] = cl.layer_deserialize(s["stored"]).upload()
    return cl.compressed_fc_forward(s["layer"], s["X"], s["bias"], relu=True, out=s["out"], workspace=s["ws"])


# --------------------------------------------------------------------------- #
# what a pass cannot do without, and how far another correct one may be off
# --------------------------------------------------------------------------- #
def _coded_bytes(L):
    """The two Huffman-coded streams and the codebook: a layer's content, whatever the layout."""
    st = L.stats()
    return (st["val_bits"] + st["idx_bits"]) / 8.0 + 1024


def work(case):
    c, kind = case, case["kind"]
    if kind in ("fc", "load", "decode"):
        L = _layer(c["M"], c["K"], c["density"], c["r"], c["k"])
        if kind == "decode":
            return {"bytes": _coded_bytes(L) + 2 * L.stats()["entries"] + 4.0 * c["M"] * c["K"], "flops": 0}
        B = c.get("batch", 1)
        return {"bytes": _coded_bytes(L) + 4.0 * (B * (c["K"] + c["M"]) + c["M"]), "flops": 2.0 * L.stats()["nnz"] * B}
    if kind == "stack":
        layers = _stack_layers(c)
        return {"bytes": sum(_coded_bytes(L) + 4.0 * L.M for L in layers) + 4.0 * c["batch"] * (c["k0"] + c["m3"]),
                "flops": 2.0 * c["batch"] * sum(L.stats()["nnz"] for L in layers)}
    if kind == "group":
        layers = _group(c).layers
        return {"bytes": sum(_coded_bytes(L) + 4.0 * (c["batch"] * (L.K + L.M) + L.M) for L in layers),
                "flops": 2.0 * c["batch"] * sum(L.stats()["nnz"] for L in layers)}
    if kind == "conv":
        _, L = _conv(c)
        P = (c["H"] + 2 * c["pad"] - c["R"]) // c["stride"] + 1
        return {"bytes": _coded_bytes(L) + 4.0 * (c["batch"] * (c["C"] * c["H"] * c["W"] + c["OC"] * P * P) + c["OC"]),
                "flops": 2.0 * L.stats()["nnz"] * P * P * c["batch"]}
    if kind == "net":
        net = _net()
        flops = 0.0
        for op, shape in zip(net.layers, net.shapes[1:]):
            if hasattr(op, "layer"):
                flops += 2.0 * op.layer.stats()["nnz"] * (shape[1] * shape[2] if len(shape) == 3 else 1)
        coded = sum(_coded_bytes(op.layer) for op in net.layers if hasattr(op, "layer"))
        return {"bytes": coded + 4.0 * c["batch"] * (3 * 227 * 227 + 1000), "flops": flops * c["batch"]}
    # compress: the weights in, the stored form out (about 11 bits per surviving weight)
    return {"bytes": 4.0 * c["M"] * c["K"] + 1.4 * c["density"] * c["M"] * c["K"], "flops": 0}


def tolerance(case):
    if case["kind"] in ("decode", "compress"):
        return "exact"
    if case.get("path") == "bf16":
        return {"rel": 1e-4}                 # two bf16 terms per operand: 2^-16 per product, up to three layers
    if case["kind"] == "net":
        return {"rel": 2e-5}                 # eight fp32 layers, one after the other
    return {"rel": 1e-5}                     # fp32 sums
