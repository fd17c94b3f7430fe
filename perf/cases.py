"""The calls that users of this library make, as cases to be measured.

The library runs the 3x3 convolutions of a pruned network (pattern and connectivity sparsity).  A
user packs the layers of a network once and then calls conv2d / conv2d_pool2x2 / maxpool2x2 on
activations that live on the GPU.  A case is therefore either one layer or the 3x3 layers of one of
the two networks whose shapes this repository carries, with the batch, data type, memory layout,
stride and sparsity that such a program has.
"""
import math

import numpy as np
import torch

import paper_1909_05073_amd as P
from pconv_inputs import LayerSpec, make_layer, resnet50_conv3x3_shapes, vgg16_conv_shapes

CENTRED = [m for m in range(512) if bin(m).count("1") == 4 and (m >> 4) & 1]


def _layer(name, n, c_in, c_out, h, w, dtype="f32", layout="nchw", stride=1, masks="table8", dist="zipf",
           counts="pm30", keep=3.6, relu=True, bias=True):
    return dict(name=name, kind="layer", n=n, c_in=c_in, c_out=c_out, h=h, w=w, dtype=dtype, layout=layout,
                stride=stride, masks=masks, dist=dist, counts=counts, keep=keep, relu=relu, bias=bias)


def _net(name, net, n, dtype, layout="nchw"):
    return dict(name=name, kind="net", net=net, n=n, dtype=dtype, layout=layout,
                keep=3.6 if net == "vgg16" else 2.5)


def listed():
    return [
        # the smallest call: one little layer, one image; launch and host time are all of it
        _layer("f32_16ch_16x16_b1", 1, 16, 16, 16, 16, dist="uniform", counts="bernoulli", keep=2.0, relu=False),
        # one ordinary layer of a network that serves single images
        _layer("f32_256ch_56x56_b1", 1, 256, 256, 56, 56, relu=False),
        # image classification, one image at a time: the whole chain of layers and pools
        _net("vgg16_f32_b1", "vgg16", 1, "f32"),
        # the same network with a full batch: throughput (the largest case)
        _net("vgg16_f32_b32", "vgg16", 32, "f32"),
        # many images, strong and very uneven pruning
        _layer("f32_512ch_28x28_b64_uneven", 64, 512, 512, 28, 28, masks="table12", dist="uniform",
               counts="geometric", keep=8.0, relu=False),
        # sizes that are multiples of nothing, patterns of the user's own, no bias
        _layer("f32_odd_b3", 3, 99, 150, 37, 45, masks="random16", dist="uniform", counts="bernoulli", keep=2.0,
               bias=False),
        # down-sampling layer of a residual network, fp32
        _layer("f32_stride2_128ch_56x56_b16", 16, 128, 128, 56, 56, stride=2, keep=2.5),
        # channels-last fp32 activations, as some frameworks keep them
        _layer("f32_nhwc_128ch_28x28_b8", 8, 128, 128, 28, 28, layout="nhwc"),
        # residual network in bf16 with a full batch: throughput
        _net("resnet50_bf16_b32", "resnet50", 32, "bf16"),
        # the same layers for one image: latency
        _net("resnet50_bf16_b1", "resnet50", 1, "bf16"),
        # channels-last bf16, middling batch
        _net("resnet50_bf16_nhwc_b8", "resnet50", 8, "bf16", "nhwc"),
        # bf16 with odd sizes and few kernels kept
        _layer("bf16_odd_b5", 5, 100, 130, 27, 31, dtype="bf16", counts="bernoulli", keep=6.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    if rng.random() < 0.25:
        net = rng.choice(["vgg16", "resnet50", "resnet50"])
        n = _log_int(rng, 1, 24 if net == "vgg16" else 48)
        c = _net("", net, n, "f32" if net == "vgg16" else "bf16",
                 "nchw" if net == "vgg16" else rng.choice(["nchw", "nhwc"]))
        del c["name"]
        return c
    while True:
        n, c_in, c_out = _log_int(rng, 1, 64), _log_int(rng, 8, 512), _log_int(rng, 8, 512)
        h = _log_int(rng, 7, 224)
        w = h if rng.random() < 0.6 else max(7, min(224, int(h * rng.uniform(0.6, 1.6))))
        if rng.random() < 0.5:                       # half of the layers have the usual round channel counts
            c_in, c_out = (max(8, c // 32 * 32) for c in (c_in, c_out))
        keep = rng.choice([2.0, 2.5, 3.6, 5.0, 8.0])
        c = _layer("", n, c_in, c_out, h, w, dtype=rng.choice(["f32", "f32", "bf16"]),
                   layout=rng.choice(["nchw", "nchw", "nhwc"]), stride=rng.choice([1, 1, 1, 2]),
                   masks=rng.choice(["table4", "table8", "table12", "random16"]), dist=rng.choice(["zipf", "uniform"]),
                   counts=rng.choice(["pm30", "bernoulli", "geometric"]), keep=keep, relu=rng.random() < 0.7,
                   bias=rng.random() < 0.8)
        del c["name"]
        k = work(c)
        if 2e5 < k["flops"] < 1.2e10 and k["bytes"] < 4e8:
            return c


def _specs(case):
    """The case's layers as (spec, bias used, pooled afterwards)."""
    if case["kind"] == "layer":
        return [LayerSpec("layer", case["n"], case["c_in"], case["c_out"], case["h"], case["w"], stride=case["stride"],
                          dtype=case["dtype"], num_patterns={"table4": 4, "table12": 12}.get(case["masks"], 8),
                          pattern_dist=case["dist"], keep_div=case["keep"], count_dist=case["counts"], relu=case["relu"])]
    if case["net"] == "vgg16":
        return [LayerSpec("vgg", case["n"], ci, co, s, s, dtype=case["dtype"], keep_div=1.0 if i == 0 else case["keep"],
                          num_patterns=1 if i == 0 else 8, pattern_dist="dense" if i == 0 else "zipf",
                          count_dist="all" if i == 0 else "pm30", pool_after=pool)
                for i, (ci, co, s, pool) in enumerate(vgg16_conv_shapes())]
    return [LayerSpec("rn50", case["n"], c, c, s, s, stride=st, dtype=case["dtype"], keep_div=case["keep"])
            for c, s, st in resnet50_conv3x3_shapes()]


def _weights(case, spec, seed):
    L = make_layer(spec, seed)
    if case.get("masks") == "random16":
        # a pattern table of the user's own: 16 four-tap masks with the centre
        rng = np.random.default_rng(seed + 1)
        L["table"] = np.sort(rng.choice(CENTRED, 16, replace=False)).astype(np.uint16)
        L["pattern_id"] = rng.integers(0, 16, L["pattern_id"].shape).astype(np.uint8)
    return L


def _activations(spec, layout, gen, dtype):
    shape = (spec.n, spec.c_in, spec.h, spec.w) if layout == "nchw" else (spec.n, spec.h, spec.w, spec.c_in)
    return torch.randn(shape, device="cuda", generator=gen).clamp_(min=0).to(dtype)


def prepare(case, seed):
    dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    layout = case["layout"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    layers = []
    chained = case["kind"] == "net" and case["net"] == "vgg16"
    for i, s in enumerate(_specs(case)):
        L = _weights(case, s, seed + 1000 * i)
        ly = dict(relu=s.relu, stride=s.stride,
                  h=P.pconv_pack(L["w"], L["pattern_id"], L["conn"], L["table"], case["dtype"]),
                  bias=torch.from_numpy(L["bias"]).cuda() if case.get("bias", True) else None)
        if i == 0 or not chained:
            ly["x"] = _activations(s, layout, gen, dtype)
        if case["kind"] == "net":
            # a network keeps its activation buffers; a single layer's output is allocated by the call
            out = (s.n, s.c_out, s.h_out, s.w_out) if layout == "nchw" else (s.n, s.h_out, s.w_out, s.c_out)
            ly["fuse"] = bool(s.pool_after) and P.pconv_pool2x2_fusion(ly["h"], s.n, s.h, s.w, layout, case["dtype"]) == 2
            ly["pool"] = bool(s.pool_after) and not ly["fuse"]
            ly["ends_block"] = bool(s.pool_after)
            if ly["fuse"]:
                out = (s.n, s.c_out, s.h_out // 2, s.w_out // 2)
            ly["y"] = torch.empty(out, device="cuda", dtype=dtype)
        layers.append(ly)
    return dict(case=case, layers=layers, chained=chained)


def run(state):
    case, layers = state["case"], state["layers"]
    layout = case["layout"]
    if case["kind"] == "layer":
        ly = layers[0]
        return P.conv2d(ly["h"], ly["x"], ly["bias"], stride=ly["stride"], relu=ly["relu"], layout=layout)
    if not state["chained"]:
        return [P.conv2d(ly["h"], ly["x"], ly["bias"], stride=ly["stride"], relu=ly["relu"], layout=layout, out=ly["y"])
                for ly in layers]
    cur = layers[0]["x"]
    maps = []                                        # what each block of the network hands on
    for ly in layers:
        if ly["fuse"]:
            cur = P.conv2d_pool2x2(ly["h"], cur, ly["bias"], relu=ly["relu"], out=ly["y"])
        else:
            cur = P.conv2d(ly["h"], cur, ly["bias"], relu=ly["relu"], layout=layout, out=ly["y"])
            if ly["pool"]:
                cur = P.maxpool2x2(cur, layout)
        if ly["ends_block"]:
            maps.append(cur)
    return maps


def work(case):
    """Weights kept (on average over the drawn masks), inputs and outputs of every layer once."""
    el = 4 if case["dtype"] == "f32" else 2
    byts = flops = 0.0
    for s in _specs(case):
        if s.count_dist == "geometric":
            m = s.c_in / s.keep_div
            kernels = s.c_out * m * (1.0 - (1.0 - 1.0 / m) ** s.c_in) if m > 1.0 else float(s.c_out)
        else:
            kernels = s.c_out * s.c_in / s.keep_div
        nnz = kernels * (9 if s.pattern_dist == "dense" else 4)
        out = s.c_out * ((s.h_out // 2) * (s.w_out // 2) if s.pool_after else s.h_out * s.w_out)
        flops += 2.0 * nnz * s.n * s.h_out * s.w_out
        byts += el * (s.n * (s.c_in * s.h * s.w + out) + nnz) + 2.0 * kernels + 4.0 * s.c_out
    return {"bytes": byts, "flops": flops}


def tolerance(case):
    # Measured against sums in 64 bits and multiplied by about four: fp32 0.7e-7 to 1.3e-7 in the
    # 2-norm and up to 3.7e-6 for a single value (sums of up to some thousand terms); bf16 1.66e-3,
    # which is the rounding of the output, and one step of bf16 (2^-7 at most) for a single value.
    if case["dtype"] == "bf16":
        return {"rel": 7e-3, "max": 1.6e-2}
    return {"rel": 6e-7, "max": 1.6e-5}
