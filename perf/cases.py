"""The work this library is used for, as cases that can be timed.

A case is a dict of plain values.  `listed()` gives the fixed ones, `draw(rng)` one more of the
same ranges, `prepare` builds what a program holds before the call (weights packed, layouts
built, inputs on the GPU), `run` makes one pass through the public entry points.

Five kinds of case:
  net        an op list through build_net / Net.run with its default options (one replayed graph)
  conv       one fused sparse convolution on plain tensors (cadnn_sparse_conv2d)
  dense      one unpruned convolution from raw device weights (cadnn_dense_conv2d)
  fc         one sparse fully connected layer (cadnn_sparse_fc)
  depthwise  one fused depthwise layer (cadnn_depthwise_conv2d)
  pool       one pooling layer between convolutions
"""
from __future__ import annotations

import json
import os
import statistics

import numpy as np
import torch

import paper_1905_00571_amd as cad
import workloads as wl


def _net(family, dtype, n, size, **options):
    return dict({"kind": "net", "family": family, "dtype": dtype, "n": n, "size": size}, **options)


def _conv(dtype, n, cin, cout, h, w, k, stride, pad, sparsity, residual):
    return {"kind": "conv", "dtype": dtype, "n": n, "cin": cin, "cout": cout, "h": h, "w": w, "k": k,
            "stride": stride, "pad": pad, "sparsity": sparsity, "residual": residual}


def listed():
    def named(name, case):
        return dict({"name": name}, **case)

    return [
        # the smallest call: one pruned 3x3 layer on one image, where host work and the launch count
        named("layer-3x3-f32", _conv("f32", 1, 64, 64, 56, 56, 3, 1, 1, 0.9, False)),
        # a strided layer with odd sizes on two images: a grid reduction called on its own
        named("layer-strided-f32", _conv("f32", 2, 288, 384, 35, 35, 3, 2, 0, 0.8, False)),
        # an unpruned layer from raw weights: what a program with dense checkpoints calls
        named("dense-layer-f16", {"kind": "dense", "dtype": "f16", "n": 32, "cin": 256, "cout": 256, "h": 14, "w": 14,
                                  "k": 3, "stride": 1, "pad": 1, "residual": False}),
        # one residual block on one image: a small chain of launches
        named("bottleneck-f32", _net("bottleneck", "f32", 1, 56, sparsity=0.85)),
        # single-image latency of the benchmark network with the kernel choice saved for it
        named("resnet50-f32-n1", _net("resnet50", "f32", 1, 224, recipe="mixed", saved="resnet50_c2_f32_n1.json")),
        # the same network in 2-byte storage: one image, a small batch, a throughput batch
        named("resnet50-f16-n1", _net("resnet50", "f16", 1, 224, recipe="uniform", sparsity=0.8)),
        named("resnet50-f16-n8", _net("resnet50", "f16", 8, 224, recipe="uniform", sparsity=0.8)),
        named("resnet50-f16-n32", _net("resnet50", "f16", 32, 224, recipe="uniform", sparsity=0.8)),
        # a batch in fp32 storage
        named("resnet50-f32-n8", _net("resnet50", "f32", 8, 224, recipe="mixed")),
        # large images and the big fully connected layers
        named("vgg16-f32-n1", _net("vgg16", "f32", 1, 224)),
        # depthwise layers, channel counts that are no powers of two, residual adds without ReLU
        named("mobilenet-v2-f16-n16", _net("mobilenet_v2", "f16", 16, 224)),
        # ragged rows, rectangular filters, branches and concatenations
        named("inception-v3-f32-n1", _net("inception_v3", "f32", 1, 299)),
    ]


def _log(rng, lo, hi):
    """An integer in [lo, hi], spread over its logarithm."""
    return max(lo, min(hi, int(round(float(lo) * (float(hi) / lo) ** rng.random()))))


_IMAGES_AT_224 = 32     # no drawn net does more than this many 224 x 224 images of the residual network, 80 % sparse


def _draw_net(rng):
    dtype = rng.choice(["f32", "f16"])
    family = rng.choice(["resnet50", "resnet50", "vgg16", "mobilenet_v1", "mobilenet_v2", "inception_v3", "bottleneck"])
    top = {"resnet50": 32, "vgg16": 8, "mobilenet_v1": 32, "mobilenet_v2": 32, "inception_v3": 12, "bottleneck": 32}[family]
    if dtype == "f32":
        top //= 4
    size = {"vgg16": rng.randint(224, 255), "bottleneck": _log(rng, 7, 80), "inception_v3": rng.randint(150, 310)}.get(
        family, rng.randint(96, 288))
    options, kept = {}, 0.2
    if family == "resnet50":
        options["recipe"] = rng.choice(["mixed", "uniform"])
    if family == "bottleneck" or options.get("recipe") == "uniform":
        options["sparsity"] = round(rng.uniform(0.5, 0.95), 2)
        kept = max(0.2, 1.0 - options["sparsity"])
    if family in ("resnet50", "inception_v3"):
        room = _IMAGES_AT_224 / (1.0 if dtype == "f16" else 4.0) * 224 * 224 * 0.2 / kept
        top = max(1, min(top, int(room / (size * size))))
    return _net(family, dtype, _log(rng, 1, top), size, **options)


def _draw_conv(rng):
    k = rng.choice([1, 1, 3, 3, 3, 5, 7])
    stride = rng.choice([1, 1, 1, 2])
    if k == 5:
        stride = 1
    h = _log(rng, 7, 112)
    w = h if rng.random() < 0.7 else _log(rng, 7, 112)
    cin, cout = _log(rng, 16, 512), _log(rng, 16, 512)
    if k > 3:
        cin, cout = min(cin, 192), min(cout, 192)
    n = _log(rng, 1, 16)
    while n > 1 and n * cin * cout * k * k * h * w // (stride * stride) > 12 * 10 ** 9:
        n //= 2
    return _conv(rng.choice(["f32", "f16"]), n, cin, cout, h, w, k, stride, k // 2, round(rng.uniform(0.5, 0.95), 2),
                 rng.random() < 0.3)


def _draw_dense(rng):
    c = _draw_conv(rng)
    if c["dtype"] == "f32":
        c["n"] = max(1, c["n"] // 4)
    return {"kind": "dense", "dtype": c["dtype"], "n": c["n"], "cin": c["cin"], "cout": c["cout"], "h": c["h"],
            "w": c["w"], "k": c["k"], "stride": c["stride"], "pad": c["pad"], "residual": c["residual"]}


def draw(rng):
    kind = rng.choice(["net"] * 5 + ["conv"] * 2 + ["dense", "fc", "depthwise", "pool"])
    if kind == "net":
        return _draw_net(rng)
    if kind == "conv":
        return _draw_conv(rng)
    if kind == "dense":
        return _draw_dense(rng)
    dtype = rng.choice(["f32", "f16"])
    if kind == "fc":
        return {"kind": "fc", "dtype": dtype, "n": _log(rng, 1, 64), "cin": _log(rng, 512, 25088), "cout": _log(rng, 256, 4096),
                "sparsity": round(rng.uniform(0.8, 0.97), 2)}
    case = {"kind": kind, "dtype": dtype, "n": _log(rng, 1, 32), "channels": _log(rng, 32, 1024), "h": _log(rng, 7, 112)}
    case["w"] = case["h"]
    if kind == "depthwise":
        case.update(k=3, stride=rng.choice([1, 2]), pad=1)
        return case
    case["op"] = rng.choice(["max", "mean", "global"])
    if case["op"] != "global":
        case["k"], case["stride"], case["pad"] = rng.choice([(3, 2, 1), (2, 2, 0), (3, 1, 1), (3, 2, 0)])
    return case


# ---- what the cases are made of ----------------------------------------------------------

def _ops(case):
    family = case["family"]
    if family == "resnet50":
        return wl.resnet50_ops(uniform=case["sparsity"]) if case["recipe"] == "uniform" else wl.resnet50_ops()
    if family == "bottleneck":
        return wl.bottleneck_conv2x_ops(case["sparsity"])
    return {"vgg16": wl.vgg16_ops, "mobilenet_v1": wl.mobilenet_v1_ops, "mobilenet_v2": wl.mobilenet_v2_ops,
            "inception_v3": wl.inception_v3_ops}[family]()


def _in_shape(case):
    return (case["n"], 256 if case["family"] == "bottleneck" else 3, case["size"], case["size"])


def _dtypes(case):
    return (cad.F16, torch.float16) if case["dtype"] == "f16" else (cad.F32, torch.float32)


def _weights(gen, cout, cin, kh, kw, sparsity, device_tensor=False):
    """He-normal filters whose smallest magnitudes are zero (the pruned checkpoints this library
    serves keep the largest weights of a layer), drawn on the GPU."""
    w = torch.randn(cout, cin, kh, kw, device="cuda", generator=gen)
    if sparsity > 0.0:
        w *= w.abs() > statistics.NormalDist().inv_cdf((1.0 + sparsity) / 2.0)
    w *= (2.0 / (cin * kh * kw)) ** 0.5
    return w if device_tensor else w.cpu().numpy()


def _bias(gen, cout):
    return torch.randn(cout, device="cuda", generator=gen) * 0.01


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    ctype, ttype = _dtypes(case)
    if case["kind"] == "net":
        ops, shape = _ops(case), _in_shape(case)
        weights, biases = [], []
        for op in ops:
            if op.kind not in ("conv", "dwconv", "fc"):
                weights.append(None)
                biases.append(None)
                continue
            kh, kw = (1, 1) if op.kind == "fc" else (op.kh or op.k, op.kw or op.k)
            w = _weights(gen, op.cout, 1 if op.kind == "dwconv" else op.cin, kh, kw, op.sparsity)
            weights.append(wl.embed_filter(w, op.k) if op.kh or op.kw else w)
            biases.append(_bias(gen, op.cout).cpu().numpy())
        net = cad.build_net(ops, weights, biases, shape, ctype)
        if "saved" in case:
            with open(os.path.join(os.path.dirname(cad.__file__), "tuned", case["saved"])) as f:
                net.set_variants(json.load(f)["variants"])
        x = torch.randn(shape, device="cuda", generator=gen)
        if case["family"] == "bottleneck":
            x.relu_()
        return {"case": case, "net": net, "x": x.to(ttype)}

    n = case["n"]
    if case["kind"] == "fc":
        h = cad.cadnn_pack_weights(_weights(gen, case["cout"], case["cin"], 1, 1, case["sparsity"]), ctype)
        cad.cadnn_fc_prepare(h)
        x = torch.randn(n, case["cin"], device="cuda", generator=gen).relu_().to(ttype)
        return {"case": case, "w": h, "x": x, "bias": _bias(gen, case["cout"])}

    channels = case["cin"] if "cin" in case else case["channels"]
    x = torch.randn(n, channels, case["h"], case["w"], device="cuda", generator=gen).relu_().to(ttype)
    state = {"case": case, "x": x}
    if case["kind"] == "depthwise":
        state["w"] = cad.cadnn_pack_weights(_weights(gen, channels, 1, case["k"], case["k"], 0.0), ctype)
        cad.cadnn_depthwise_prepare(state["w"])
        state["bias"] = _bias(gen, channels)
    elif case["kind"] in ("conv", "dense"):
        k, cout = case["k"], case["cout"]
        state["bias"] = _bias(gen, cout)
        state["residual"] = None
        if case["residual"]:
            ho, wo = (wl.conv_out_size(s, k, case["stride"], case["pad"]) for s in (case["h"], case["w"]))
            state["residual"] = torch.randn(n, cout, ho, wo, device="cuda", generator=gen).to(ttype)
        if case["kind"] == "dense":
            state["w"] = _weights(gen, cout, channels, k, k, 0.0, device_tensor=True).to(ttype)
        else:
            state["w"] = cad.cadnn_pack_weights(_weights(gen, cout, channels, k, k, case["sparsity"]), ctype)
            cad.cadnn_conv2d_prepare(state["w"], n, case["h"], case["w"], case["stride"], case["pad"])
    return state


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "net":
        return state["net"].run(state["x"])
    if kind == "conv":
        return cad.cadnn_sparse_conv2d(state["w"], state["x"], case["stride"], case["pad"], state["bias"],
                                       state["residual"], True)
    if kind == "dense":
        return cad.cadnn_dense_conv2d(state["w"], state["x"], case["stride"], case["pad"], state["bias"],
                                      state["residual"], True)
    if kind == "fc":
        return cad.cadnn_sparse_fc(state["w"], state["x"], state["bias"], True)
    if kind == "depthwise":
        return cad.cadnn_depthwise_conv2d(state["w"], state["x"], case["stride"], case["pad"], state["bias"], True)
    if case["op"] == "global":
        return cad.cadnn_global_avgpool(state["x"])
    pool = cad.cadnn_maxpool2d if case["op"] == "max" else cad.cadnn_avgpool2d
    return pool(state["x"], case["k"], case["stride"], case["pad"])


# ---- what a pass cannot do without -------------------------------------------------------

def work(case):
    """Multiply-adds over the nonzero weights (all weights of an unpruned layer), and the bytes of
    the input, the output and the weights (a nonzero counts as its value and a 16-bit index).  The
    tensors between the layers of a net are not counted: a fused pass need not move them."""
    elem = 2 if case["dtype"] == "f16" else 4
    if case["kind"] == "net":
        ops, shape = _ops(case), _in_shape(case)
        cur = {0: shape}
        flops, nbytes = 0.0, float(np.prod(shape)) * elem
        out = shape
        for op in ops:
            n, c, h, w = cur[op.src]
            if op.kind == "concat":
                out = (n, sum(cur[b][1] for b in op.srcs), h, w)
            elif op.kind == "avgpool":
                out = (n, c, 1, 1)
            elif op.kind == "fc":
                out = (n, op.cout, 1, 1)
            else:
                out = (n, op.cout if op.kind == "conv" else c, wl.conv_out_size(h, op.k, op.stride, op.pad),
                       wl.conv_out_size(w, op.k, op.stride, op.pad))
            if op.kind in ("conv", "dwconv", "fc"):
                fan_in = op.cin if op.kind == "fc" else (1 if op.kind == "dwconv" else op.cin) * (op.kh or op.k) * (op.kw or op.k)
                kept = op.cout * fan_in * (1.0 - op.sparsity)
                flops += 2.0 * kept * n * out[2] * out[3]
                nbytes += kept * (elem + (2 if op.sparsity > 0.0 else 0)) + 4.0 * op.cout
            cur[op.dst] = out
        return {"bytes": nbytes + float(np.prod(out)) * elem, "flops": flops}
    n = case["n"]
    if case["kind"] == "fc":
        kept = case["cin"] * case["cout"] * (1.0 - case["sparsity"])
        return {"bytes": kept * (elem + 2) + n * (case["cin"] + case["cout"]) * elem + 4.0 * case["cout"], "flops": 2.0 * kept * n}
    channels = case["cin"] if "cin" in case else case["channels"]
    x = float(n * channels * case["h"] * case["w"])
    if case["kind"] == "pool" and case["op"] == "global":
        return {"bytes": (x + n * channels) * elem, "flops": x}
    k = case["k"]
    pixels = float(n * wl.conv_out_size(case["h"], k, case["stride"], case["pad"]) *
                   wl.conv_out_size(case["w"], k, case["stride"], case["pad"]))
    if case["kind"] == "pool":
        return {"bytes": (x + channels * pixels) * elem, "flops": channels * pixels * k * k}
    if case["kind"] == "depthwise":
        return {"bytes": (x + channels * pixels) * elem + channels * (k * k * elem + 4.0), "flops": 2.0 * channels * pixels * k * k}
    kept = case["cout"] * channels * k * k * (1.0 - case.get("sparsity", 0.0))
    maps = x + case["cout"] * pixels * (2 if case["residual"] else 1)
    return {"bytes": maps * elem + kept * (elem + (2 if case["kind"] == "conv" else 0)) + 4.0 * case["cout"],
            "flops": 2.0 * kept * pixels}


def tolerance(case):
    # Sums are taken in 32 bits.  Against an evaluation in 64 bits the relative error measures, in
    # fp32 storage, 1.1e-7 (pruned 3x3 layer) to 2.1e-7 (the strided one, 518 terms a sum) and 6e-8 to
    # 1.5e-7 for whole networks; it grows with the square root of the terms, up to 4608 of them in
    # an unpruned layer of the range, about 5e-7.  In fp16 storage, one rounding per tensor, it
    # measures 2.1e-4 for a layer and 3.0e-4 to 4.4e-4 for whole networks.  Four times that is stated.
    if case["kind"] == "pool" and case["op"] == "max":
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 2e-6}
    return {"rel": 2e-3}
