"""The calls this library is timed with: Tucker-2 layers, the dense layer beside them, and whole residual networks.

The sizes are those of workloads.py, of the benchmark and of the two networks in bottleneck.py, with one ragged layer;
``draw`` spreads over the same ranges.  Three kinds of case:

* ``tucker``: one Tucker-2 convolution layer with packed weights (TuckerConv2d);
* ``dense``: the undecomposed layer, the t2 of the rank selection's threshold test (DenseConv2d);
* ``resnet18`` / ``resnet50``: the residual stages of the networks, every 3x3 convolution in Tucker-2 form.

``call`` says how the user's program makes the call: ``bound`` through the zero-argument launcher on fixed buffers (a
serving loop), ``fresh`` as layer(x) with a new output tensor per call, ``eager`` / ``graph`` for the networks.
"""
from __future__ import annotations

import math

import torch

from paper_2211_03715_amd import binding as B
from paper_2211_03715_amd import roofline
from paper_2211_03715_amd.bottleneck import TuckerResNet18Body, TuckerResNetBody
from paper_2211_03715_amd.layer import DenseConv2d, TuckerConv2d
from paper_2211_03715_amd.workloads import Layer


def _layer_case(kind, batch, C, N, H, W, R1, R2, K=3, stride=1, layout="nchw", epilogue="none", call="bound"):
    return {"kind": kind, "batch": batch, "C": C, "N": N, "H": H, "W": W, "R1": R1, "R2": R2, "K": K, "stride": stride,
            "pad": K // 2, "layout": layout, "epilogue": epilogue, "call": call}


def _network_case(kind, batch, layout, call):
    return {"kind": kind, "batch": batch, "layout": layout, "call": call}


def listed():
    cases = {
        # One batch-1 layer of the headline sweep in a serving loop, as the second layer of its basic block: the smallest
        # call, all launch and latency.
        "tucker_b1_56": _layer_case("tucker", 1, 64, 64, 56, 56, 16, 16, epilogue="bias_residual_relu"),
        # The other end of that sweep (few pixels, many channels) called the torch way, with folded batch-norm and ReLU.
        "tucker_b1_7_nhwc": _layer_case("tucker", 1, 512, 512, 7, 7, 128, 128, layout="nhwc", epilogue="bias_relu", call="fresh"),
        # Nothing divides anything: odd image, channel counts and ranks that fill no block, 5x5 taps.
        "tucker_b3_ragged": _layer_case("tucker", 3, 100, 150, 37, 29, 24, 40, K=5, epilogue="bias_relu", call="fresh"),
        # A small batch of the down-sampling layer between two stages.
        "tucker_b8_56_s2": _layer_case("tucker", 8, 128, 256, 56, 56, 32, 64, stride=2, epilogue="bias_relu"),
        # Ordinary batches: the down-sampling layer, and the second layer of a 14x14 basic block with its shortcut.
        "tucker_b32_56_s2": _layer_case("tucker", 32, 128, 256, 56, 56, 32, 64, stride=2),
        "tucker_b32_14_nhwc": _layer_case("tucker", 32, 256, 256, 14, 14, 64, 64, layout="nhwc", epilogue="bias_residual_relu"),
        # The largest batch of the throughput set.
        "tucker_b256_28": _layer_case("tucker", 256, 128, 128, 28, 28, 32, 32),
        # One large image: the first layers of a VGG-16-shaped network.
        "tucker_b1_224": _layer_case("tucker", 1, 64, 64, 224, 224, 64, 32, epilogue="bias_relu"),
        # The original convolution that the latency table of the rank selection needs beside the Tucker layer.
        "dense_b8_28": _layer_case("dense", 8, 128, 128, 28, 28, 32, 32),
        # Whole networks: one image at a time eagerly, one image at a time from a HIP graph, and a batch.
        "resnet18_b1": _network_case("resnet18", 1, "nchw", "eager"),
        "resnet50_b1_nhwc_graph": _network_case("resnet50", 1, "nhwc", "graph"),
        "resnet50_b32_nhwc": _network_case("resnet50", 32, "nhwc", "eager"),
    }
    return [dict(case, name=name) for name, case in cases.items()]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(("tucker", "dense", "resnet18", "resnet50"), (14, 3, 2, 1))[0]
    layout = rng.choice(("nchw", "nhwc"))
    if kind.startswith("resnet"):
        return _network_case(kind, _log_int(rng, 1, 32 if kind == "resnet18" else 16), layout, rng.choice(("eager", "graph")))
    while True:
        K, stride = rng.choice((1, 3, 3, 3, 3, 5)), rng.choice((1, 1, 1, 2))
        C, N = _log_int(rng, 24, 512), _log_int(rng, 24, 512)
        multiple = 4 if layout == "nhwc" else rng.choice((1, 16))
        C, N = max(1, C // multiple) * multiple, max(1, N // multiple) * multiple
        R1, R2 = (max(4, int(round(n * rng.uniform(0.125, 0.5)))) for n in (C, N))
        H = _log_int(rng, 7, 224)
        W = H if rng.random() < 0.7 else max(7, min(224, int(H * rng.uniform(0.6, 1.6))))
        case = _layer_case(kind, _log_int(rng, 1, 256), C, N, H, W, R1, R2, K, stride, layout,
                           rng.choice(("none", "bias_relu", "bias_residual_relu")), rng.choice(("bound", "fresh")))
        w = work(case)
        if w["bytes"] <= 220e6 and w["flops"] <= 12e9:    # the largest batched layers listed; far below resnet50_b32
            return case


def _layer(case):
    return Layer(*(case[k] for k in ("batch", "C", "N", "H", "W", "R1", "R2", "K", "stride", "pad")))


def _network(case, seed):
    body = TuckerResNetBody if case["kind"] == "resnet50" else TuckerResNet18Body
    return body(case["batch"], seed=seed, layout=B.LAYOUT_NHWC if case["layout"] == "nhwc" else B.LAYOUT_NCHW)


def prepare(case, seed):
    device = torch.device("cuda", 0)
    gen = torch.Generator(device=device).manual_seed(int(seed))

    def normal(shape, scale=1.0):
        return torch.randn(shape, device=device, generator=gen) * scale

    if case["kind"].startswith("resnet"):
        net = _network(case, 1000 * int(seed))
        x = torch.relu(normal(net.in_shape))              # the stem ends in a ReLU
        state = {"net": net, "x": x, "y": net.y}
        if case["call"] == "graph":
            state["graph"] = net.capture(x)
        else:
            net(x)                                        # a network binds its calls to its input buffer once
        return state
    L = _layer(case)
    nhwc = case["layout"] == "nhwc"
    make = TuckerConv2d if case["kind"] == "tucker" else DenseConv2d
    conv = make(L, layout=B.LAYOUT_NHWC if nhwc else B.LAYOUT_NCHW)
    x = normal((L.batch, L.H, L.W, L.C) if nhwc else (L.batch, L.C, L.H, L.W))
    if case["kind"] == "tucker":
        weights = (normal((L.C, L.R1), L.C ** -0.5), normal((L.R1, L.R2, L.K, L.K), (L.R1 * L.K * L.K) ** -0.5),
                   normal((L.R2, L.N), L.R2 ** -0.5))
    else:
        weights = (normal((L.C, L.N, L.K, L.K), (L.C * L.K * L.K) ** -0.5),)
    conv.pack(*weights)
    epilogue = {}
    if case["epilogue"] != "none":
        epilogue = {"bias": normal((L.N,), 0.1), "relu": True}
    if case["epilogue"] == "bias_residual_relu":
        epilogue["residual"] = normal(conv.out_shape())
    state = {"conv": conv, "x": x, "weights": weights, "epilogue": epilogue}
    if case["call"] == "bound":
        state["y"] = torch.empty(conv.out_shape(), device=device)
        state["launch"] = conv.bind(x, state["y"], **epilogue)
    return state


def run(state):
    if "launch" in state:
        state["launch"]()
        return state["y"]
    if "graph" in state:
        state["graph"].replay()
        return state["y"]
    if "net" in state:
        return state["net"](state["x"])
    return state["conv"](state["x"], **state["epilogue"])


def _layer_work(kind, L, bias, residual):
    """Compulsory bytes and FLOPs of one layer: the factored form for a Tucker layer."""
    y = L.batch * L.N * L.Ho * L.Wo
    extra = 4 * ((L.N if bias else 0) + (y if residual else 0))
    if kind == "tucker":
        return roofline.bytes_compulsory(L) + extra, roofline.flops(L)
    return 4 * (L.batch * L.C * L.H * L.W + y + L.C * L.N * L.K * L.K) + extra, roofline.dense_flops(L)


def _network_layers(case):
    """(kind, layer) of every convolution of the network, with the shortcut operand its epilogue reads."""
    deep, batch, out = case["kind"] == "resnet50", case["batch"], []
    C, h = 64, 56
    for stage, count in enumerate((3, 4, 6, 3) if deep else (2, 2, 2, 2)):
        M = 64 << stage
        rank = (lambda n: max(8, int(round(0.3 * n / 8.0)) * 8)) if deep else (lambda n: n // 4)
        for i in range(count):
            s, C_out = 2 if i == 0 and stage else 1, 4 * M if deep else M
            if deep:
                out.append(("dense", Layer(batch, C, M, h, h, 1, 1, 1, 1, 0)))
                out.append(("tucker", Layer(batch, M, M, h, h, rank(M), rank(M), 3, s, 1)))
                out.append(("dense", Layer(batch, M, C_out, h // s, h // s, 1, 1, 1, 1, 0)))
            else:
                out.append(("tucker", Layer(batch, C, M, h, h, rank(C), rank(M), 3, s, 1)))
                out.append(("tucker", Layer(batch, M, M, h // s, h // s, rank(M), rank(M), 3, 1, 1)))
            if s != 1 or C_out != C:
                out.append(("dense", Layer(batch, C, C_out, h, h, 1, 1, 1, s, 0)))
            C, h = C_out, h // s
    return out


def work(case):
    if not case["kind"].startswith("resnet"):
        nbytes, flops = _layer_work(case["kind"], _layer(case), case["epilogue"] != "none", case["epilogue"] == "bias_residual_relu")
        return {"bytes": nbytes, "flops": flops}
    # A network cannot do without its weights, its input and its output: intermediates are not counted.
    layers = _network_layers(case)
    first, last = layers[0][1], [L for _, L in layers][-1]
    weights = sum((L.C * L.R1 + L.R1 * L.R2 * L.K * L.K + L.R2 * L.N if kind == "tucker" else L.C * L.N * L.K * L.K) + L.N for kind, L in layers)
    flops = sum(roofline.flops(L) if kind == "tucker" else roofline.dense_flops(L) for kind, L in layers)
    return {"bytes": 4 * (weights + case["batch"] * (first.C * first.H * first.W + last.N * last.Ho * last.Wo)), "flops": flops}


def tolerance(case):
    # fp32 inputs and sums.  Against the same path in 64 bits the listed cases and thirty drawn ones are off by 1.2e-7 to
    # 9.7e-7 (the networks, up to 53 convolutions deep: 4.9e-7 to 7.2e-7) and, at the worst single output, by 0.7e-6 to
    # 7.1e-6 of the larger of its value and the rms: about four times the largest of each.
    return {"rel": 4e-6, "max": 3e-5}
