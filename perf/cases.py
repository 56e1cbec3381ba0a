"""The work whose speed is measured: forward passes of fused + pruned residual
networks, and single fused convolutions, through the public entry points.

A case is a dict of plain values:

    net      "block" (one basic block), "cifar" (3 x 3 stem, three stages), "basic" (ImageNet
             stem, four stages of basic blocks), "bottleneck" (the same of 1x1-3x3-1x1 blocks),
             "conv" (one convolution operator)
    depth    layers of the network: 20 / 32 / 56, 18 / 34, 50
    dtype    "f32", "bf16", "f16"
    batch    images of one pass
    size     rows and columns of an image
    permille pruning rate of the filters inside a block
    rates    0, or the seed of one rate per convolution, uniform in 100 .. 700 permille
    out      pruning rate of a block's output filters (0: kept)
    fuse     0, or how many stages are aggressively fused and pruned back (the fusion option x/n)
    graph    True: replayed from a captured graph, False: enqueued operator by operator

A "conv" case has batch, rows, cols, filters, channels, window, stride, add (a shortcut is added)
and dtype instead.
"""
import math

import numpy as np
import torch

import synth
from paper_2010_16165_amd import binding as B
from paper_2010_16165_amd import network

_STAGES = {18: (2, 2, 2, 2), 34: (3, 4, 6, 3), 50: (3, 4, 6, 3)}
# 2 x multiply-adds of the unpruned network for one image of 224 x 224 (32 x 32: CIFAR)
_FLOPS = {20: 0.082e9, 32: 0.138e9, 56: 0.25e9, 18: 3.6e9, 34: 7.3e9, 50: 8.2e9}
# no drawn pass multiplies more than the largest listed one
_MOST_FLOPS = 1.15e12


def _net(name, net, depth, dtype, batch, size, permille=300, rates=0, out=0, fuse=0, graph=True):
    return {"name": name, "net": net, "depth": depth, "dtype": dtype, "batch": batch, "size": size,
            "permille": permille, "rates": rates, "out": out, "fuse": fuse, "graph": graph}


def listed():
    return [
        # one CIFAR basic block in single precision, one image: the smallest call there is
        _net("block_f32_b1", "block", 0, "f32", 1, 32, permille=250, graph=False),
        # the latency of a small network on one image, as a device that sees one image at a time runs it
        _net("resnet20_bf16_b1", "cifar", 20, "bf16", 1, 32),
        # single precision for a whole network: the numbers that a 16-bit deployment is checked against
        _net("resnet20_f32_b32", "cifar", 20, "f32", 32, 32, graph=False),
        # CIFAR-size throughput
        _net("resnet56_bf16_b128", "cifar", 56, "bf16", 128, 32, permille=400),
        # one operator by itself, ragged channels and extent, with a shortcut: a caller with an
        # executor of its own
        {"name": "conv3x3_bf16_57x38", "net": "conv", "dtype": "bf16", "batch": 6, "rows": 57, "cols": 38,
         "filters": 102, "channels": 77, "window": 3, "stride": 1, "add": True},
        # ImageNet-size latency on one image
        _net("resnet18_bf16_b1", "basic", 18, "bf16", 1, 224),
        # ordinary ImageNet throughput, basic blocks
        _net("resnet18_bf16_b64", "basic", 18, "bf16", 64, 224),
        # every non-fused operator pruned, output filters of the blocks among them
        _net("resnet34_bf16_b20_out", "basic", 34, "bf16", 20, 224, out=300, graph=False),
        # the fusion option 2/4: two stages without additions, pruned back
        _net("resnet18_f16_b12_fused", "basic", 18, "f16", 12, 224, fuse=2),
        # ordinary ImageNet throughput, bottleneck blocks
        _net("resnet50_bf16_b64", "bottleneck", 50, "bf16", 64, 224, permille=500),
        # an odd extent, an odd batch and irregular channel counts, without a graph
        _net("resnet50_f16_b9_193", "bottleneck", 50, "f16", 9, 193, rates=7, graph=False),
        # the largest: irregular channel counts at a large batch
        _net("resnet50_f16_b256", "bottleneck", 50, "f16", 256, 224, rates=201016169),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    net = rng.choice(["block", "cifar", "cifar", "basic", "basic", "basic", "bottleneck", "bottleneck",
                      "bottleneck", "conv", "conv"])
    dtype = rng.choice(["bf16", "bf16", "f16"])
    graph = rng.random() < 0.5
    if net == "conv":
        stride = rng.choice([1, 1, 2])
        c = {"net": "conv", "dtype": dtype, "batch": _log(rng, 1, 64), "rows": _log(rng, 7, 80),
             "cols": _log(rng, 7, 80), "filters": _log(rng, 10, 512), "channels": _log(rng, 10, 512),
             "window": rng.choice([1, 3, 3]), "stride": stride, "add": stride == 1 and rng.random() < 0.5}
        return c
    if net == "block":
        c = _net("", "block", 0, rng.choice(["f32", dtype]), _log(rng, 1, 128), rng.randint(14, 32),
                 permille=rng.randint(100, 500), graph=graph)
    elif net == "cifar":
        dtype = rng.choice(["f32", dtype, dtype])
        # (56 layers of random weights grow past the largest f16)
        c = _net("", "cifar", rng.choice([20, 32] if dtype == "f16" else [20, 32, 56]), dtype, _log(rng, 1, 64 if dtype == "f32" else 512), 32,
                 permille=rng.choice([0, 100, 200, 300, 400]), graph=graph)
    else:
        depth = 50 if net == "bottleneck" else rng.choice([18, 18, 34])
        size = rng.choice([224, 224, rng.randint(96, 224)])
        most = min(256, int(_MOST_FLOPS / (_FLOPS[depth] * (size / 224) ** 2)))
        irregular = net == "bottleneck" and rng.random() < 0.5
        option = rng.random() if net == "basic" else 1.0
        c = _net("", net, depth, dtype, _log(rng, 1, most), size, permille=rng.choice([100, 200, 300, 400, 500]),
                 rates=rng.randint(1, 10 ** 6) if irregular else 0, out=300 if option < 0.15 else 0,
                 fuse=rng.randint(1, 4) if option > 0.85 and net == "basic" else 0, graph=graph)
    del c["name"]
    return c


def _description(case, seed):
    """The pre-trained network the case prunes and fuses (synth's plain-data format)."""
    net, size, pm, out = case["net"], case["size"], case["permille"], case["out"]
    if net == "block":
        return synth.make_block_model(seed, case["dtype"], 16, size, pm, out)
    if net == "cifar":
        return synth.make_cifar_resnet(seed, case["dtype"], (case["depth"] - 2) // 6, pm, size=size,
                                       out_permille=out)
    make = synth.make_imagenet_basic_resnet if net == "basic" else synth.make_imagenet_bottleneck_resnet
    m = make(seed, case["dtype"], _STAGES[case["depth"]], pm, size=size, out_permille=out)
    if case["rates"]:   # the rates belong to the case, not to the seed: they are sizes
        rng = np.random.default_rng([case["rates"], 2])
        for blk in m["blocks"]:
            pms = [int(np.floor(rng.uniform(100, 700))) for _ in range(2)]
            blk["prune_permille"] = pms + blk["prune_permille"][2:]
    return m


def _optimised(case, seed):
    return network.optimise(_description(case, seed), aggressive=case["fuse"] > 0,
                            fuse_stages=case["fuse"] or None)


def _activations(n, h, w, c, dt, gen, relu):
    t = B.DeviceTensor.empty(n, h, w, c, dt)
    t.data.zero_()
    x = torch.randn((n, h, w, c), generator=gen, device="cuda")
    t.data[..., :c] = torch.relu(x) if relu else x
    return t


def _conv_extent(case):
    p = case["window"] // 2
    return [(e + 2 * p - case["window"]) // case["stride"] + 1 for e in (case["rows"], case["cols"])]


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dt, n = B.DTYPES[case["dtype"]], case["batch"]
    if case["net"] == "conv":
        k, c, r = case["filters"], case["channels"], case["window"]
        rng = np.random.default_rng(seed)
        w = (rng.standard_normal((k, c, r, r), dtype=np.float32) * np.float32(math.sqrt(2.0 / (c * r * r))))
        shape = B.shape_of(w, case["stride"], r // 2)
        packed = B.upload_blob(B.fupr_pack(shape, w, rng.standard_normal(k, dtype=np.float32) * np.float32(0.1), dt))
        p, q = _conv_extent(case)
        x = _activations(n, case["rows"], case["cols"], c, dt, gen, relu=True)
        res = (_activations(n, p, q, k, dt, gen, relu=True), 1, 0) if case["add"] else None
        return {"shape": shape, "x": x, "packed": packed, "res": res,
                "flags": B.FUSE_RELU | (B.FUSE_ADD if res else 0), "y": B.DeviceTensor.empty(n, p, q, k, dt)}
    model, _ = network.build(_optimised(case, seed))
    c, h, w = model.in_shape
    # a block's input is another block's output
    x = _activations(n, h, w, c, dt, gen, relu=case["net"] == "block")
    out, ws = model.alloc(n)
    state = {"model": model, "x": x, "y": out, "ws": ws, "graph": None}
    if case["graph"]:
        stream = torch.cuda.Stream()
        torch.cuda.synchronize()
        state["graph"] = model.fupr_graph_create(x, out, ws, B.C.c_void_p(stream.cuda_stream))
        state["stream"] = stream
    return state


def run(state):
    if "shape" in state:
        B.fupr_conv_fused(state["shape"], state["x"], state["packed"], state["res"], state["flags"], state["y"])
    elif state["graph"] is not None:
        state["model"].fupr_graph_launch(state["graph"], B.current_stream())
    else:
        state["model"].fupr_forward(state["x"], state["y"], state["ws"])
    return state["y"].data


def work(case):
    """Multiply-adds at the pruned filter counts; the images and every parameter read
    once, the result written once (a network's intermediate tensors are not counted)."""
    esize, n = (4 if case["dtype"] == "f32" else 2), case["batch"]
    if case["net"] == "conv":
        k, c, r = case["filters"], case["channels"], case["window"]
        p, q = _conv_extent(case)
        pixels = n * case["rows"] * case["cols"] * c + n * p * q * k * (2 if case["add"] else 1)
        return {"flops": 2.0 * n * p * q * k * c * r * r, "bytes": esize * float(pixels + k * c * r * r) + 4.0 * k}
    plan = _optimised(case, 1)
    model, _ = network.build(plan, base_address=1 << 20)   # sizes only: this model cannot run
    flops = sum(model.op_stats(n, i)["flops"] for i in range(model.num_ops))
    params = sum(esize * L.W.size + 4 * L.bias.size for L in plan["layers"])
    c, h, w = plan["in_shape"]
    y = model.output_shape(n)
    return {"flops": flops, "bytes": float(params + esize * n * (c * h * w + y.H * y.W * y.C))}


def tolerance(case):
    """About four times what the same pass with its sums in another order (another kernel
    family, another schedule) was seen to differ by: 2-norm and largest difference.  In a
    network a rounding that falls the other way is carried on (bf16: 3.5e-3 and 1.5e-2, f16:
    3.6e-4 and 1.3e-3); in one operator single roundings differ (1.7e-5, and half a unit in the
    last place of bf16, 5.7e-3)."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-4}
    if case["net"] == "conv":
        return {"rel": 2e-4, "max": 2e-2}
    return {"rel": 1.4e-2, "max": 6e-2} if case["dtype"] == "bf16" else {"rel": 1.5e-3, "max": 6e-3}
