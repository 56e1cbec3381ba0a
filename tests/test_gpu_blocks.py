"""GPU tests of the launches that hold a whole block: against a plain float64
evaluation that rounds where tensors are stored, and against one kernel per operator."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fx():
    import torch
    from paper_2010_16165_amd import binding as B
    assert torch.cuda.is_available()
    return B, torch


class Net:
    """Operators with seeded weights, their float64 evaluation, and a model of them."""

    def __init__(self, fx, dtype, n, in_shape, seed):
        self.B, self.torch = fx
        self.dtype, self.dt, self.n, self.in_shape = dtype, self.B.DTYPES[dtype], n, in_shape
        self.rng = np.random.default_rng(seed)
        c, h, w = in_shape
        x = np.maximum(self.rng.standard_normal((n, c, h, w)), 0).astype(np.float32)
        self.x, self.ops, self.blobs = x, [], []
        self.tensors = [self.stored(self.torch.from_numpy(x).double())]

    def stored(self, v):
        t = {"bf16": self.torch.bfloat16, "f16": self.torch.float16, "f32": self.torch.float32}[self.dtype]
        return v.to(t).double()

    def conv(self, tin, k, r, stride=1, add=-1, cat=-1, cat_stride=1, relu=True, add_stride=1, add_at=0):
        B, torch = self.B, self.torch
        a = self.tensors[tin]
        c = a.shape[1]
        if cat >= 0:
            # the channels between the two tensors are zeros of the first, with zero weights
            split = (c + B.CAT_ALIGN - 1) // B.CAT_ALIGN * B.CAT_ALIGN
            b = self.tensors[cat][:, :, ::cat_stride, ::cat_stride][:, :, :a.shape[2], :a.shape[3]]
            a = torch.cat([torch.nn.functional.pad(a, (0, 0, 0, 0, 0, split - c)), b], 1)
        w = (self.rng.standard_normal((k, a.shape[1], r, r)) * np.sqrt(2.0 / (a.shape[1] * r * r))).astype(np.float32)
        if cat >= 0:
            w[:, c:split] = 0.0
        bias = (self.rng.standard_normal(k) * 0.1).astype(np.float32)
        shape = B.shape_of(w, stride, r // 2)
        self.blobs.append(B.upload_blob(B.fupr_pack(shape, w, bias, self.dt)))
        v = torch.nn.functional.conv2d(a, self.stored(torch.from_numpy(w).double()),
                                       torch.from_numpy(bias).double(), stride, r // 2)
        if add >= 0:
            r = self.tensors[add][:, :, ::add_stride, ::add_stride][:, :, :v.shape[2], :v.shape[3]]
            v[:, add_at:add_at + r.shape[1]] += r
        self.tensors.append(self.stored(torch.relu(v) if relu else v))
        flags = (B.FUSE_RELU if relu else 0) | (B.FUSE_ADD if add >= 0 else 0) | (B.FUSE_CAT if cat >= 0 else 0)
        self.ops.append(B.OpDesc(B.OP_CONV, tin, add, shape, self.blobs[-1].data_ptr(), flags, add_stride, add_at, None,
                                 cat, cat_stride if cat >= 0 else 0))
        return len(self.ops)

    def check(self, tile_switch, tile, expect, takes=True):
        """The forced tile runs as one launch of `expect` if it takes the shape; the network's output
        against both references."""
        B, torch = self.B, self.torch
        m = B.Model(self.dt, self.in_shape, self.ops, self.blobs)
        assert B._lib.fupr_model_set_table(m._h, None) in (B.FUPR_OK, B.ERR_ARG)   # no one-kernel schedule
        m.fuse_blocks(True)
        B.fupr_tuning_set(tile_switch, tile)
        try:
            kernels = [m.launch_stats(self.n, i)["kernel"] for i in range(m.num_launches_at(self.n))]
            assert sum(k.startswith(expect) for k in kernels) == takes, kernels
            print(self.dtype, self.n, self.in_shape, kernels, flush=True)
            xd = B.DeviceTensor.from_nchw(self.x, self.dt)
            out, ws = m.alloc(self.n)
            ws.fill_(255)              # NaN wherever nothing is written
            out.data.fill_(7.0)
            m.fupr_forward(xd, out, ws)
            torch.cuda.synchronize()
            got = torch.from_numpy(np.ascontiguousarray(out.to_nchw())).double()
            assert out.padding_is_zero()
            again, ws2 = m.alloc(self.n)
            ws2.fill_(255)
            m.fupr_forward(xd, again, ws2)
            m.set_schedule(B.SCHEDULE_PER_LAYER)
            apart, _ = m.alloc(self.n)
            m.fupr_forward(xd, apart, ws)
            torch.cuda.synchronize()
            assert torch.equal(out.data, again.data)
        finally:
            B.fupr_tuning_set(tile_switch, None)
        # A stored value may round the other way after sums in another order.  Were every rounding of the
        # two evaluations independent (2^-8 or 2^-11 of the value at most, 0.29 of that in the mean
        # square), the nine stored tensors of a chain would add up to sqrt(2 * 9) * 0.29 = 1.2 units.
        unit = {"bf16": 2.0 ** -8, "f16": 2.0 ** -11, "f32": 2.0 ** -20}[self.dtype]
        want = self.tensors[-1]
        other = torch.from_numpy(np.ascontiguousarray(apart.to_nchw())).double()
        for ref in (want, other):
            assert float((got - ref).norm() / ref.norm()) <= 1.5 * unit
            assert float((got - ref).abs().max()) <= 4 * unit * float(ref.abs().max())


# dtype, images, rows, columns, channels in, 3 x 3 filters, its stride, wide filters, next filters (0: none),
# how the block's input comes back: added, concatenated, or not at all
BOTTLENECKS = [
    ("bf16", 2, 9, 11, 24, 32, 1, 128, 32, "add"),        # less than a group of filters, one pair of tiles
    ("f16", 1, 1, 1, 8, 16, 1, 16, 16, "none"),           # smallest there is: one pixel, one tile of filters
    ("bf16", 3, 7, 7, 77, 45, 1, 300, 51, "add"),         # ragged channels everywhere, tiles across images
    ("f16", 1, 15, 13, 40, 102, 2, 264, 130, "cat"),      # stride 2, two tensors, last group nearly empty
    ("bf16", 2, 14, 14, 128, 128, 1, 512, 100, "cat"),
    ("f16", 2, 5, 40, 96, 144, 1, 272, 240, "add"),       # more than 128 filters in the 3 x 3
    ("bf16", 1, 8, 8, 64, 64, 1, 256, 0, "add"),          # nothing behind the block
    ("f16", 2, 6, 6, 136, 240, 2, 320, 300, "cat"),
]


TILES = [(1, 8), (2, 8), (4, 8), (2, 4), (4, 4)]      # tiles of 16 pixels, waves


@pytest.mark.parametrize("tile", range(len(TILES)))
@pytest.mark.parametrize("case", BOTTLENECKS, ids=lambda c: "-".join(map(str, c)))
def test_bottleneck_block(fx, case, tile):
    dtype, n, h, w, c, k1, stride, k2, k3, back = case
    wide = k2 if back == "add" else 56
    net = Net(fx, dtype, n, (16, h, w), seed=sum(case[1:9]) + tile)
    # (tensors that live side by side, so that the workspace has buffers for the block's five)
    t = [net.conv(0, 512, 1) for _ in range(4)]
    t_in = net.conv(net.conv(t[0], 512, 1, add=t[1]), 512, 1, add=net.conv(t[2], 512, 1, add=t[3]))
    t_in = net.conv(t_in, wide, 1)            # the block's input
    t_x = net.conv(t_in, c, 1)
    if back == "add" and stride == 1:
        t_mid = net.conv(t_x, k1, 3)
        t_y = net.conv(t_mid, k2, 1, add=t_in)
    elif back == "cat":
        t_mid = net.conv(t_x, k1, 3, stride)
        t_y = net.conv(t_mid, k2, 1, cat=t_in, cat_stride=stride)
    else:
        t_mid = net.conv(t_x, k1, 3, stride)
        t_y = net.conv(t_mid, k2, 1)
    if k3:
        t_h = net.conv(t_y, k3, 1)
        net.conv(t_h, 24, 1, cat=t_y)          # reads both tensors that the launch writes
    else:
        net.conv(t_y, 24, 3)
    # what a wave can hold: 32 filters of the 3 x 3 convolution, eight tiles of the third
    mt, waves = TILES[tile]
    per_wave = -(-(-(-k3 // 16)) // waves)
    net.check("bottleneck_tile", tile, "bottleneck_", k1 <= 32 * waves and mt * (4 if per_wave > 2 else per_wave) <= 8)


RECTANGLES = [(2, 8), (4, 4), (4, 8), (7, 7), (8, 8), (7, 14), (8, 16), (14, 14)]
# dtype, images, rows, columns, channels, first filters, its stride, second filters, shortcut: the block's
# input, its every other pixel in channels from 8 on, another tensor, none
BASIC_BLOCKS = [
    ("f32", 1, 32, 32, 16, 12, 1, 16, "input"),
    ("bf16", 2, 9, 11, 24, 45, 1, 24, "input"),           # ragged channels, rectangles over the edges
    ("f16", 1, 1, 1, 8, 16, 1, 16, "none"),               # one pixel: every tap but one outside
    ("f32", 2, 15, 13, 20, 23, 2, 40, "strided"),         # stride 2, zero-padded shortcut
    ("bf16", 3, 14, 17, 64, 77, 1, 100, "other"),
    ("f16", 1, 30, 28, 16, 130, 2, 48, "strided"),        # second pass over the filters
]


@pytest.mark.parametrize("rectangle", range(len(RECTANGLES)))
@pytest.mark.parametrize("wf", [1, 2, 4, 8])
@pytest.mark.parametrize("case", BASIC_BLOCKS, ids=lambda c: "-".join(map(str, c)))
def test_basic_block(fx, case, rectangle, wf):
    dtype, n, h, w, c, k1, stride, k2, back = case
    net = Net(fx, dtype, n, (16, h, w), seed=sum(case[1:8]) + 8 * rectangle + wf)
    t = [net.conv(0, 128, 1) for _ in range(4)]       # (for the workspace, as above)
    t_x = net.conv(net.conv(t[0], 128, 1, add=t[1]), 128, 1, add=net.conv(t[2], 128, 1, add=t[3]))
    t_x = net.conv(t_x, c, 1)
    t_r = net.conv(t_x, k2, 1) if back == "other" else -1
    t_mid = net.conv(t_x, k1, 3, stride)
    add = {"input": t_x, "strided": t_x, "other": t_r, "none": -1}[back]
    net.conv(net.conv(t_mid, k2, 3, add=add, add_stride=stride, add_at=8 if back == "strided" else 0), 24, 1)
    rows, cols = (-(-e // stride) for e in (h, w))
    th, tw = min(RECTANGLES[rectangle][0], rows), min(RECTANGLES[rectangle][1], cols)
    tiles = [-(-(-(-px // 16)) // (8 // wf)) for px in ((th + 2) * (tw + 2), th * tw)]
    fits = any(tiles[0] <= a and tiles[1] <= b for a, b in [(2, 1), (3, 2), (4, 3), (6, 4), (8, 7), (16, 13)])
    net.check("basic_tile", f"{rectangle}x{wf}", "basic_block_", fits)


# Rows of the rectangle as tiles (the last two rectangles): rectangles over the edges, rows of taps that end within a
# step of the reduction, in one step, on a whole one; two passes over the filters
BY_ROWS = [
    ("bf16", 2, 14, 14, 8, 16, 8, "input"),
    ("f16", 1, 17, 31, 24, 45, 24, "input"),
    ("bf16", 3, 28, 15, 64, 77, 100, "other"),
    ("f16", 1, 30, 28, 37, 130, 48, "none"),
    ("bf16", 1, 15, 14, 128, 64, 128, "input"),
]


@pytest.mark.parametrize("rows", [6, 14])
@pytest.mark.parametrize("wf", [2, 4, 8])
@pytest.mark.parametrize("case", BY_ROWS, ids=lambda c: "-".join(map(str, c)))
def test_basic_block_by_rows(fx, case, wf, rows):
    dtype, n, h, w, c, k1, k2, back = case
    net = Net(fx, dtype, n, (16, h, w), seed=sum(case[1:7]) + wf + rows)
    t = [net.conv(0, 128, 1) for _ in range(4)]       # (for the workspace, as above)
    t_x = net.conv(net.conv(t[0], 128, 1, add=t[1]), 128, 1, add=net.conv(t[2], 128, 1, add=t[3]))
    t_x = net.conv(t_x, c, 1)
    t_r = net.conv(t_x, k2, 1) if back == "other" else -1
    t_mid = net.conv(t_x, k1, 3)
    add = {"input": t_x, "other": t_r, "none": -1}[back]
    net.conv(net.conv(t_mid, k2, 3, add=add), 24, 1)
    net.check("basic_tile", f"{len(RECTANGLES) + (rows == 14)}x{wf}", f"basic_block_{rows}x14r", wf >= 4)


def test_one_pass_sees_one_schedule(fx):
    """A tuning switch that another thread turns while passes are enqueued: each pass has the launches and the
    tensors of one setting or of the other, never of both."""
    import threading
    B, torch = fx
    net = Net(fx, "bf16", 8, (16, 28, 28), seed=5)
    t = net.conv(0, 64, 1)
    for _ in range(3):
        t = net.conv(net.conv(t, 45, 3), 64, 3, add=t)
    net.conv(t, 24, 1)
    m = B.Model(net.dt, net.in_shape, net.ops, net.blobs)
    assert B._lib.fupr_model_set_table(m._h, None) in (B.FUPR_OK, B.ERR_ARG)
    m.fuse_blocks(True)
    xd = B.DeviceTensor.from_nchw(net.x, net.dt)
    out, ws = m.alloc(net.n)

    def one():
        out.data.fill_(7.0)
        m.fupr_forward(xd, out, ws)
        torch.cuda.synchronize()
        return out.data.clone()

    want, launches = [], []
    done = threading.Event()

    def turn():
        while not done.is_set():
            B.fupr_tuning_set("basic_fuse", 0)
            B.fupr_tuning_set("basic_fuse", None)

    try:
        for value in (None, 0):
            B.fupr_tuning_set("basic_fuse", value)
            launches.append(m.num_launches_at(net.n))
            want.append(one())
        assert launches[0] < launches[1]
        thread = threading.Thread(target=turn)
        thread.start()
        try:
            for _ in range(200):
                got = one()
                assert any(torch.equal(got, w) for w in want)
        finally:
            done.set()
            thread.join()
    finally:
        B.fupr_tuning_set("basic_fuse", None)


def block_model(fx, dtype, n, in_shape, k1, k2, add, seed):
    """A model that is one basic block, on the caller's tensors, and its per-layer twin."""
    net = Net(fx, dtype, n, in_shape, seed)
    net.conv(net.conv(0, k1, 3), k2, 3, add=0 if add else -1)
    B = net.B
    models = [B.Model(net.dt, in_shape, net.ops, net.blobs) for _ in range(2)]
    for m in models:
        assert B._lib.fupr_model_set_table(m._h, None) in (B.FUPR_OK, B.ERR_ARG)   # no one-kernel schedule
    models[0].fuse_blocks(True)
    models[1].set_schedule(B.SCHEDULE_PER_LAYER)
    assert models[0].num_launches_at(n) == 1 and models[1].num_launches_at(n) == 2
    return net, models


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("how", ["in place", "in place with the shortcut", "shifted"])
def test_block_whose_output_overlaps_its_input(fx, dtype, how):
    """A launch of the whole block would write pixels that its other workgroups still read: such a call runs as
    two launches, and gives their bits."""
    B, torch = fx
    n, c, h, w = 2, 16, 20, 24
    net, (m, apart) = block_model(fx, dtype, n, (c, h, w), 12, c, how == "in place with the shortcut", 11)
    x = B.DeviceTensor.from_nchw(net.x, net.dt)
    want, ws = apart.alloc(n)
    apart.fupr_forward(x, want, ws)
    elements = n * h * w * c
    base = torch.zeros(2 * elements, dtype=x.data.dtype, device="cuda")
    base[:elements] = x.data.flatten()
    at = 3 * w * c if how == "shifted" else 0
    xin = B.DeviceTensor(base[:elements].view(n, h, w, c), c, net.dt)
    out = B.DeviceTensor(base[at:at + elements].view(n, h, w, c), c, net.dt)
    _, ws2 = m.alloc(n)
    ws2.fill_(255)
    m.fupr_forward(xin, out, ws2)
    torch.cuda.synchronize()
    assert torch.equal(out.data, want.data)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("add", [False, True])
def test_block_on_tensors_with_wider_strides(fx, dtype, add):
    """The caller's strides, on both sides of the block and for its shortcut; what lies between C and the
    stride is zeros."""
    B, torch = fx
    n, c, h, w, k2 = 3, 20, 11, 18, 20
    net, (m, _) = block_model(fx, dtype, n, (c, h, w), 23, k2, add, 12)
    unit = {"bf16": 2.0 ** -8, "f32": 2.0 ** -20}[dtype]
    want = net.tensors[-1]
    # (an output's stride goes up to the packed filters)
    for xcs, ycs in ((24, 20), (40, 20)) if dtype == "f32" else ((24, 24), (40, 24), (24, 32), (48, 32)):
        print(dtype, add, xcs, ycs, flush=True)
        x = B.DeviceTensor.from_nchw(net.x, net.dt, c_stride=xcs)
        out = B.DeviceTensor.empty(n, h, w, k2, net.dt, c_stride=ycs)
        out.data.fill_(7.0)
        _, ws = m.alloc(n)
        ws.fill_(255)
        m.fupr_forward(x, out, ws)
        torch.cuda.synchronize()
        assert out.padding_is_zero()
        got = torch.from_numpy(np.ascontiguousarray(out.to_nchw())).double()
        # two stored tensors, each rounded once in either evaluation
        assert float((got - want).norm() / want.norm()) <= unit
        assert float((got - want).abs().max()) <= 4 * unit * float(want.abs().max())


@pytest.mark.parametrize("rows", [6, 14])
@pytest.mark.parametrize("layer", [0, 1])
def test_infinite_weights_beside_a_padded_step_by_rows(fx, rows, layer):
    """With three chunks to a row of taps the fourth of its step is the next row's first: its weights, infinite
    here, meet zeros that stand for nothing, and must not be multiplied."""
    B, torch = fx
    n, c, h, w = 1, 8, 28, 28
    net = Net(fx, "bf16", n, (c, h, w), 13)
    rng = net.rng
    blobs, ops = [], []
    for i in range(2):
        wt = rng.uniform(0.01, 0.1, (8, 8, 3, 3)).astype(np.float32)
        if i == layer:
            wt[0, 0, 1, 0] = np.inf                      # first chunk of the second row of taps
        shape = B.shape_of(wt, 1, 1)
        blobs.append(B.upload_blob(B.fupr_pack(shape, wt, np.full(8, 0.1, np.float32), net.dt)))
        ops.append(B.OpDesc(B.OP_CONV, i, -1, shape, blobs[-1].data_ptr(), B.FUSE_RELU, 1, 0))
    m = B.Model(net.dt, (c, h, w), ops, blobs)
    assert B._lib.fupr_model_set_table(m._h, None) in (B.FUPR_OK, B.ERR_ARG)
    m.fuse_blocks(True)
    B.fupr_tuning_set("basic_tile", f"{len(RECTANGLES) + (rows == 14)}x4")
    try:
        assert [s["kernel"] for s in [m.launch_stats(n, 0)]] == [f"basic_block_{rows}x14r"]
        x = B.DeviceTensor.from_nchw(np.abs(net.x) + 0.5, net.dt)
        out, ws = m.alloc(n)
        m.fupr_forward(x, out, ws)
        torch.cuda.synchronize()
    finally:
        B.fupr_tuning_set("basic_tile", None)
    y = out.data[..., :8].float()
    inner = y[:, 3:-3, 3:-3]                             # (zeros outside the image times infinity are NaN)
    assert bool(torch.isposinf(inner[..., 0]).all())
    if layer == 1:
        assert bool(torch.isfinite(y[..., 1:]).all())
    else:
        assert bool(torch.isposinf(inner).all())         # every filter reads the infinite channel


def test_sub_batches_of_blocks_by_rows(fx):
    """The order of a block's sums depends on whether its tiles are rows, which the whole batch decides: parts of
    it give the same bits, with the count forced and without."""
    import synth
    from paper_2010_16165_amd import network
    B, torch = fx
    model = synth.make_imagenet_basic_resnet(31, "bf16", (1, 1, 1, 1), 300, widths=(16, 24, 32, 40), size=112, classes=9)
    n = 96
    m, _ = network.build(network.optimise(model))
    kernels = [m.launch_stats(n, i)["kernel"] for i in range(m.num_launches_at(n))]
    assert "basic_block_14x14r" in kernels, kernels
    x = B.DeviceTensor.from_nchw(synth.make_input(31, n, model["in_shape"]), B.BF16)
    whole = None
    try:
        for parts in (1, 2, 3, 4, None):
            print("sub-batches:", parts, flush=True)
            B.fupr_tuning_set("split", parts)
            out, ws = m.alloc(n)
            ws.fill_(255)
            m.fupr_forward(x, out, ws)
            torch.cuda.synchronize()
            whole = out.data.clone() if whole is None else whole
            assert torch.equal(whole, out.data)
    finally:
        B.fupr_tuning_set("split", None)


# images, rows, columns, channels in, filters of the 3 x 3 and of the 1 x 1 convolution
BESIDE = [(1, 14, 14, 64, 90, 128), (2, 15, 9, 45, 20, 33), (3, 7, 7, 136, 200, 72), (1, 1, 1, 8, 16, 80), (5, 13, 37, 24, 40, 264)]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("tap", [None, 0, 2, "window first"])
@pytest.mark.parametrize("tile", ["", "0x2x2", "2x1x4", "4x2x4", "6x4x1", "7x2x2", "10x4x1", "0x1x8"])
@pytest.mark.parametrize("case", BESIDE, ids=lambda c: "-".join(map(str, c)))
def test_projection_beside_the_first_convolution(fx, case, tile, tap, dtype):
    """A block's stride-2 convolution and its projection in one launch, in either order and with each tile of the
    1 x 1 convolution: against both references, and the bits of the two launches."""
    B, torch = fx
    n, h, w, c, k1, k2 = case
    net = Net(fx, dtype, n, (16, h, w), seed=sum(case))
    t_x = net.conv(net.conv(0, 24, 1), c, 1)
    if tap == "window first":
        t_1 = net.conv(t_x, k1, 3, stride=2)
        t_p = net.conv(t_x, k2, 1, stride=2, relu=False)
    else:
        t_p = net.conv(t_x, k2, 1, stride=2, relu=False)
        t_1 = net.conv(t_x, k1, 3, stride=2)
    net.conv(net.conv(t_1, k2, 3, add=t_p), 24, 1)
    B.fupr_tuning_set("basic_fuse", 0)
    try:
        m = B.Model(net.dt, net.in_shape, net.ops, net.blobs)
        assert B._lib.fupr_model_set_table(m._h, None) in (B.FUPR_OK, B.ERR_ARG)
        m.fuse_blocks(True)
        B.fupr_tuning_set("window_tile", tile or None)
        B.fupr_tuning_set("two_tap", tap if tap != "window first" else None)
        x = B.DeviceTensor.from_nchw(net.x, net.dt)
        outs = []
        for two in (None, 0):
            B.fupr_tuning_set("conv_two", two)
            kernels = [m.launch_stats(n, i)["kernel"] for i in range(m.num_launches_at(n))]
            assert ("conv_w+conv1x1p_w" in kernels) == (two is None and tile != "10x4x1"), kernels
            out, ws = m.alloc(n)
            ws.fill_(255)
            m.fupr_forward(x, out, ws)
            torch.cuda.synchronize()
            outs.append(out.data.clone())
        assert torch.equal(*outs)
        B.fupr_tuning_set("conv_two", None)
        net.check("window_tile", tile or None, "conv_w+conv1x1p_w", takes="conv_w+conv1x1p_w" in [
            m.launch_stats(n, i)["kernel"] for i in range(m.num_launches_at(n))])
    finally:
        for switch in ("basic_fuse", "window_tile", "conv_two", "two_tap"):
            B.fupr_tuning_set(switch, None)


def test_sub_batches_of_launches_of_two_operators(fx):
    """Parts of a batch run a projection beside its block's first convolution, and the mean with the layer behind it,
    with the bits of the whole."""
    import synth
    from paper_2010_16165_amd import network
    B, torch = fx
    model = synth.make_imagenet_basic_resnet(17, "bf16", (1, 1, 1, 1), 300, widths=(16, 24, 40, 64), size=64, classes=9)
    n = 27
    m, _ = network.build(network.optimise(model))
    x = B.DeviceTensor.from_nchw(synth.make_input(17, n, model["in_shape"]), B.BF16)
    whole = None
    try:
        B.fupr_tuning_set("basic_fuse", 0)
        kernels = [m.launch_stats(n, i)["kernel"] for i in range(m.num_launches_at(n))]
        assert kernels.count("conv_w+conv1x1p_w") >= 2 and "mean_fc" in kernels, kernels
        for parts in (1, 2, 3):
            print("sub-batches:", parts, flush=True)
            B.fupr_tuning_set("split", parts)
            out, ws = m.alloc(n)
            ws.fill_(255)
            m.fupr_forward(x, out, ws)
            torch.cuda.synchronize()
            whole = out.data.clone() if whole is None else whole
            assert torch.equal(whole, out.data)
    finally:
        for switch in ("basic_fuse", "split"):
            B.fupr_tuning_set(switch, None)


# images, rows, columns, channels, filters: a whole pass of the lanes, one chunk, ragged channels, the largest image
MEAN_FC = [(1, 7, 7, 512, 1000), (32, 1, 1, 8, 10), (3, 3, 5, 45, 65), (2, 16, 8, 256, 129), (5, 8, 9, 333, 16)]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("case", MEAN_FC, ids=lambda c: "-".join(map(str, c)))
def test_mean_and_the_layer_behind_it(fx, case, dtype):
    """The global mean and fc in one launch, and in two with the switch off: against both references
    (Net.check's bound, derived for nine stored tensors; there are five here)."""
    B, torch = fx
    n, h, w, c, k = case
    net = Net(fx, dtype, n, (8, h, w), seed=sum(case))
    t = net.conv(net.conv(0, 24, 3), c, 1)
    net.ops.append(B.OpDesc(B.OP_AVGPOOL, t, -1, B.conv_shape(1, 1, 1, 1, 1, 0), None, 0, 1, 0, None, -1, 0))
    net.tensors.append(net.stored(net.tensors[t].mean((2, 3), keepdim=True)))
    net.conv(t + 1, k, 1, relu=bool(n & 1))
    net.check("mean_fc", None, "mean_fc")
    net.check("mean_fc", 0, "mean_fc", takes=False)


# channels in, rows, columns, images, filters of the 3 x 3 convolutions: (filters, stride, tensor that is added or -1, its
# stride).  Every size of work item of the row kernel, images that are not square, tiles of half rows
ROW_NETS = [
    (16, 6, 16, 2, [(24, 1, -1, 1), (24, 1, 1, 1)]),
    (8, 4, 48, 1, [(16, 1, -1, 1), (16, 1, 1, 1)]),
    (8, 2, 64, 3, [(16, 1, -1, 1)]),
    (16, 12, 8, 2, [(32, 1, -1, 1), (24, 1, -1, 1)]),
    (16, 8, 8, 2, [(32, 1, -1, 1), (64, 1, -1, 1), (50, 1, -1, 1), (64, 1, 2, 1)]),
    (16, 8, 16, 1, [(64, 1, -1, 1)]),
    (8, 12, 32, 2, [(16, 1, -1, 1), (32, 2, -1, 1), (32, 1, 1, 2), (20, 1, -1, 1)]),
    (20, 4, 96, 2, [(13, 1, -1, 1), (30, 2, -1, 1), (27, 1, -1, 1), (30, 1, 2, 1), (12, 1, -1, 1)]),
    (32, 16, 16, 1, [(48, 2, -1, 1), (41, 1, -1, 1), (48, 1, 1, 1)]),
]


def row_model(fx, net):
    """The model of a Net twice: as its kernel of row layers runs it, and tap by tap."""
    B, _ = fx
    models = []
    for rows in (None, 0):
        B.fupr_tuning_set("resident_rows", rows)
        try:
            models.append(B.Model(net.dt, net.in_shape, net.ops, net.blobs))
        finally:
            B.fupr_tuning_set("resident_rows", None)
    assert [m.launch_stats(net.n, 0)["kernel"] for m in models] == ["resident_network", "resident_network_taps"]
    return models


def with_mean(B, net, classes):
    """Net with a global mean and a layer behind it."""
    t = len(net.ops)
    net.ops.append(B.OpDesc(B.OP_AVGPOOL, t, -1, B.conv_shape(1, 1, 1, 1, 1, 0), None, 0, 1, 0, None, -1, 0))
    net.tensors.append(net.stored(net.tensors[t].mean((2, 3), keepdim=True)))
    net.conv(t + 1, classes, 1, relu=False)
    return net


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("case", ROW_NETS, ids=lambda c: "-".join(map(str, c[:4])))
def test_row_layers(fx, case, dtype):
    """Networks of row layers against their float64 evaluation and against the kernel that goes tap by tap (the bounds of
    Net.check: no more than nine stored tensors), the same bits every time."""
    B, torch = fx
    c, h, w, n, layers = case
    net = Net(fx, dtype, n, (c, h, w), seed=h * w + c)
    for i, (k, stride, add, add_stride) in enumerate(layers):
        net.conv(i, k, 3, stride=stride, add=add, add_stride=add_stride)
    with_mean(B, net, 10)
    xd = B.DeviceTensor.from_nchw(net.x, net.dt)
    outs = []
    for m in row_model(fx, net):
        for _ in range(2):
            out, ws = m.alloc(n)
            out.data.fill_(7.0)
            m.fupr_forward(xd, out, ws)
            torch.cuda.synchronize()
            assert out.padding_is_zero()
            outs.append(torch.from_numpy(np.ascontiguousarray(out.to_nchw())).double())
    assert torch.equal(outs[0], outs[1])
    unit = {"bf16": 2.0 ** -8, "f16": 2.0 ** -11}[dtype]
    for ref in (net.tensors[-1], outs[2]):
        assert float((outs[0] - ref).norm() / ref.norm()) <= 1.5 * unit
        assert float((outs[0] - ref).abs().max()) <= 4 * unit * float(ref.abs().max())


class Positive:
    """A generator whose normal numbers are all positive."""

    def __init__(self, seed):
        self.rng = np.random.default_rng(seed)

    def standard_normal(self, shape):
        return np.abs(self.rng.standard_normal(shape))


# channels in, rows, columns, stride: 1 - 8 chunks of channels a tap, each size of work item
INFINITE = ([(8 * c, 8, 16, 1) for c in range(1, 9)] + [(8 * c, 16, 16, 1) for c in range(1, 5)]
            + [(8 * c, 16, 32, 2) for c in range(1, 5)] + [(8, 32, 32, 2), (16, 32, 32, 2), (48, 8, 8, 1), (16, 16, 8, 1)])


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("case", INFINITE, ids=lambda c: "-".join(map(str, c)))
def test_row_layers_keep_infinities_to_their_window(fx, case, dtype):
    """With positive weights a pixel of -Inf makes -Inf of what sees it, or NaN, both 0 behind the ReLU; all else is as
    in a float64 evaluation.  One of +Inf makes +Inf; NaN only at stride 1 with 2 or 6 chunks a tap, where zeros that fill
    a step up meet a pixel of the same window."""
    B, torch = fx
    c, h, w, stride = case
    unit = {"bf16": 2.0 ** -8, "f16": 2.0 ** -11}[dtype]
    for relu in (True, False):
        for channel in (0, c - 1):
            for row, col in ((h // 2 + 1, 3), (h - 1, w - 1)):
                net = Net(fx, dtype, 2, (c, h, w), seed=h * w + c)
                net.rng = Positive(c)
                net.x[0, channel, row, col] = -np.inf if relu else np.inf
                net.tensors[0] = net.stored(torch.from_numpy(net.x).double())
                net.conv(0, 32, 3, stride=stride, relu=relu)
                with_mean(B, net, 10)
                m, _ = row_model(fx, net)
                out, ws = m.alloc(2)
                m.fupr_forward(B.DeviceTensor.from_nchw(net.x, net.dt), out, ws)
                torch.cuda.synchronize()
                got = np.ascontiguousarray(out.to_nchw())[:, :, 0, 0]
                want = net.tensors[-1].numpy()[:, :, 0, 0]
                at = (channel, row, col, got, want)
                if not relu:
                    seen = np.isinf(got[0]) | np.isnan(got[0]) if stride == 1 and c // 8 % 4 == 2 else got[0] == np.inf
                    assert seen.all() and (want[0] == np.inf).all(), at
                    got, want = got[1:], want[1:]
                assert np.abs(got - want).max() <= 4 * unit * np.abs(want).max(), at


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("relu", [False, True])
def test_mean_and_the_layer_behind_it_keep_what_is_no_number(fx, relu, dtype):
    """NaN and infinities come out of the one launch as out of the two.  Behind a ReLU NaN is 0 in either: one takes
    the larger of two numbers, the other of two 16-bit patterns, and every NaN of the matrix unit has a sign."""
    B, torch = fx
    net = Net(fx, dtype, 4, (512, 5, 3), seed=5)
    net.ops.append(B.OpDesc(B.OP_AVGPOOL, 0, -1, B.conv_shape(1, 1, 1, 1, 1, 0), None, 0, 1, 0, None, -1, 0))
    net.tensors.append(net.stored(net.tensors[0].mean((2, 3), keepdim=True)))
    net.conv(1, 130, 1, relu=relu)
    bias = net.blobs[-1].view(torch.int32)         # (the blob's first floats)
    bias[5], bias[77] = 0x7fc00000, 0xffc00000 - 2 ** 32
    m = B.Model(net.dt, net.in_shape, net.ops, net.blobs)
    assert B._lib.fupr_model_set_table(m._h, None) in (B.FUPR_OK, B.ERR_ARG)
    m.fuse_blocks(True)
    x = net.x.copy()
    x[0, 3, 2, 1] = np.nan
    x[1, 9, 4, 2] = np.inf
    x[2, 4, 0, 0] = x[2, 36, 4, 1] = np.inf        # channels of two steps, so of two waves
    xd = B.DeviceTensor.from_nchw(x, net.dt)
    got = []
    for switch in (None, 0):
        B.fupr_tuning_set("mean_fc", switch)
        try:
            assert (m.launch_stats(4, m.num_launches_at(4) - 1)["kernel"] == "mean_fc") == (switch is None)
            out, ws = m.alloc(4)
            m.fupr_forward(xd, out, ws)
            torch.cuda.synchronize()
        finally:
            B.fupr_tuning_set("mean_fc", None)
        got.append(np.ascontiguousarray(out.to_nchw())[:, :, 0, 0])
    one, two = got
    assert np.isnan(two[:, 6]).any() != relu and np.isnan(two[3, 5]) != relu and np.isinf(two[1]).any()
    assert np.array_equal(np.isnan(one), np.isnan(two))
    assert np.array_equal(np.isinf(one), np.isinf(two)) and np.array_equal(one[np.isinf(one)], two[np.isinf(two)])
    unit = {"bf16": 2.0 ** -8, "f16": 2.0 ** -11}[dtype]
    fine = np.delete(np.arange(130), (5, 77))
    assert np.abs(one[3] - two[3])[fine].max() <= 4 * unit * np.abs(two[3, fine]).max()
